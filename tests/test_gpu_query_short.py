"""GPU parity of dkv_query_attn on short blocks (at most 256 query rows per
segment), which take a kernel of their own: row counts at the edges of its
row and key waves, split and unsplit calls, and both load policies.

The probabilities of the P V product are two bf16 parts, each off by at most
2^-17 of itself with a sign that its key's scores set at random.  An output's
error then passes t * 2^-17 * sqrt(sum p^2 v^2) with probability 2 exp(-t^2 / 2)
(Hoeffding): t = 6.5 for the million outputs of these tests.  The values have
unit variance, so the outputs of a row scatter by sqrt(sum p^2), and the largest
of its 64 and more is below 1.3 times that in one row of a million: errors stay
below 6.5 / 1.3 * 2^-17 = 3.8e-5 of the row's largest output (measured 7.2e-6).
"""

import numpy as np
import pytest
import torch

from _helpers import row_rel_err
from test_gpu_query import _run, d  # noqa: F401  (d: the library fixture)

pytestmark = pytest.mark.gpu

TOL = 5 * 2.0 ** -17


@pytest.mark.parametrize("dim", [64, 128])
@pytest.mark.parametrize("G,n_q", [(1, 1), (16, 1), (16, 2), (1, 32), (1, 33), (4, 16), (5, 13), (8, 16), (3, 43),
                                   (16, 16), (1, 255), (7, 37)])
@pytest.mark.parametrize("T", [31, 700, 9000, 14000])
def test_row_edges(d, dim, G, n_q, T):  # noqa: F811
    """1 to 259 rows (the last one past the short kernels), keys from less
    than a tile to many slices per segment (blocks of more than 128 rows take
    the short kernel at 14,000 positions only), the block longer than a tile."""
    rng = np.random.default_rng([dim, G, n_q, T])
    got, want = _run(d, rng, 1, 3, G, T, dim, 0.6, 2, n_q, cap=n_q + 5)
    assert np.isfinite(got).all()
    assert row_rel_err(got.reshape(-1, dim), want.reshape(-1, dim)) <= TOL


@pytest.mark.parametrize("dim", [64, 128])
@pytest.mark.parametrize("G,n_q", [(4, 3), (4, 12), (4, 30), (4, 60)])
@pytest.mark.parametrize("hint", [1 << 20, 4096, 0], ids=["streamed", "few", "unknown"])
def test_hints(d, dim, G, n_q, hint):  # noqa: F811
    """A hint past the last-level cache's share selects the streamed loads, a
    small one few workgroups (long slices over several segments), none the
    widest split; some segments are empty."""
    rng = np.random.default_rng([7, n_q, hint % 1000])
    keep = rng.permutation(np.array([0.0, 0.02, 0.3, 0.9, 1.0, 0.5])).reshape(2, 3, 1)
    got, want = _run(d, rng, 2, 3, G, 5000, dim, keep, 1, n_q, hint=hint)
    assert row_rel_err(got.reshape(-1, dim), want.reshape(-1, dim)) <= TOL


@pytest.mark.parametrize("hint", [(1 << 63) - 1, (1 << 63) - 128, 1 << 40])
def test_largest_hints(d, hint):  # noqa: F811
    """Any positive hint is valid: the largest ones split the call as widely as
    a merely large one: 256 slices of the keys and a fixed cost of 384 keys per
    segment, of which at most 384 / 66 + 1 = 7 a segment hold no key (at least
    16,900 keys and costs in all), and one piece more per segment boundary."""
    seen = {}

    def inspect(ws, seg_len, rows_hint, wsb):
        meta = ws[:3 * 8].cpu().view(torch.int32).numpy().reshape(3, 2)
        seen["first"], seen["count"] = meta[:, 0], meta[:, 1]

    got, want = _run(d, np.random.default_rng(17), 1, 3, 4, 9000, 128, 0.6, 1, 3, hint=hint, inspect=inspect)
    assert row_rel_err(got.reshape(-1, 128), want.reshape(-1, 128)) <= TOL
    assert 256 - 3 * 7 <= seen["count"].sum() <= 258
    assert 0 <= seen["first"][0] <= 7 and (np.diff(seen["first"]) >= seen["count"][:-1]).all()


@pytest.mark.parametrize("nseg", [255, 256, 257, 511, 512, 513])
@pytest.mark.parametrize("G,n_q", [(2, 3), (4, 12), (4, 30)])
def test_many_segments(d, G, n_q, nseg):  # noqa: F811
    """Split calls about the edges of one and two segments per thread of the
    prefix (256 threads for up to 64 rows, 512 above), of one segment per
    workgroup (256) and of the short kernels (512); unequal segments, every
    fifth without context."""
    rng = np.random.default_rng([nseg, n_q])
    keep = rng.uniform(0.1, 1.0, size=(nseg, 1, 1))
    keep[::5] = 0.0
    seen = {}

    def inspect(ws, seg_len, rows_hint, wsb):
        seen["split"] = wsb > 0

    got, want = _run(d, rng, nseg, 1, G, 2500, 64, keep, 1, n_q, inspect=inspect)
    assert seen["split"]
    assert np.isfinite(got).all()
    assert row_rel_err(got.reshape(-1, 64), want.reshape(-1, 64)) <= TOL
