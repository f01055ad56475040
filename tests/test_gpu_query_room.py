"""Query blocks over a packed cache whose unused rows hold NaN: the free rows
behind every segment, and what lies before the first and after the last.  No
row past a segment's own keys may reach a product (0 * NaN is NaN), whichever
kernel takes the block and wherever its last tile ends."""

import numpy as np
import pytest
import torch

import oracle as o
from _helpers import bits, row_rel_err
from test_gpu_query import _bf16, d  # noqa: F401  (d: the library fixture)

pytestmark = pytest.mark.gpu

DEV = "cuda"


@pytest.mark.parametrize("dim", [64, 128])
@pytest.mark.parametrize("G,n_q", [(1, 1), (4, 8), (3, 20), (8, 16), (4, 60), (4, 70), (8, 40)])
@pytest.mark.parametrize("keys", [[0, 5, 33], [63, 1000, 95], [9001, 8999, 12345]], ids=["few", "unsplit", "split"])
def test_rows_past_a_segment(d, dim, G, n_q, keys):  # noqa: F811
    """Segments of unequal lengths with 70 free rows behind each (two tiles of
    the short kernels, more than one of the long)."""
    rng = np.random.default_rng([dim, G, n_q, keys[0]])
    Hkv, room = len(keys), n_q + 70
    scale = 1.0 / np.sqrt(dim)
    off = 64 + np.concatenate([[0], np.cumsum(np.array(keys) + room)])
    rows = int(off[-1]) + 64
    k = torch.full((rows, dim), float("nan"), dtype=torch.bfloat16)
    v = torch.full((rows, dim), float("nan"), dtype=torch.bfloat16)
    for s, n in enumerate(keys):
        k[off[s]:off[s] + n + n_q] = _bf16(rng, (n + n_q, dim))
        v[off[s]:off[s] + n + n_q] = _bf16(rng, (n + n_q, dim))
    q = _bf16(rng, (1, n_q, Hkv * G, dim))
    total = sum(keys) + Hkv * n_q
    need = d.dkv_query_workspace_bytes(1, Hkv * G, Hkv, dim, n_q, total)
    assert (need > 0) == (keys[0] == 9001)
    out = torch.full((1, n_q, Hkv * G, dim), float("nan"), dtype=torch.float32, device=DEV)
    so, sl = torch.tensor(off[:-1], dtype=torch.int64), torch.tensor(keys, dtype=torch.int32)
    d.dkv_query_attn(q.to(DEV), 0, room, k.to(DEV), v.to(DEV), so.to(DEV), sl.to(DEV), scale, out,
                     torch.empty(need, dtype=torch.uint8, device=DEV) if need else None, Hkv, rows_hint=total)
    got = out.cpu().numpy()
    assert np.isfinite(got).all()
    want = o.query_attn(bits(q), bits(k.nan_to_num(0.0)), bits(v.nan_to_num(0.0)), so.numpy(), sl.numpy(), 0, scale,
                        Hkv, o.BF16)
    # probabilities in two bf16 parts, as in test_gpu_query_short: sqrt(keys) * 2^-17
    assert row_rel_err(got.reshape(-1, dim), want.reshape(-1, dim)) <= np.sqrt(max(keys) + n_q) * 2.0 ** -17
