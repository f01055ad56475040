"""dkv_topk_pattern where its launch changes: entries just below, at and above
64 workgroups' chunks of 4,096 (histogram copies from there on), ragged ends,
whole groups of iterations and parts of one, and more entries than 1,024
workgroups' first groups hold.  Exact."""

import numpy as np
import pytest
import torch

import oracle as o

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1, 63 * 4096), (1, 1, 63 * 4096 + 1), (1, 3, 87381 + 7), (7, 11, 13),
                                   (1, 1, 1023), (1, 2, 512), (1, 1, 3073), (1, 1, 4095), (1, 1, 4096), (1, 1, 4097),
                                   (1, 3, 2731), (5, 64, 16381)])
@pytest.mark.parametrize("levels", [5, 1024, 1 << 30])
def test_export_launch_sizes(shape, levels):
    import paper_2609_32663_amd as d
    n = int(np.prod(shape))
    rng = np.random.default_rng([n, levels])
    p = (rng.integers(0, levels, size=shape) / levels).astype(np.float32)
    p.reshape(-1)[rng.integers(0, n, size=9)] = np.nan
    probs = torch.from_numpy(p).cuda()
    for k in (1, n // 5, n - 3):
        pat = torch.full(shape, 7, dtype=torch.uint8, device="cuda")
        ws = torch.full((d.dkv_topk_workspace_bytes(*shape),), 0x5A, dtype=torch.uint8, device="cuda")
        d.dkv_topk_pattern(probs, k, pat, ws)
        np.testing.assert_array_equal(pat.cpu().numpy(), o.topk_mask(p, k))
