"""Appends of a few keys where the number of workgroups decides how many keys each of them takes: both sides of the line, every number of keys
and a last workgroup that is not full, against the oracle's codes."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


# One key a workgroup up to 512 workgroups (256 for sub-vectors longer than 16), then two, four, eight.
@pytest.mark.parametrize("d_k,m,H", [(64, 8, 64), (80, 8, 64), (96, 8, 16), (128, 8, 64), (160, 8, 32), (144, 4, 64), (64, 2, 128)])
@pytest.mark.parametrize("B", [1, 2, 3, 4, 5, 9])
def test_keys_per_workgroup(d_k, m, H, B):
    import paper_2601_10155_amd as lk
    rng = np.random.default_rng(d_k + B)
    cb = rng.standard_normal((H, m, 256, d_k // m)).astype(np.float32)
    cb[:, :, 200] = cb[:, :, 100]                                 # ties: the lower index
    for dtype in ("float16", "float32"):
        x = rng.standard_normal((B, H, 1, d_k)).astype(dtype)
        x[B - 1, 0, 0] = cb[0, :, 100].reshape(-1).astype(dtype)
        dev = [torch.from_numpy(a).cuda() for a in (x, cb)]
        assert np.array_equal(lk.lookat_encode_keys(*dev).cpu().numpy(), oracle.encode_keys(x, cb))
