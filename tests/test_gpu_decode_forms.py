"""Attention decode at head sizes between the kernels' own (padded to the next one) and at subspace counts without a vector
load, on views of longer caches, with memory around the output watched."""
import math

import numpy as np
import pytest
import torch

import oracle
from bars import assert_out_close, assert_scores_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lk():
    import paper_2601_10155_amd as pkg
    pkg.load_library()
    return pkg


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# head sizes at both ends of each padded range; m with and without a vector load, up to 32
@pytest.mark.parametrize("d_k,m", [(8, 2), (24, 3), (40, 8), (56, 7), (72, 4), (96, 8), (96, 32), (112, 16), (120, 1), (136, 2),
                                   (160, 10), (248, 31), (248, 8), (64, 32), (32, 1), (256, 32)])
@pytest.mark.parametrize("L,splits", [(1, 0), (64, 1), (193, 0), (500, 7), (2501, 0), (4200, 1)])
def test_decode_padded_head_sizes(lk, d_k, m, L, splits):
    rng = np.random.default_rng(d_k * 100 + m + L)
    B, H, Lmax = 2, 3, L + 5
    lut = rng.standard_normal((B, H, m, 256)).astype(np.float32)
    codes = rng.integers(0, 256, size=(B, H, Lmax, m), dtype=np.uint8)
    v = rng.standard_normal((B, H, Lmax, d_k)).astype(np.float16)
    v[:, :, L:] = np.nan     # rows past the context must not count
    scale = 1.0 / math.sqrt(d_k)
    ref, s_ref = oracle.attend_decode(lut, codes[:, :, :L], v[:, :, :L], scale, want_scores=True)
    n = B * H * d_k
    guard = torch.full((n + 512,), 7.0, device="cuda")
    out = guard[256:256 + n].view(B, H, d_k)
    scores = torch.empty((B, H, L), dtype=torch.float32, device="cuda")
    lk.lookat_attend_decode(dev(lut), dev(codes)[:, :, :L], dev(v)[:, :, :L], scale, num_splits=splits, out=out, scores_out=scores)
    assert_out_close(out.cpu().numpy(), ref, "attend_decode, padded head sizes", s_ref, scale)
    assert_scores_close(scores.cpu().numpy(), lut, codes[:, :, :L], s_ref)
    assert bool((guard[:256] == 7.0).all()) and bool((guard[256 + n:] == 7.0).all())


@pytest.mark.parametrize("m", [2, 4, 8, 16])
@pytest.mark.parametrize("L,dtype", [(1, "float16"), (64, "float16"), (513, "float32"), (1100, "float16"), (2065, "float32")])
def test_fused_step_lone_workgroups(lk, m, L, dtype):
    """d_k = 128: up to 256 (b,h) take the instance for workgroups that have a compute unit to themselves (whole tiles
    requested, the next one in flight), 257 the other; both add in the same order, so equal inputs give equal bits."""
    H, d_k = 257, 128
    assert lk.decode_step_entries_per_workgroup(1, H, d_k, m, L) == 1
    g = torch.Generator(device="cuda").manual_seed(m * 10000 + L)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    cb, q, k = rnd(H, m, 256, d_k // m), rnd(1, H, d_k).to(getattr(torch, dtype)), rnd(1, H, d_k).to(getattr(torch, dtype))
    codes = torch.randint(0, 256, (1, H, L + 3, m), generator=g, device="cuda", dtype=torch.uint8)
    v = rnd(1, H, L + 3, d_k).half()
    c1, c2 = codes.clone(), codes.clone()
    many = lk.lookat_decode_step(q, k, cb, c1[:, :, :L], v[:, :, :L], 0.3)
    lone = lk.lookat_decode_step(q[:, :256].contiguous(), k[:, :256].contiguous(), cb[:256], c2[:, :256, :L], v[:, :256, :L], 0.3)
    assert torch.equal(many[:, :256], lone)
    assert torch.equal(c1[:, :256], c2[:, :256]) and torch.equal(c2[:, 256], codes[:, 256])
