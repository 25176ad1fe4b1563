"""Causal scores of short blocks of queries on the kernel that keeps the codebook in LDS: every entry of the block against
the products in float64, at the edges of its query groups, key blocks and shares, with memory around the scores watched."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lk():
    import paper_2601_10155_amd as pkg
    pkg.load_library()
    return pkg


# B, H, T, L: one key, ragged 16- and 32-key blocks, L odd (scalar stores), T at the ends of groups of 16 and of the range
# per dtype, more batch entries than shares, heads that are no multiple of the 8 dies, wavefronts whose share spans batch
# entries, blocks that no query sees (T close to L)
@pytest.mark.parametrize("d_k,m", [(128, 16), (128, 8), (128, 4), (128, 2), (64, 16), (64, 8), (64, 4), (64, 2)])
@pytest.mark.parametrize("dtype,B,H,T,L", [("float16", 1, 3, 1, 1), ("float16", 2, 5, 5, 33), ("float16", 3, 1, 8, 500),
                                           ("float16", 1, 9, 16, 1031), ("float16", 2, 8, 17, 200), ("float16", 11, 2, 23, 100),
                                           ("float16", 2, 3, 23, 23), ("float16", 2, 12, 32, 9001), ("float16", 4, 13, 24, 4096),
                                           ("float32", 2, 12, 24, 9000), ("float32", 4, 13, 50, 4100), ("float32", 1, 8, 64, 26001)])
def test_short_blocks(lk, d_k, m, dtype, B, H, T, L):
    g = torch.Generator(device="cuda").manual_seed(d_k + m + T + L)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    cb = rnd(H, m, 256, d_k // m) * torch.logspace(-2, 2, m, device="cuda")[None, :, None, None]   # subspaces of unequal size
    q = (rnd(B, H, T, d_k) / 8).to(getattr(torch, dtype))
    codes = torch.randint(0, 256, (B, H, L + 3, m), generator=g, device="cuda", dtype=torch.uint8)[:, :, :L]
    n = B * H * T * L
    guard = torch.full((n + 128,), 7.0, device="cuda")
    out = guard[64:64 + n].view(B, H, T, L)
    lk.lookat_score_prefill(q, cb, codes, scores_out=out)
    assert bool((guard[:64] == 7.0).all()) and bool((guard[64 + n:] == 7.0).all())
    sub = torch.arange(m, device="cuda")
    unseen = torch.arange(L, device="cuda")[None, :] > torch.arange(L - T, L, device="cuda")[:, None]
    for b in range(B):
        for h in range(H):
            keys = cb[h][sub, codes[b, h].long()].reshape(L, d_k).double()
            ref = q[b, h].double() @ keys.t()
            bar = 1e-4 * (q[b, h].double().abs() @ keys.abs().t())
            got = out[b, h].double()
            assert bool((torch.isinf(got) & (got < 0) == unseen).all())
            assert bool(((got - ref).abs() <= bar)[~unseen].all())
