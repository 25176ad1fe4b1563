"""Causal scores of long blocks, whose score rows are dealt to workgroups in strips: every entry against the products in
float64, with memory around the scores watched."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lk():
    import paper_2601_10155_amd as pkg
    pkg.load_library()
    return pkg


# B, H, T, L: a strip with one query more or less, strips that no key of a panel is visible to, more than three strips, launches that
# fill the chip and that do not, L odd (scalar stores), heads that are no multiple of the 8 dies
@pytest.mark.parametrize("d_k,m", [(128, 16), (128, 2), (64, 8), (64, 4)])
@pytest.mark.parametrize("dtype,B,H,T,L", [("float16", 1, 3, 769, 769), ("float16", 2, 33, 513, 640), ("float32", 1, 9, 1100, 1101),
                                           ("float16", 1, 2, 300, 2000), ("float16", 1, 17, 1030, 1536), ("float32", 1, 3, 257, 260),
                                           ("float16", 1, 33, 2049, 2052), ("float32", 1, 40, 512, 1024)])
def test_strips(lk, d_k, m, dtype, B, H, T, L):
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
