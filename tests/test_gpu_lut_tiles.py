"""Tables of many queries per head (matrix-core kernel): every entry against the products in float64 where 32-query tiles span
batch entries, end ragged or hold one query of each, with memory around the tables watched."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_k,m", [(64, 4), (64, 8), (64, 16), (64, 32), (256, 16)])
@pytest.mark.parametrize("dtype", ["float16", "float32"])
@pytest.mark.parametrize("B,H,T", [(257, 3, 1), (11, 2, 31), (9, 3, 33), (1, 2, 287), (4, 1, 64), (3, 5, 100)])
def test_table_tiles(d_k, m, dtype, B, H, T):
    import paper_2601_10155_amd as lk
    lk.load_library()
    g = torch.Generator(device="cuda").manual_seed(d_k + m + B + T)
    d_sub = d_k // m
    q = torch.randn(B, H, T, d_k, generator=g, device="cuda").to(getattr(torch, dtype))
    cb = torch.randn(H, m, 256, d_sub, generator=g, device="cuda")
    n = B * H * T * m * 256
    guard = torch.full((n + 128,), 7.0, device="cuda")
    out = guard[64:64 + n].view(B, H, T, m, 256)
    lk.lookat_build_lut(q, cb, lut_out=out)
    assert bool((guard[:64] == 7.0).all()) and bool((guard[64 + n:] == 7.0).all())
    qs = q.double().view(B, H, T, m, 1, d_sub)
    for i in range(m):       # products and sums of d_sub of them in fp32: at most d_sub roundings of 2^-24 each
        c = cb[:, i].double().view(1, H, 1, 256, d_sub)
        ref, mag = (qs[:, :, :, i] * c).sum(-1), (qs[:, :, :, i] * c).abs().sum(-1)
        assert bool(((out[:, :, :, i].double() - ref).abs() <= d_sub * 2.0 ** -24 * mag).all())
