"""Tables of few queries: the workgroups of one subspace in a row, or those of one query, on both sides of the line between the two orders,
against fp64 products."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# (head, subspace) pairs in multiples of eight and not, sub-vectors of 4, 8, 10, 12, 16, 20, 32 and 64 coordinates; one query a workgroup and more;
# and more workgroups than a grid's last dimension takes
@pytest.mark.parametrize("d_k,m,H", [(8, 2, 3), (16, 4, 4), (8, 1, 5), (64, 8, 32), (80, 8, 5), (40, 4, 3), (24, 2, 4), (48, 4, 25), (48, 3, 3), (80, 4, 16),
                                     (160, 8, 32), (64, 4, 25), (80, 4, 25), (48, 3, 31), (32, 1, 7), (128, 4, 32), (64, 1, 3), (128, 2, 4)])
@pytest.mark.parametrize("B,T", [(1, 1), (5, 1), (3, 11), (255, 1)])
def test_either_order(d_k, m, H, B, T):
    check(d_k, m, H, B, T)


@pytest.mark.parametrize("d_sub", [24, 40])
def test_more_workgroups_than_the_last_dimension_takes(d_sub):
    check(d_sub, 1, 1, 1, 65536 * 16 + 5)


def check(d_k, m, H, B, T):
    import paper_2601_10155_amd as lk
    g = torch.Generator(device="cuda").manual_seed(d_k + H)
    cb = torch.randn(H, m, 256, d_k // m, device="cuda", generator=g)
    q = torch.randn(B, H, T, d_k, device="cuda", generator=g).half()
    got = lk.lookat_build_lut(q, cb)
    for t in range(0, T, 65536):           # (in pieces: fp64 products of a piece at a time)
        x = q[:, :, t:t + 65536].double().reshape(B, H, -1, m, d_k // m).transpose(2, 3)
        c = cb.double().transpose(-1, -2).contiguous()
        ref, size = (x @ c).transpose(2, 3), (x.abs() @ c.abs()).transpose(2, 3)
        # an fp32 chain of n products is within n 2^-24 of the summands' magnitude
        assert ((got[:, :, t:t + 65536].double() - ref).abs() <= (d_k // m + 1) * 2.0 ** -24 * size).all()
