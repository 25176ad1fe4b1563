"""Appends of a few keys and tables of a few queries, every number of keys that a workgroup takes and sub-vector lengths around the
pieces in which a centroid's row is read, against the oracle; tables of many queries for the longest sub-vectors of the matrix-core
kernel."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lk():
    import paper_2601_10155_amd as pkg
    pkg.load_library()
    return pkg


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# sub-vectors of 5, 12, 16, 20, 32, 36, 64, 80 and 136 coordinates; 1 to 9 keys of a head, one each or several of a sequence
@pytest.mark.parametrize("d_k,m", [(80, 16), (96, 8), (64, 4), (160, 8), (64, 2), (144, 4), (128, 2), (160, 2), (136, 1)])
@pytest.mark.parametrize("dtype", ["float16", "float32"])
@pytest.mark.parametrize("B,N", [(1, 1), (2, 1), (4, 1), (5, 1), (3, 3), (9, 4)])
def test_few_keys_and_queries(lk, d_k, m, dtype, B, N):
    rng = np.random.default_rng(d_k + m + B)
    cb = rng.standard_normal((3, m, 256, d_k // m)).astype(np.float32)
    cb[:, :, 200] = cb[:, :, 100]                                 # ties: the lower index
    x = rng.standard_normal((B, 3, N, d_k)).astype(dtype)
    x[0, 0, 0] = cb[0, :, 100].reshape(-1).astype(dtype)
    assert np.array_equal(lk.lookat_encode_keys(dev(x), dev(cb)).cpu().numpy(), oracle.encode_keys(x, cb))
    got = lk.lookat_build_lut(dev(x), dev(cb)).cpu().numpy()
    ref = oracle.build_lut(x, cb)
    size = np.abs(x.astype(np.float64).reshape(B, 3, N, m, 1, -1)) @ np.abs(cb.astype(np.float64))[None, :, None].swapaxes(-1, -2)
    # an fp32 chain of n products is within n 2^-24 of the summands' magnitude (and the oracle rounds once more)
    assert (np.abs(got - ref.reshape(got.shape)) <= (d_k // m + 1) * 2.0 ** -24 * size.reshape(got.shape)).all()


@pytest.mark.parametrize("d_k,m", [(64, 2), (128, 4), (128, 2)])
@pytest.mark.parametrize("B,T", [(1, 256), (3, 101), (2, 300)])   # whole tiles of 32 queries, tiles across batch entries, a ragged end
@pytest.mark.parametrize("dtype", ["float16", "float32"])
def test_tables_of_long_sub_vectors(lk, d_k, m, B, T, dtype):
    rng = np.random.default_rng(d_k + T)
    cb = rng.standard_normal((2, m, 256, d_k // m)).astype(np.float32)
    q = rng.standard_normal((B, 2, T, d_k)).astype(dtype)
    got = lk.lookat_build_lut(dev(q), dev(cb)).cpu().numpy()
    x = q.astype(np.float64).reshape(B, 2, T, m, 1, -1)
    c = cb.astype(np.float64)[None, :, None].swapaxes(-1, -2)
    ref, size = (x @ c).reshape(got.shape), (np.abs(x) @ np.abs(c)).reshape(got.shape)
    assert (np.abs(got - ref) <= (d_k // m + 1) * 2.0 ** -24 * size).all()


def test_few_tables_of_long_sub_vectors_stay_on_the_vector_kernel(lk):
    """One head, one subspace of 64: 256 queries take as long as 255 (4 us; 8 on the matrix cores)."""
    g = torch.Generator(device="cuda").manual_seed(1)
    cb = torch.randn((1, 1, 256, 64), generator=g, device="cuda")
    q = torch.randn((1, 1, 256, 64), generator=g, device="cuda").half()
    e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    best = {}
    for _ in range(12):
        for T in (255, 256):
            x, out = q[:, :, :T].contiguous(), torch.empty((1, 1, T, 1, 256), device="cuda")
            e[0].record()
            for _ in range(50):
                lk.lookat_build_lut(x, cb, lut_out=out)
            e[1].record()
            torch.cuda.synchronize()
            best[T] = min(best.get(T, 1e9), e[0].elapsed_time(e[1]))
    assert best[256] < 1.45 * best[255], best


# around 768 tables, from which the matrix cores take over; at 300 queries either side
@pytest.mark.parametrize("H,T,d_k,m", [(1, 256, 64, 1), (3, 256, 64, 1), (1, 769, 64, 1), (1, 383, 64, 2), (1, 385, 64, 2), (3, 300, 128, 2), (4, 300, 128, 4)])
@pytest.mark.parametrize("dtype", ["float16", "float32"])
def test_tables_have_the_bits_of_smaller_calls(lk, H, T, d_k, m, dtype):
    g = torch.Generator(device="cuda").manual_seed(T + d_k)
    cb = torch.randn((H, m, 256, d_k // m), generator=g, device="cuda")
    q = torch.randn((1, H, T, d_k), generator=g, device="cuda").to(getattr(torch, dtype))
    pieces = [lk.lookat_build_lut(q[:, :, t:t + 200].contiguous(), cb) for t in range(0, T, 200)]
    assert torch.equal(lk.lookat_build_lut(q, cb), torch.cat(pieces, 2))


@pytest.mark.parametrize("H,d_k,m,Nc", [(33, 64, 16, 4099), (35, 64, 8, 1030), (3, 64, 16, 1024), (3, 64, 16, 1025), (129, 24, 8, 70),
                                         (129, 16, 8, 4099), (3, 24, 8, 1000)])
def test_learning_with_the_smaller_workgroup(lk, H, d_k, m, Nc):
    """One or two pieces of four coordinates (single ones in the last two) per workgroup, with more workgroups than compute units or few
    keys; (129, 24, 8, 70) has three pieces per workgroup, and 1024 threads."""
    rng = np.random.default_rng(H + Nc)
    cb = rng.standard_normal((H, m, 256, d_k // m)).astype(np.float32)
    calib = rng.standard_normal((H, Nc, d_k)).astype(np.float32)
    ref, _ = oracle.kmeans_step(calib, cb)
    got, _ = lk.lookat_kmeans_step(dev(calib), dev(cb))
    assert np.array_equal(got.cpu().numpy(), ref)
