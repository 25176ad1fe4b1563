"""Codebook updates of sets that end at, before and behind the edge of a chunk of 4096 keys (from the second chunk on, its lists are built while the
members of the one before are fetched), with clusters from none to all of the keys, bit for bit against the oracle."""
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


# four pieces of 16 coordinates in one workgroup, one piece (512 threads), several workgroups per subspace, lengths that are no multiple of four
@pytest.mark.parametrize("H,d_k,m", [(2, 64, 4), (24, 64, 16), (1, 128, 2), (2, 40, 4)])
@pytest.mark.parametrize("N", [4095, 4096, 4097, 4160, 8192, 12289])
def test_updates_at_the_edges_of_chunks(lk, H, d_k, m, N):
    rng = np.random.default_rng(N + d_k)
    cb = rng.standard_normal((H, m, 256, d_k // m)).astype(np.float32)
    cb[:, :, 128:] += 100                                        # centroids without members
    x = rng.standard_normal((H, N, d_k)).astype(np.float32)
    x[0, :, :d_k // m] = cb[0, 0, 7] + x[0, :, :d_k // m] * 1e-3  # one centroid with all of them
    got, assign = lk.lookat_kmeans_step(torch.from_numpy(x).cuda(), torch.from_numpy(cb).cuda())
    assert np.array_equal(assign.cpu().numpy(), oracle.encode_keys(x[None], cb)[0])
    assert np.array_equal(got.cpu().numpy(), oracle.kmeans_step(x, cb)[0])
