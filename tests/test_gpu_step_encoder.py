"""The fused steps' encoder (fp32 ranking, the fp64 rule for what it cannot decide) where candidates are equal, nearly equal, not numbers or
outside the range of fp32 squares: the appended codes against the oracle, on every kernel that encodes."""
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


KINDS = 14


def head(kind, m, d, dtype, rng):
    """Codebook [m, 256, d] and key [m, d]."""
    c = rng.standard_normal((m, 256, d)).astype(np.float32)
    k = rng.standard_normal((m, d)).astype(np.float32)
    a, b = 37, (38 if kind == 1 else 37 + 64)
    if kind in (1, 2):                 # equal centroids in one wavefront's 64, and in two
        c[:, b] = c[:, a]
        k = c[:, b] + np.float32(1e-3)
    elif kind == 3:
        c[:] = 0.25                    # all equal
    elif kind in (4, 5):               # a key that is not a number, or infinite, in one subspace
        k[m // 2, 0] = np.nan if kind == 4 else np.inf
    elif kind in (6, 7):               # a centroid that is not a number: the first (nothing compares below it), another
        c[:, 0 if kind == 6 else 100, d - 1] = np.nan
    elif kind == 8:                    # squares below fp32's range
        c, k = c * np.float32(1e-27), k * np.float32(1e-27)
    elif kind == 9:                    # and beyond it
        c, k = c * np.float32(1e25), k * np.float32(1e4 if dtype == "float16" else 1e25)
    elif kind == 10:                   # halfway between two centroids that nothing else is near
        c[:, 3:] += 50
        c[:, 200], c[:, 5] = 1.5, -0.5
        k[:] = 0.5
    elif kind == 11:
        k[:] = 0
        c[:, 250:] = 0
    elif kind == 12:                   # within fp32's rounding of halfway
        c[:, 3:] += 50
        c[:, 70], c[:, 6] = 1 + rng.random((m, d), dtype=np.float32) * 1e-6, -1
        k[:] = 0
    elif kind == 13:
        c[:, 9] = np.inf
    return c, k.astype(dtype)


@pytest.mark.parametrize("d_k,m", [(d, m) for d in (64, 128) for m in (2, 4, 8, 16)])
@pytest.mark.parametrize("dtype", ["float16", "float32"])
# a compute unit each, whole and in ranges; two workgroups a compute unit, whole and in ranges; paired entries; grouped queries
@pytest.mark.parametrize("form", ["lone", "ranges", "many", "many ranges", "paired", "group2", "group4", "group8"])
@pytest.mark.parametrize("L", [1, 530])      # the new key in a first tile, in a second one
def test_new_codes(lk, d_k, m, dtype, form, L):
    group = int(form[5:]) if form.startswith("group") else 1
    if (group == 8 and m == 16 and d_k == 128) or (form == "paired" and d_k == 128 and m == 2):
        pytest.skip("no such instance")
    rng = np.random.default_rng(d_k + m)
    B, H = {"many": (1, 257), "many ranges": (1, 257), "paired": (2, KINDS)}.get(form, (1, KINDS))
    books, keys = zip(*(head(h % KINDS, m, d_k // m, dtype, rng) for h in range(KINDS)))
    cb = np.stack([books[h % KINDS] for h in range(H)])
    k = np.stack([np.stack([keys[h % KINDS].reshape(-1) for h in range(H)])] * B)
    codes = torch.full((B, H, L + 2, m), 0xEE, dtype=torch.uint8, device="cuda")
    v = torch.zeros((B, H, L + 2, d_k), dtype=torch.float16, device="cuda")
    q = torch.ones((B, H * group, d_k), dtype=getattr(torch, dtype), device="cuda")
    args = (q, dev(k), dev(cb), codes[:, :, :L], v[:, :, :L], 0.1)
    if group > 1:
        lk.lookat_decode_step_gqa(*args)
    elif form == "paired":
        lk.lookat_probe_decode_step_entries(2, *args)
    elif "ranges" in form:
        lk.lookat_decode_step_split(*args, num_splits=3)
    else:
        lk.lookat_decode_step(*args)
    ref = oracle.encode_keys(k[:, :KINDS, None], cb[:KINDS])[:, :, 0]
    got = codes.cpu().numpy()
    for h in range(0, H, 1 if H == KINDS else 15):
        assert np.array_equal(got[:, h, L - 1], ref[:, h % KINDS]), f"head {h}"
    assert (got[:, :, :L - 1] == 0xEE).all() and (got[:, :, L:] == 0xEE).all()
