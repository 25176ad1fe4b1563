"""Cache fills for every form of the ranking encoder (two sizes of workgroup, one or two fp16 terms per value, notes of undecided keys that
fill up and are worked off in between) against the exact scan of all centroids, code for code."""
import pytest
import torch

pytestmark = pytest.mark.gpu

H = 2


@pytest.fixture(scope="module")
def lk():
    import paper_2601_10155_amd as pkg
    pkg.load_library()
    return pkg


def _inputs(kind, d_sub, M, B, N, dtype, H=H):
    g = torch.Generator(device="cuda").manual_seed(d_sub + N)
    cb = torch.randn((H, M, 256, d_sub), generator=g, device="cuda")
    keys = torch.randn((B, H, N, M, d_sub), generator=g, device="cuda")
    if kind == "near ties":         # every other key between two centroids, 0 to 1e-3 of their distance off the middle
        i = torch.randint(0, 256, (2, B, H, N, M, 1), generator=g, device="cuda")
        rows = [cb.view(1, H, 1, M, 256, d_sub).expand(B, H, 1, M, 256, d_sub).permute(0, 1, 3, 2, 4, 5).reshape(B, H, M, 256, d_sub)
                .gather(3, j.permute(0, 1, 3, 2, 4).expand(B, H, M, N, d_sub)).permute(0, 1, 3, 2, 4) for j in i]
        off = torch.tensor([0.0, 1e-8, 1e-6, 1e-4, 1e-3], device="cuda")[torch.randint(0, 5, (B, H, N, 1, 1), generator=g, device="cuda")]
        keys[:, :, 1::2] = (rows[0] * (0.5 + off) + rows[1] * (0.5 - off))[:, :, 1::2]
    elif kind == "pairs of centroids":   # every key has two equally near ones: the lower index, and none is ever decided
        cb[:, :, 1::2] = cb[:, :, 0::2]
    elif kind == "repeated keys":   # the same with few values: zeros, -0.0 once, two others, NaN, and one key in eight of its own
        cb[:, :, 1::2] = cb[:, :, 0::2]
        few = torch.stack([torch.zeros_like(keys[:, :, 0]), keys[:1, :, 0].expand_as(keys[:, :, 0]), keys[:1, :, 1].expand_as(keys[:, :, 0]),
                           torch.full_like(keys[:, :, 0], float("nan"))])
        which = torch.tensor([0, 0, 0, 1, 1, 2, 3], device="cuda")
        for j in range(7):
            keys[:, :, j::8] = few[which[j]][:, :, None]
        keys[:, :, 8:9] = -0.0
    elif kind == "filler":          # no scale serves this codebook: every centroid is a candidate for every key
        cb[:, :, 200:] = 1e30
    elif kind == "magnitudes":      # norms over six orders of magnitude
        cb *= torch.tensor([1.0, 1e-3, 1e-6], device="cuda")[torch.randint(0, 3, (H, M, 256, 1), generator=g, device="cuda")]
        keys *= torch.tensor([1.0, 1e-3], device="cuda")[torch.randint(0, 2, (B, H, N, 1, 1), generator=g, device="cuda")]
    elif kind == "far keys":
        keys *= 300.0
    elif kind == "subnormal keys":  # fp16 keys below 2^-14
        cb *= 1e-5
        keys *= 1e-5
    return keys.view(B, H, N, M * d_sub).to(getattr(torch, dtype)), cb.contiguous()


# every length up to 64 that a head size can have; few pairs per wavefront (two terms of everything) and many, a ragged last block
@pytest.mark.parametrize("d_sub", [d for d in range(2, 65) if d % 4 == 0 or d % 2 == 0 or d <= 31])
@pytest.mark.parametrize("dtype", ["float16", "float32"])
@pytest.mark.parametrize("N", [797, 30001])
def test_every_length_matches_the_exact_scan(lk, monkeypatch, N, d_sub, dtype):
    m = 8 if d_sub % 2 else (4 if d_sub % 4 else 2)
    keys, cb = _inputs("near ties", d_sub, m, 1, N, dtype)
    keys[0, 0, 5, 0] = float("nan")
    keys[0, 1, 6, d_sub - 1] = float("inf")
    keys[0, 0, N - 1, m * d_sub - 1] = -float("inf")                # the last element of a slab
    got = lk.lookat_encode_keys(keys, cb).clone()
    monkeypatch.setenv("LOOKAT_ENCODE_EXACT", "1")
    ref = lk.lookat_encode_keys(keys, cb)
    assert torch.equal(got, ref), f"{int((got != ref).sum())} of {ref.numel()} codes differ"


# sub-vectors that fill an operand and sub-vectors that are padded: 512 threads, 256 with up to four coordinates (3 x 20011 keys of 12 to 32: 256
# in two terms).  Ten pairs of key blocks per wavefront: 640 notes where none is decided.
@pytest.mark.parametrize("d_sub", [3, 4, 7, 8, 12, 16, 24, 32, 48, 64])
@pytest.mark.parametrize("dtype", ["float16", "float32"])
@pytest.mark.parametrize("kind,B,N", [("near ties", 1, 90001), ("near ties", 3, 66671), ("pairs of centroids", 1, 300001),
                                      ("repeated keys", 1, 300001), ("repeated keys", 3, 20011),
                                      ("filler", 1, 300001), ("magnitudes", 1, 200001), ("far keys", 1, 90001),
                                      ("subnormal keys", 1, 200001)])
def test_large_fills_match_the_exact_scan(lk, monkeypatch, kind, B, N, d_sub, dtype):
    m = 8 if d_sub % 2 else 2       # (head sizes are multiples of 8)
    keys, cb = _inputs(kind, d_sub, m, B, N * 2 // m, dtype)
    got = lk.lookat_encode_keys(keys, cb).clone()
    monkeypatch.setenv("LOOKAT_ENCODE_EXACT", "1")
    ref = lk.lookat_encode_keys(keys, cb)
    assert torch.equal(got, ref), f"{int((got != ref).sum())} of {ref.numel()} codes differ"


def _compare(lk, monkeypatch, keys, cb):
    got = lk.lookat_encode_keys(keys, cb).clone()
    monkeypatch.setenv("LOOKAT_ENCODE_EXACT", "1")
    ref = lk.lookat_encode_keys(keys, cb)
    assert torch.equal(got, ref), f"{int((got != ref).sum())} of {ref.numel()} codes differ"


# 17 to 33 pairs per wavefront where none, or few different keys, are decided: more than the 832 notes hold
@pytest.mark.parametrize("d_sub,m,heads,N", [(3, 8, 2, 200003), (4, 16, 2, 200003), (16, 16, 32, 4155), (32, 8, 64, 5180), (64, 4, 128, 5690)])
@pytest.mark.parametrize("dtype", ["float16", "float32"])
@pytest.mark.parametrize("kind", ["pairs of centroids", "repeated keys"])
def test_notes_of_small_workgroups_fill_up(lk, monkeypatch, kind, d_sub, m, heads, N, dtype):
    _compare(lk, monkeypatch, *_inputs(kind, d_sub, m, 1, N, dtype, heads))


# 5 to 8 coordinates: 256 threads, one term; fp32 keys also in two terms (129 (head, subspace) pairs, 17 pairs of key blocks)
@pytest.mark.parametrize("d_sub,m,heads,N", [(7, 8, 48, 1500), (8, 8, 40, 700), (8, 1, 129, 1080), (6, 4, 33, 1080)])
@pytest.mark.parametrize("dtype", ["float16", "float32"])
@pytest.mark.parametrize("kind", ["near ties", "repeated keys"])
def test_forms_of_short_sub_vectors(lk, monkeypatch, kind, d_sub, m, heads, N, dtype):
    _compare(lk, monkeypatch, *_inputs(kind, d_sub, m, 1, N, dtype, heads))
