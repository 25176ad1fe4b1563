"""The library's choice of ranges per (b,h): what it promises about workspaces and callers that bring none."""
import ctypes
import math

import numpy as np
import pytest


def _lk():
    import paper_2601_10155_amd as pkg
    pkg.load_library()
    return pkg


def test_auto_splits_invariants():
    lk = _lk()
    for d_k, m in ((32, 4), (64, 4), (96, 8), (128, 8), (256, 16)):
        for BH in (1, 7, 12, 32, 64, 100, 128, 129, 200, 256, 257, 264, 300, 384, 520, 1000, 5000):
            for L in (1, 64, 300, 1024, 2048, 3000, 8192, 32768):
                S = lk.attend_decode_auto_splits(1, BH, d_k, m, L)
                assert 1 <= S <= 256 and (S == 1 or L >= 256 * S) and BH * S <= max(BH, 4096)
                if 128 < BH <= 256 or L < 512:
                    assert S == 1
                assert lk.attend_decode_workspace_bytes(1, BH, d_k, m, L) == (0 if S == 1 else BH * S * (d_k + 2) * 4)
                assert lk.attend_decode_gqa_workspace_bytes(1, BH, 1, d_k, m, L) == lk.attend_decode_workspace_bytes(1, BH, d_k, m, L)
    for group, fill in ((2, 512), (4, 256), (8, 256)):        # grouped queries: ranges of at least 1024 keys
        for BH in (1, 3, 32, 64, 200, 300, 600):
            for L, most in ((1, 1), (1024, 1), (1025, 2), (2047, 2), (2048, 2), (2049, 3), (4096, 4), (300000, 256)):
                S = min(most, max(1, fill // BH))
                assert lk.attend_decode_gqa_workspace_bytes(1, BH, group, 64, 4, L) == (0 if S == 1 else BH * group * S * 66 * 4)
    # no die (all ranges of a (b,h) share one of the eight, with 32 compute units) gets a few workgroups more than it runs at once
    for BH in range(1, 33):
        for d_k, m in ((32, 4), (64, 4), (128, 8)):
            for L in (4096, 6144, 8192, 16000, 32768):
                on_a_die = (BH + 7) // 8 * lk.attend_decode_auto_splits(1, BH, d_k, m, L)
                assert on_a_die <= 32 or on_a_die >= 48, (BH, d_k, L, on_a_die)
    assert [lk.attend_decode_auto_splits(1, BH, 128, 8, 32768) for BH in (1, 2, 4, 9, 20)] == [32, 32, 32, 16, 8]
    assert lk.attend_decode_auto_splits(1, 80, 64, 4, 4096) >= 2 and lk.attend_decode_auto_splits(1, 128, 32, 4, 8192) >= 2
    # long contexts of few pairs are cut, a little over one workgroup per compute unit too
    assert lk.attend_decode_auto_splits(1, 32, 128, 8, 8192) == 8
    assert lk.attend_decode_auto_splits(1, 264, 128, 8, 8192) > 1


@pytest.mark.gpu
@pytest.mark.parametrize("B,H,L", [(1, 3, 2048), (11, 24, 4133)])
def test_auto_splits_without_a_workspace(B, H, L):
    """Where one range needed no workspace, a call that brings none is still taken (with one range), and the library's
    choice gives the same result to the bar of the split count tests."""
    import torch
    from paper_2601_10155_amd.binding import _Shape, load_library
    lk = _lk()
    lib = load_library()
    d_k, m = 128, 8
    assert lk.attend_decode_auto_splits(B, H, d_k, m, L) > 1
    g = torch.Generator(device="cuda").manual_seed(B * L)
    lut = torch.randn((B, H, m, 256), generator=g, device="cuda")
    codes = torch.randint(0, 256, (B, H, L, m), generator=g, device="cuda", dtype=torch.uint8)
    v = torch.randn((B, H, L, d_k), generator=g, device="cuda").half()
    scale = 1.0 / math.sqrt(d_k)
    ref = lk.lookat_attend_decode(lut, codes, v, scale, num_splits=1)
    assert float((lk.lookat_attend_decode(lut, codes, v, scale) - ref).abs().max()) <= 2e-5
    out = torch.empty_like(ref)
    shape = _Shape(B, H, d_k, m, 256)
    rc = lib.lookat_attend_decode(ctypes.byref(shape), L, lut.data_ptr(), codes.data_ptr(), L * m, v.data_ptr(), L * d_k, scale, 0,
                                  None, 0, out.data_ptr(), None, torch.cuda.current_stream().cuda_stream)
    assert rc == 0 and torch.equal(out, ref)
    lk.lookat_attend_decode_noalloc(lut, codes, v, scale, out)
    assert torch.equal(out, lk.lookat_attend_decode(lut, codes, v, scale))

    cb = torch.randn((H, m, 256, d_k // m), generator=g, device="cuda")
    q, k = torch.randn((B, H, d_k), generator=g, device="cuda"), torch.randn((B, H, d_k), generator=g, device="cuda")
    one = lk.lookat_decode_step(q, k, cb, codes, v, scale)
    assert float((lk.lookat_decode_step_split(q, k, cb, codes, v, scale) - one).abs().max()) <= 2e-5
    rc = lib.lookat_decode_step_split(ctypes.byref(shape), L, q.data_ptr(), k.data_ptr(), 2, cb.data_ptr(), codes.data_ptr(), L * m,
                                      v.data_ptr(), L * d_k, scale, 0, None, 0, out.data_ptr(), torch.cuda.current_stream().cuda_stream)
    assert rc == 0 and torch.equal(out, one)
    out.zero_()
    rc = lib.lookat_decode_step_gqa(ctypes.byref(shape), 1, L, q.data_ptr(), k.data_ptr(), 2, cb.data_ptr(), codes.data_ptr(), L * m,
                                    v.data_ptr(), L * d_k, scale, 0, None, 0, out.data_ptr(), torch.cuda.current_stream().cuda_stream)
    assert rc == 0 and torch.equal(out, one)


@pytest.mark.gpu
@pytest.mark.parametrize("d_k,m,B,H,L,cut", [(128, 4, 22, 12, 2048, False), (128, 8, 24, 12, 2100, False), (128, 4, 48, 8, 2500, False),
                                             (64, 4, 22, 12, 3500, False), (128, 8, 22, 12, 2600, True), (128, 4, 23, 12, 2048, True),
                                             (128, 8, 1, 12, 1024, False), (128, 8, 1, 12, 1400, True)])
def test_fused_step_is_cut_where_it_gains(d_k, m, B, H, L, cut):
    """Where one range is served by paired batch entries, or is two tiles per wavefront, the library cuts only what gains by it."""
    import torch
    lk = _lk()
    assert lk.attend_decode_auto_splits(B, H, d_k, m, L) > 1 or not cut
    assert lk.decode_step_entries_per_workgroup(B, H, d_k, m, L) == (1 if B % 2 else 2)      # (odd batches have no pairs)
    g = torch.Generator(device="cuda").manual_seed(L)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    codes = torch.randint(0, 256, (B, H, L, m), generator=g, device="cuda", dtype=torch.uint8)
    v, q, k, cb = rnd(B, H, L, d_k).half(), rnd(B, H, d_k), rnd(B, H, d_k), rnd(H, m, 256, d_k // m)
    one = lk.lookat_decode_step(q, k, cb, codes, v, d_k ** -0.5)
    ws = torch.zeros(max(16, lk.decode_step_split_workspace_bytes(B, H, d_k, m, L)), dtype=torch.uint8, device="cuda")
    got = lk.lookat_decode_step_split(q, k, cb, codes, v, d_k ** -0.5, workspace=ws)
    assert bool(ws.any()) == cut                      # (the ranges' partial results)
    assert torch.equal(got, one) if not cut else float((got - one).abs().max()) <= 2e-5


@pytest.mark.gpu
def test_auto_splits_with_a_smaller_workspace():
    """The library's choice adapts to the workspace it is given, down to the count it asked for before it chose by predicted times."""
    import torch
    from paper_2601_10155_amd.binding import _Shape, load_library
    lk, lib = _lk(), load_library()
    d_k, m = 128, 8
    for B, H, L in ((1, 12, 4096), (1, 32, 8192), (1, 3, 2048), (11, 24, 4133)):
        shape = _Shape(B, H, d_k, m, 256)
        per = B * H * (d_k + 2) * 4
        auto = lk.attend_decode_auto_splits(B, H, d_k, m, L)
        base = max(1, min(256 // (B * H), -(-L // 2048)))
        assert auto > base
        g = torch.Generator(device="cuda").manual_seed(L)
        lut = torch.randn((B, H, m, 256), generator=g, device="cuda")
        codes = torch.randint(0, 256, (B, H, L, m), generator=g, device="cuda", dtype=torch.uint8)
        v = torch.randn((B, H, L, d_k), generator=g, device="cuda").half()
        ref = lk.lookat_attend_decode(lut, codes, v, d_k ** -0.5, num_splits=1)
        for held in range(0, auto + 1):
            need = 0 if held <= 1 else held * per
            ws = torch.zeros(auto * per + 16, dtype=torch.uint8, device="cuda")
            out = torch.zeros_like(ref)
            rc = lib.lookat_attend_decode(ctypes.byref(shape), L, lut.data_ptr(), codes.data_ptr(), L * m, v.data_ptr(), L * d_k,
                                          d_k ** -0.5, 0, ws.data_ptr(), need, out.data_ptr(), None,
                                          torch.cuda.current_stream().cuda_stream)
            if base > 1 and held < base:
                assert rc == -5                      # as it always was
            else:
                assert rc == 0 and float((out - ref).abs().max()) <= 2e-5
                assert not bool(ws[need:].any())     # nothing beyond what was given
            # and through the package: a workspace that is too small for any choice is replaced, a smaller one is used
            got = lk.lookat_attend_decode(lut, codes, v, d_k ** -0.5, workspace=ws[:max(need, 16)], out=torch.empty_like(ref))
            assert float((got - ref).abs().max()) <= 2e-5
            assert not bool(ws[max(need, 16):].any())
