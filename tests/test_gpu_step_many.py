"""Fused steps of more (b,h) than a launch of one workgroup per compute unit takes, whole and in ranges: the appended codes and the outputs against
the oracle, from a cache whose newest row is stale."""
import pytest
import torch

import oracle  # noqa: F401
from bars import assert_out_close
from test_gpu_parity import _step_case, dev

pytestmark = pytest.mark.gpu

B, H, TIMES = 1, 8, 33        # 264 (b,h): 33 on a die's 32 compute units; an odd batch, which has no pairs


@pytest.fixture(scope="module")
def lk():
    import paper_2601_10155_amd as pkg
    pkg.load_library()
    return pkg


# contexts of one key, one tile more than the wavefronts of a workgroup, three tiles each, and several rounds of the loop
@pytest.mark.parametrize("d_k,m", [(d, m) for d in (64, 128) for m in (2, 4, 8, 16)])
@pytest.mark.parametrize("kind,dtype", [("recipe", "float32"), ("peaked", "float16"), ("aligned", "float16")])
@pytest.mark.parametrize("L", [1, 513, 1537, 4133])
def test_steps_of_many_heads(lk, d_k, m, kind, dtype, L):
    stale, room = 0xAB, L + 67
    c = _step_case("C2" if d_k == 64 else "C3", B, H, room, L, d_k, m, dtype, 9100 + d_k + m, kind)
    many = lambda a: dev(a).repeat(TIMES, *[1] * (a.ndim - 1))
    q, k, cb, values = many(c["q"]), many(c["k_new"]), dev(c["cb"]), many(c["values"])
    rows = torch.full((B * TIMES, H, room, m), stale, dtype=torch.uint8, device="cuda")
    rows[:, :, :L - 1] = dev(c["codes"][:, :, :L - 1])
    for ranges in (1, 2, 3):
        cache = rows.clone()
        args = (q, k, cb, cache[:, :, :L], values[:, :, :L], c["scale"])
        out = lk.lookat_decode_step(*args) if ranges == 1 else lk.lookat_decode_step_split(*args, num_splits=ranges)
        assert torch.equal(cache[:, :, :L], dev(c["codes"]).expand(B * TIMES, H, L, m)), f"codes, {ranges} ranges"
        assert (cache[:, :, L:] == stale).all()
        out = out.view(TIMES, B, H, d_k)
        assert torch.equal(out, out[:1].expand_as(out)), f"the copies differ, {ranges} ranges"
        assert_out_close(out[0].cpu().numpy(), c["out"], f"decode_step of many heads, {ranges} ranges, {kind} queries", c["scores"], c["scale"])
