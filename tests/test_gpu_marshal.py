"""The native marshalling of the binding: where it takes a call the result is the Python path's, bit for bit, and what it
does not take (views that need a copy, subclasses, missing outputs, wrong types and shapes) behaves as before."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lk():
    import paper_2601_10155_amd as pkg
    pkg.load_library()
    return pkg


class Off:
    """Stands in for the native module and takes nothing."""
    def __getattr__(self, name):
        return lambda *a: None


@pytest.fixture()
def both(lk, monkeypatch):
    from paper_2601_10155_amd import binding

    def run(call):
        """(native result, python result, did the native module take the call)"""
        taken = []
        native = binding._marshal

        class Watch:
            def __getattr__(self, name):
                def f(*a):
                    rc = getattr(native, name)(*a)
                    taken.append(rc is not None)
                    return rc
                return f
        monkeypatch.setattr(binding, "_marshal", Watch())
        a = call()
        monkeypatch.setattr(binding, "_marshal", Off())
        b = call()
        monkeypatch.setattr(binding, "_marshal", native)
        return a, b, taken[0]
    return run


def case(B=2, H=4, L=300, d_k=64, m=4, group=1, dtype=torch.float16):
    g = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    return {"cb": rnd(H, m, 256, d_k // m), "q": rnd(B, H * group, d_k).to(dtype), "k": rnd(B, H, d_k).to(dtype),
            "codes": torch.randint(0, 256, (B, H, L + 9, m), generator=g, device="cuda", dtype=torch.uint8)[:, :, :L],
            "values": rnd(B, H, L + 9, d_k).half()[:, :, :L], "out": torch.zeros((B, H * group, d_k), device="cuda")}


@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
def test_calls_that_are_taken(lk, both, dtype):
    c = case(dtype=dtype)
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    sc = 1 / math.sqrt(64)
    step = (c["q"], c["k"], c["cb"], c["codes"], c["values"], sc)
    lut = lk.lookat_build_lut(c["q"].unsqueeze(2), c["cb"]).view(2, 4, 4, 256)
    scores = torch.empty((2, 4, 300), device="cuda")
    g = case(group=4, dtype=dtype)
    keys = torch.randn((2, 4, 70, 64), device="cuda").to(dtype)
    calls = [lambda: lk.lookat_decode_step(*step, out=c["out"]),
             lambda: lk.lookat_decode_step_split(*step, num_splits=3, workspace=ws, out=c["out"]),
             lambda: lk.lookat_decode_step_split(*step, out=c["out"]),
             lambda: lk.lookat_decode_step_gqa(g["q"], g["k"], g["cb"], g["codes"], g["values"], sc, workspace=ws, out=g["out"]),
             lambda: lk.lookat_attend_decode(lut, c["codes"], c["values"], sc, num_splits=2, workspace=ws, out=c["out"], scores_out=scores),
             lambda: lk.lookat_build_lut(c["q"].unsqueeze(2), c["cb"], lut_out=lut),
             lambda: lk.lookat_encode_keys(keys, c["cb"], codes_out=torch.empty((2, 4, 70, 4), dtype=torch.uint8, device="cuda")),
             lambda: lk.lookat_encode_keys(keys, c["cb"], cache=c["codes"], position=11),
             lambda: lk.lookat_score_prefill(keys, c["cb"], c["codes"], scores_out=torch.empty((2, 4, 70, 300), device="cuda"))]
    for n, call in enumerate(calls):
        a, b, taken = both(lambda: call().clone())
        assert taken, f"call {n} was left to the Python path"
        assert torch.equal(a, b), f"call {n}"
    stream = torch.cuda.Stream()                      # the current stream, not the default one
    with torch.cuda.stream(stream):
        stream.wait_stream(torch.cuda.default_stream())
        a, b, taken = both(lambda: lk.lookat_decode_step(*step, out=c["out"]).clone())
    stream.synchronize()
    assert taken and torch.equal(a, b)


def test_calls_that_are_left(lk, both):
    c = case()
    sc = 0.125
    odd = torch.randn((2, 4, 128), device="cuda").half()[:, :, ::2]            # needs a copy

    class Sub(torch.Tensor):
        pass
    for call in (lambda: lk.lookat_decode_step(c["q"], c["k"], c["cb"], c["codes"], c["values"], sc),
                 lambda: lk.lookat_decode_step(odd, c["k"], c["cb"], c["codes"], c["values"], sc, out=c["out"]),
                 lambda: lk.lookat_decode_step(c["q"].as_subclass(Sub), c["k"], c["cb"], c["codes"], c["values"], sc, out=c["out"]),
                 lambda: lk.lookat_decode_step_split(c["q"], c["k"], c["cb"], c["codes"], c["values"], sc, num_splits=3, out=c["out"])):
        a, b, taken = both(lambda: call().clone())
        assert not taken and torch.equal(a.as_subclass(torch.Tensor), b.as_subclass(torch.Tensor))
    bad = [(ValueError, dict(values=c["values"][:, :, :200])), (ValueError, dict(cb=c["cb"][:3])), (ValueError, dict(out=c["out"][:1])),
           (ValueError, dict(codes=c["codes"].int())), (ValueError, dict(k=c["k"].float())), (ValueError, dict(q=c["q"].cpu())),
           (TypeError, dict(q=c["q"].double(), k=c["k"].double())), (ValueError, dict(codes=c["codes"].transpose(0, 1)))]
    for error, change in bad:
        d = dict(c, **change)
        with pytest.raises(error):
            lk.lookat_decode_step(d["q"], d["k"], d["cb"], d["codes"], d["values"], sc, out=d["out"])
    with pytest.raises(lk.LookatError):               # the library's own refusals come through the native path too
        lk.lookat_decode_step(c["q"], c["k"], c["cb"], c["codes"], torch.empty(c["values"].numel() + 1, dtype=torch.float16, device="cuda")[1:]
                              .view(2, 4, 300, 64), sc, out=c["out"])
    with pytest.raises(lk.LookatError):
        lk.lookat_decode_step_split(c["q"], c["k"], c["cb"], c["codes"], c["values"], sc, num_splits=70000,
                                    workspace=torch.empty(1 << 28, dtype=torch.uint8, device="cuda"), out=c["out"])


def test_no_workspace_and_no_output_where_the_library_chooses(lk, both):
    """The ranges are the library's choice: a missing workspace and a missing output are allocated by the native module, with the
    Python path's result, shape and type; explicit counts are left to it."""
    c, g = case(L=3000, d_k=128, m=8), case(L=3000, d_k=128, m=8, group=4)
    sc = 128 ** -0.5
    assert lk.attend_decode_auto_splits(2, 4, 128, 8, 3000) > 1
    lut = lk.lookat_build_lut(c["q"].unsqueeze(2), c["cb"]).view(2, 4, 8, 256)
    scores = torch.empty((2, 4, 3000), device="cuda")
    step = (c["q"], c["k"], c["cb"], c["codes"], c["values"], sc)
    gqa = (g["q"], g["k"], g["cb"], g["codes"], g["values"], sc)
    small = torch.empty(16, dtype=torch.uint8, device="cuda")
    for n, call in enumerate([lambda: lk.lookat_attend_decode(lut, c["codes"], c["values"], sc),
                              lambda: lk.lookat_attend_decode(lut, c["codes"], c["values"], sc, out=c["out"], scores_out=scores),
                              lambda: lk.lookat_decode_step_split(*step), lambda: lk.lookat_decode_step_split(*step, out=c["out"]),
                              lambda: lk.lookat_decode_step_gqa(*gqa), lambda: lk.lookat_decode_step_gqa(*gqa, out=g["out"])]):
        a, b, taken = both(call)
        assert taken, f"call {n} was left to the Python path"
        assert a.shape == b.shape and a.dtype == b.dtype and a.device == b.device and torch.equal(a, b), f"call {n}"
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        stream.wait_stream(torch.cuda.default_stream())
        a, b, taken = both(lambda: lk.lookat_decode_step_split(*step))
    stream.synchronize()
    assert taken and torch.equal(a, b)
    for call in (lambda: lk.lookat_attend_decode(lut, c["codes"], c["values"], sc, num_splits=2, out=c["out"]),
                 lambda: lk.lookat_attend_decode(lut, c["codes"], c["values"], sc, num_splits=1),
                 lambda: lk.lookat_decode_step_gqa(*gqa, workspace=small, out=g["out"])):
        a, b, taken = both(lambda: call().clone())
        assert not taken and torch.equal(a, b)
    graph = torch.cuda.CUDAGraph()                     # recorded: workspace and output come from the graph's own pool
    with torch.cuda.graph(graph):
        out = lk.lookat_decode_step_split(*step)
    for _ in range(3):
        out.zero_()
        graph.replay()
        assert torch.equal(out, lk.lookat_decode_step_split(*step))
    with pytest.raises(lk.LookatError):
        lk.lookat_attend_decode(lut, c["codes"], torch.empty(c["values"].numel() + 1, dtype=torch.float16, device="cuda")[1:].view(2, 4, 3000, 128), sc)
