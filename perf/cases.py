"""The work a program has this library do, as cases that can be timed and compared.

A case is one pass through the public calls on arrays that live on the GPU: decode steps (one launch per layer,
ranges for a single long sequence, grouped queries, the three separate calls for other head sizes), filling the
code cache from a prompt, batched tables, causal scores of a prompt block and of a short chunk, and one iteration
of codebook learning.  listed() names twelve of them, draw() gives others of the same ranges.

Inputs follow the recipe of the tests and the benchmark: keys of low rank plus noise, values N(0,1) in fp16, queries
N(0,1)/8, codebooks whose centroids are sub-vectors of keys from the same generator.  Cached codes are drawn from a
skewed histogram of its own order per (head, subspace): real caches use some centroids much more than others.
"""
import math

import torch

import paper_2601_10155_amd as lk

K = 256
NOISE = 0.1


def listed():
    return [
        # One user, short context: twelve layers of twelve small heads.  Launches and host calls are what counts.
        {"name": "step_one_user", "kind": "step", "B": 1, "H": 12, "L": 1024, "spare": 0, "d_k": 64, "m": 2, "layers": 12,
         "dtype": "float16"},
        # The benchmark's batch: 32 sequences, twelve layers, every cache read once per step.
        {"name": "step_batch", "kind": "step", "B": 32, "H": 12, "L": 1024, "spare": 0, "d_k": 64, "m": 4, "layers": 12,
         "dtype": "float16"},
        # Long contexts in a batch: 2.2 GB of cache in one launch.
        {"name": "step_long_batch", "kind": "step", "B": 8, "H": 32, "L": 32768, "spare": 0, "d_k": 128, "m": 8, "layers": 1,
         "dtype": "float16"},
        # One user in the middle of a long document: few (batch, head) pairs, a cache longer than its content.
        {"name": "split_one_user", "kind": "split", "B": 1, "H": 32, "L": 8003, "spare": 189, "d_k": 128, "m": 8,
         "layers": 1, "dtype": "float16"},
        # Eight query heads on each of four key/value heads, long contexts.
        {"name": "grouped_long", "kind": "grouped", "B": 8, "H": 4, "group": 8, "L": 32768, "spare": 0, "d_k": 128, "m": 8,
         "layers": 1, "dtype": "float16"},
        # A head size the fused step does not take: append, tables and attention as three calls, ragged context.
        {"name": "calls_head_96", "kind": "calls", "B": 4, "H": 16, "L": 2501, "spare": 59, "d_k": 96, "m": 8, "layers": 1,
         "dtype": "float16"},
        # The prompt of that batch enters the cache: fp32 keys.
        {"name": "fill_fp32", "kind": "fill", "B": 32, "H": 12, "N": 1024, "d_k": 64, "m": 4, "dtype": "float32"},
        # A prompt block of long heads enters the cache: fp16 keys, sixteen subspaces.
        {"name": "fill_fp16", "kind": "fill", "B": 4, "H": 32, "N": 2048, "d_k": 128, "m": 16, "dtype": "float16"},
        # Tables of a prompt block for a caller that does its own look-ups.
        {"name": "tables_block", "kind": "tables", "B": 4, "H": 32, "T": 512, "d_k": 128, "m": 16, "dtype": "float16"},
        # All causal scores of a prompt block.
        {"name": "scores_block", "kind": "scores", "B": 4, "H": 32, "T": 2048, "L": 2048, "d_k": 128, "m": 16,
         "dtype": "float16"},
        # A short chunk (drafted tokens, the last piece of a prompt) against a long cache.
        {"name": "scores_chunk", "kind": "scores", "B": 4, "H": 32, "T": 8, "L": 4096, "d_k": 128, "m": 16,
         "dtype": "float16"},
        # Codebook learning on the long-context configuration's calibration set, one iteration.
        {"name": "learn_codebooks", "kind": "learn", "H": 32, "N": 16384, "d_k": 128, "m": 8},
    ]


def _log_int(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def draw(rng):
    kind = rng.choice(["step", "step", "split", "grouped", "calls", "fill", "tables", "scores", "scores", "learn"])
    while True:
        d_k = rng.choice([64, 128])
        m = rng.choice([2, 4, 8, 16])
        H = rng.choice([4, 8, 12, 16, 25, 32, 40])
        dtype = rng.choice(["float16", "float16", "float32"])
        if kind == "step":
            c = {"B": _log_int(rng, 1, 64), "H": H, "L": _log_int(rng, 100, 32768), "layers": rng.choice([1, 2, 12])}
        elif kind == "split":
            c = {"B": rng.choice([1, 1, 2, 4]), "H": H, "L": _log_int(rng, 500, 32768), "layers": 1}
        elif kind == "grouped":
            # (group * m tables have to fit the on-chip memory: 64 with the reduction buffer)
            group = rng.choice([g for g in (2, 4, 8) if g * m <= 64])
            c = {"B": _log_int(rng, 1, 32), "H": rng.choice([2, 4, 8]), "group": group, "L": _log_int(rng, 500, 32768),
                 "layers": 1}
        elif kind == "calls":
            d_k = rng.choice([32, 64, 80, 96, 112, 128, 160, 256])
            m = rng.choice([n for n in (1, 2, 4, 5, 8, 10, 16, 32) if d_k % n == 0 and 4 <= d_k // n <= 64])
            c = {"B": _log_int(rng, 1, 32), "H": H, "L": _log_int(rng, 100, 8192), "layers": 1}
        elif kind == "fill":
            c = {"B": _log_int(rng, 1, 32), "H": H, "N": _log_int(rng, 64, 8192)}
        elif kind == "tables":
            c = {"B": _log_int(rng, 1, 8), "H": H, "T": _log_int(rng, 1, 1024)}
        elif kind == "scores":
            T = _log_int(rng, 2, 2048)
            c = {"B": _log_int(rng, 1, 8), "H": H, "T": T, "L": max(T, _log_int(rng, 256, 8192))}
        else:
            dtype = "float32"
            c = {"H": H, "N": _log_int(rng, 512, 24576)}
        if "layers" in c:
            c["spare"] = rng.choice([0, 0, 24, 100])
        c = dict({"kind": kind}, **c, d_k=d_k, m=m, dtype=dtype)
        w = work(c)
        # no more than the largest listed case costs (and, where every centroid of every key is a candidate, no
        # more than the largest listed fill)
        most = 4.5e8 if kind == "calls" else 2.0e9
        if w["bytes"] <= most and w["flops"] <= 2.2e11:
            return c


# ---- inputs ---------------------------------------------------------------------------------------------------
def _gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + salt) % (1 << 62))
    return g


def _randn(g, *shape, dtype=torch.float32):
    return torch.randn(shape, generator=g, device="cuda", dtype=dtype)


def _keys(g, A, lead, n):
    """[*lead, H, n, d_k] fp32: low rank plus noise, the mixing matrix A [H, rank, d_k] shared by all of a head's keys."""
    H, rank, d_k = A.shape
    out = _randn(g, *lead, H, n, d_k) * NOISE
    z = _randn(g, *lead, H, n, rank)
    for r in range(rank):
        out.addcmul_(z[..., r:r + 1], A[:, r, None, :])
    return out


def _codebooks(g, A, m):
    """[H, m, 256, d_sub] fp32: sub-vectors of keys from the same generator, a little inside them as means are."""
    H, _, d_k = A.shape
    c = _keys(g, A, (), K).view(H, K, m, d_k // m).transpose(1, 2)
    return (0.9 * c).contiguous()


def _codes(g, B, H, L, m):
    """[B, H, L, m] uint8 from a skewed histogram over the centroids, in an order of its own per (head, subspace)."""
    order = torch.rand((H, m, K), generator=g, device="cuda").argsort(-1).to(torch.uint8)
    u = torch.rand((B, H, L, m), generator=g, device="cuda")
    rank = (u.pow_(1.8) * K).to(torch.int64).clamp_(0, K - 1)
    hi = torch.arange(H * m, device="cuda").view(1, H, 1, m) * K
    return order.view(-1)[rank.add_(hi)]


def _mixing(g, c):
    return _randn(g, c["H"], 8 if c["d_k"] <= 64 else 16, c["d_k"])


def _layer(c, seed, salt):
    g = _gen(seed, salt)
    dt = getattr(torch, c["dtype"])
    B, H, L, d_k, m = c["B"], c["H"], c["L"], c["d_k"], c["m"]
    A = _mixing(g, c)
    rows = L + c["spare"]
    group = c.get("group", 1)
    s = {"codebooks": _codebooks(g, A, m),
         "cache": _codes(g, B, H, rows, m),
         "k_new": _keys(g, A, (B,), 1).view(B, H, d_k).to(dt),
         "q": (_randn(g, B, H * group, d_k) / 8).to(dt),
         "values": _randn(g, B, H, rows, d_k, dtype=torch.float16),
         "out": torch.empty((B, H * group, d_k), device="cuda")}
    s["codes_view"], s["values_view"] = s["cache"][:, :, :L], s["values"][:, :, :L]
    return s


def prepare(case, seed):
    c = case
    kind, d_k, m, H = c["kind"], c["d_k"], c["m"], c["H"]
    if "layers" in c:
        s = {"case": c, "scale": 1.0 / math.sqrt(d_k), "layers": [_layer(c, seed, n) for n in range(c["layers"])]}
        need = 0
        if kind == "split":
            need = lk.decode_step_split_workspace_bytes(c["B"], H, d_k, m, c["L"])
        elif kind == "grouped":
            # (the fused step and the separate call ask for the same workspace)
            need = lk.attend_decode_gqa_workspace_bytes(c["B"], H, c["group"], d_k, m, c["L"])
        elif kind == "calls":
            need = lk.attend_decode_workspace_bytes(c["B"], H, d_k, m, c["L"])
            s["lut"] = torch.empty((c["B"], H, 1, m, K), device="cuda")
        s["workspace"] = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
        return s
    g = _gen(seed, 0)
    A = _mixing(g, c)
    s = {"case": c, "codebooks": _codebooks(g, A, m)}
    if kind == "fill":
        s["keys"] = _keys(g, A, (c["B"],), c["N"]).to(getattr(torch, c["dtype"]))
        s["codes"] = torch.empty((c["B"], H, c["N"], m), dtype=torch.uint8, device="cuda")
    elif kind == "learn":
        s["calib"] = _keys(g, A, (), c["N"])
        s["new"] = torch.empty_like(s["codebooks"])
        s["assign"] = torch.empty((H, c["N"], m), dtype=torch.uint8, device="cuda")
    else:
        s["q"] = (_randn(g, c["B"], H, c["T"], d_k) / 8).to(getattr(torch, c["dtype"]))
        if kind == "tables":
            s["lut"] = torch.empty((c["B"], H, c["T"], m, K), device="cuda")
        else:
            s["codes"] = _codes(g, c["B"], H, c["L"], m)
            s["scores"] = torch.empty((c["B"], H, c["T"], c["L"]), device="cuda")
    return s


# ---- one pass ---------------------------------------------------------------------------------------------------
def run(state):
    c = state["case"]
    kind = c["kind"]
    if "layers" in c:
        scale, ws = state["scale"], state["workspace"]
        if kind == "step":
            for y in state["layers"]:
                lk.lookat_decode_step(y["q"], y["k_new"], y["codebooks"], y["codes_view"], y["values_view"], scale, out=y["out"])
        elif kind == "split":
            for y in state["layers"]:
                lk.lookat_decode_step_split(y["q"], y["k_new"], y["codebooks"], y["codes_view"], y["values_view"], scale,
                                            workspace=ws, out=y["out"])
        elif kind == "grouped":
            for y in state["layers"]:
                lk.lookat_decode_step_gqa(y["q"], y["k_new"], y["codebooks"], y["codes_view"], y["values_view"], scale,
                                          workspace=ws, out=y["out"])
        else:
            for y in state["layers"]:
                lk.lookat_encode_keys(y["k_new"].unsqueeze(2), y["codebooks"], cache=y["cache"], position=c["L"] - 1)
                lk.lookat_build_lut(y["q"].unsqueeze(2), y["codebooks"], lut_out=state["lut"])
                lk.lookat_attend_decode(state["lut"], y["codes_view"], y["values_view"], scale, workspace=ws, out=y["out"])
        return [[y["out"], y["cache"]] for y in state["layers"]]
    if kind == "fill":
        return lk.lookat_encode_keys(state["keys"], state["codebooks"], codes_out=state["codes"])
    if kind == "tables":
        return lk.lookat_build_lut(state["q"], state["codebooks"], lut_out=state["lut"])
    if kind == "scores":
        return lk.lookat_score_prefill(state["q"], state["codebooks"], state["codes"], scores_out=state["scores"])
    return list(lk.lookat_kmeans_step(state["calib"], state["codebooks"], state["new"], state["assign"]))


def work(case):
    """Each input read once, each output written once; a nearest-centroid search counts as the product of the keys
    with all centroids, a causal score as d_k multiply-adds."""
    c = case
    kind, d_k, m, H = c["kind"], c["d_k"], c["m"], c["H"]
    e = 2 if c.get("dtype") == "float16" else 4
    book = H * K * d_k * 4
    if "layers" in c:
        g = c.get("group", 1)
        BH = c["B"] * H
        rw = BH * c["L"] * (m + 2 * d_k) + BH * (1 + g) * d_k * e + BH * m + BH * g * d_k * 4 + book
        fl = BH * g * (2 * c["L"] * d_k + c["L"] * m) + BH * (1 + g) * 2 * K * d_k
        return {"bytes": c["layers"] * rw, "flops": c["layers"] * fl}
    if kind == "fill":
        n = c["B"] * H * c["N"]
        return {"bytes": n * (d_k * e + m) + book, "flops": 2 * n * K * d_k}
    if kind == "learn":
        n = H * c["N"]
        return {"bytes": n * (d_k * 4 + m) + 2 * book, "flops": 2 * n * K * d_k + n * d_k}
    n = c["B"] * H * c["T"]
    if kind == "tables":
        return {"bytes": n * (d_k * e + m * K * 4) + book, "flops": 2 * n * K * d_k}
    seen = c["L"] - (c["T"] - 1) / 2
    return {"bytes": n * (d_k * e + c["L"] * 4) + c["B"] * H * c["L"] * m + book, "flops": 2 * n * seen * d_k}


def tolerance(case):
    kind = case["kind"]
    if kind in ("fill", "learn"):
        return "exact"   # codes are bytes; the means are sums in a stated order, rounded once
    if kind in ("tables", "scores"):
        return {"rel": 4e-7, "max": 1e-5}   # fp32 sums of 4 to 128 products: 5e-8 to 1e-7 off 64 bits
    return {"rel": 2.5e-6, "max": 4e-5}      # the longest contexts (32768 keys) are 6e-7 off 64 bits


# ---- the same in 64 bits --------------------------------------------------------------------------------------
def _nearest(x, cb):
    """x [n, d_sub], cb [256, d_sub], both fp64 -> index of the nearest centroid."""
    out = torch.empty(x.shape[0], dtype=torch.int64, device=x.device)
    step = max(1, (1 << 25) // (K * x.shape[1]))
    for a in range(0, x.shape[0], step):
        out[a:a + step] = (x[a:a + step, None, :] - cb[None]).square_().sum(-1).argmin(-1)
    return out


def _encode(keys, codebooks):
    """keys [B, H, N, d_k] -> codes [B, H, N, m] uint8."""
    B, H, N, d_k = keys.shape
    m, d_sub = codebooks.shape[1], codebooks.shape[3]
    codes = torch.empty((B, H, N, m), dtype=torch.uint8, device=keys.device)
    for h in range(H):
        for i in range(m):
            x = keys[:, h, :, i * d_sub:(i + 1) * d_sub].reshape(-1, d_sub).double()
            codes[:, h, :, i] = _nearest(x, codebooks[h, i].double()).view(B, N).to(torch.uint8)
    return codes


def _tables(q, codebooks):
    """q [B, H, T, d_k] -> [B, H, T, m, 256] fp64, head by head."""
    B, H, T, d_k = q.shape
    _, m, _, d_sub = codebooks.shape
    out = torch.zeros((B, H, T, m, K), dtype=torch.float64, device=q.device)
    for j in range(d_sub):
        qj = q.view(B, H, T, m, d_sub)[..., j].double()
        out.addcmul_(qj[..., None], codebooks[:, None, :, :, j].double())
    return out


def exact(case, seed):
    c = case
    s = prepare(case, seed)
    kind, m = c["kind"], c["m"]
    if "layers" in c:
        got = []
        for y in s["layers"]:
            B, H, L, g = c["B"], c["H"], c["L"], c.get("group", 1)
            y["cache"][:, :, L - 1] = _encode(y["k_new"].unsqueeze(2), y["codebooks"])[:, :, 0]
            books = y["codebooks"].repeat_interleave(g, 0)
            lut = _tables(y["q"].unsqueeze(2), books)[:, :, 0]                     # [B, H*g, m, 256]
            out = torch.empty_like(y["out"], dtype=torch.float64)
            for b in range(B):
                for h in range(H):
                    codes = y["cache"][b, h, :L].long()
                    v = y["values"][b, h, :L].double()
                    for n in range(h * g, (h + 1) * g):
                        sc = lut[b, n].gather(1, codes.t()).sum(0)
                        out[b, n] = (torch.softmax(sc * s["scale"], 0)[:, None] * v).sum(0)
            got.append([out, y["cache"]])
        return got
    if kind == "fill":
        return _encode(s["keys"], s["codebooks"])
    if kind == "learn":
        assign = _encode(s["calib"].unsqueeze(0), s["codebooks"])[0]
        new = s["codebooks"].double()
        for h in range(c["H"]):
            for i in range(m):
                a = assign[h, :, i].long()
                x = s["calib"][h].view(c["N"], m, -1)[:, i].double()
                sums = torch.zeros_like(new[h, i]).index_add_(0, a, x)
                n = torch.bincount(a, minlength=K).double()[:, None]
                new[h, i] = torch.where(n > 0, sums / n.clamp(min=1), new[h, i])
        return [new, assign]
    if kind == "tables":
        return _tables(s["q"], s["codebooks"])
    B, H, T, L = c["B"], c["H"], c["T"], c["L"]
    scores = torch.empty((B, H, T, L), dtype=torch.float64, device="cuda")
    unseen = torch.arange(L, device="cuda")[None, :] > torch.arange(L - T, L, device="cuda")[:, None]
    for b in range(B):
        for h in range(H):
            sub = torch.arange(m, device="cuda")
            key = s["codebooks"][h][sub, s["codes"][b, h].long()].reshape(L, -1).double()
            scores[b, h] = (s["q"][b, h].double() @ key.t()).masked_fill_(unseen, -math.inf)
    return scores
