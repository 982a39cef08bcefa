"""Performance cases: the operators of the library over the sizes they run at.

A case is one operator execution through the public binding
(``rc.Plan.launch``) on device-resident inputs: the plan (a compiled
schedule), the weights and the workspace are what a program keeps between
calls; a pass is one launch.  The schedules are the ones this repository
ships for its named workloads, and, for sizes it does not name, the first
legal one of a short list per operator (what a search at sizes of that kind
settles on): fixed here, so that a pass always runs the same program
variant.
"""
from __future__ import annotations

import math

import torch

from paper_2506_01374_amd import rc

_KIND = {"gemm_f32": rc.RC_OP_GEMM_F32, "attention": rc.RC_OP_ATTENTION, "gated_mlp": rc.RC_OP_GATED_MLP,
         "moe": rc.RC_OP_MOE, "conv": rc.RC_OP_CONV2D}


def listed():
    return [
        # the smallest call: one 128-cube fp32 contraction, bound by launch and latency
        _gemm("gemm_f32_128", 128, 128, 128),
        # decode: one expert projection for 16 tokens in fp32, a stream of the weight
        _gemm("gemm_f32_m16_n2048_k7168", 16, 2048, 7168),
        # an ordinary fp32 contraction whose sizes no tile divides
        _gemm("gemm_f32_m1000_n1364_k900", 1000, 1364, 900),
        # prefill of a 32-head decoder layer, 1024 tokens
        _attention("attention_causal_b1_h32_s1024_d128", 1, 32, 1024, 128, True),
        # image tokens of a 1024 x 1024 picture, no mask
        _attention("attention_noncausal_b1_h24_s4096_d128", 1, 24, 4096, 128, False),
        # two prompts of a ragged length, the other head dimension
        _attention("attention_causal_b2_h16_s777_d64", 2, 16, 777, 64, True),
        # prefill of a large gated MLP: the largest case
        _mlp("gated_mlp_t2048_h4096_i14336", 2048, 4096, 14336),
        # decode of the same layer for 16 sequences: a stream of the weights
        _mlp("gated_mlp_t16_h4096_i14336", 16, 4096, 14336),
        # prefill of a routed layer of 64 experts, top-6
        _moe("moe_t4096_h2048_e64_i1408_top6", 4096, 2048, 64, 1408, 6),
        # decode of the same layer for 32 sequences: a few rows per expert
        _moe("moe_t32_h2048_e64_i1408_top6", 32, 2048, 64, 1408, 6),
        # a residual block's 3 x 3 convolution with bias and SiLU
        _conv("conv3x3_n2_64x64_c320_k320", 2, 64, 64, 320, 320, 3, True),
        # a plain bf16 projection of 1000 rows: 1 x 1 filters, bias, no activation
        _conv("conv1x1_n1_1x1000_c4096_k4096_noact", 1, 1, 1000, 4096, 4096, 1, False),
    ]


def _gemm(name, m, n, k):
    return {"name": name, "op": "gemm_f32", "m": m, "n": n, "k": k}


def _attention(name, b, h, s, d, causal):
    return {"name": name, "op": "attention", "b": b, "h": h, "s": s, "d": d, "causal": causal}


def _mlp(name, t, hd, i):
    return {"name": name, "op": "gated_mlp", "t": t, "hd": hd, "i": i}


def _moe(name, t, hd, e, i, topk):
    return {"name": name, "op": "moe", "t": t, "hd": hd, "e": e, "i": i, "topk": topk}


def _conv(name, n, h, w, c, k, r, act):
    return {"name": name, "op": "conv", "n": n, "h": h, "w": w, "c": c, "k": k, "r": r, "act": act}


def _log(rng, lo, hi, step=1):
    """A multiple of `step` in [lo, hi], uniform in its logarithm."""
    x = math.exp(rng.uniform(math.log(lo), math.log(hi + step)))
    return max(lo, min(hi, int(x) // step * step))


def draw(rng):
    """One more case of the same ranges (the largest stays below the listed
    2048-token MLP in work and in bytes)."""
    op = rng.choice(["gemm_f32", "gemm_f32_decode", "attention", "gated_mlp", "moe", "conv"])
    if op == "gemm_f32":
        c = _gemm("", _log(rng, 17, 2048), _log(rng, 16, 2048), _log(rng, 16, 2048))
    elif op == "gemm_f32_decode":
        c = _gemm("", rng.randint(1, 16), _log(rng, 256, 8192, 64), _log(rng, 512, 8192, 64))
    elif op == "attention":
        s = _log(rng, 64, 4096)
        most = max(1, min(64, int(32 * 4096 * 4096 / (s * s))))
        c = _attention("", 1, _log(rng, 1, most), s, rng.choice([64, 128]), rng.random() < 0.5)
        if c["h"] % 2 == 0 and rng.random() < 0.5:
            c["b"], c["h"] = 2, c["h"] // 2
    elif op == "gated_mlp":
        c = _mlp("", _log(rng, 1, 2048), _log(rng, 512, 4096, 256), _log(rng, 512, 14336, 256))
    elif op == "moe":
        e = rng.choice([8, 16, 32, 64])
        c = _moe("", _log(rng, 4, 4096), _log(rng, 512, 2048, 256), e, _log(rng, 256, 1408, 128), rng.randint(1, 6))
    else:
        r = rng.choice([1, 3, 3])
        c = _conv("", rng.randint(1, 4), _log(rng, 7, 80), _log(rng, 7, 80), _log(rng, 64, 640, 64),
                  _log(rng, 64, 640, 64), r, r == 3 or rng.random() < 0.5)
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# Operators and schedules
# ---------------------------------------------------------------------------

def _op(case):
    op = case["op"]
    if op == "gemm_f32":
        return rc.Op(_KIND[op], (case["m"], case["n"], case["k"]), 0)
    if op == "attention":
        return rc.Op(_KIND[op], (case["b"], case["h"], case["s"], case["d"]), rc.RC_FLAG_CAUSAL if case["causal"] else 0)
    if op == "gated_mlp":
        return rc.Op(_KIND[op], (case["t"], case["hd"], case["i"]), 0)
    if op == "moe":
        return rc.Op(_KIND[op], (case["t"], case["hd"], case["e"], case["i"], case["topk"]), 0)
    return rc.Op(_KIND[op], (case["n"], case["h"], case["w"], case["c"], case["k"], case["r"], case["r"], case["r"] // 2),
                 0 if case["act"] else rc.RC_FLAG_NO_ACT)


def _block(prefix, tm, tn, tk, wm, wn, grid, occ, stages=7):
    names = ("tile_m", "tile_n", "tile_k", "waves_m", "waves_n", "mfma", "stages", "vec", "unroll", "layout", "grid", "occ")
    vals = (tm, tn, tk, wm, wn, 16, stages, 8, 1, 1, grid, occ)
    return ",".join(f"{prefix}{k}={v}" for k, v in zip(names, vals))


def _gemm_texts(case):
    m, n, k = case["m"], case["n"], case["k"]
    vec = 4 if k % 4 == 0 and n % 4 == 0 else 1
    if m <= 16:
        for splits in (16, 8, 4, 2, 1):
            yield (f"tile_m=16,tile_n=64,tile_k=16,waves_m=2,waves_n=2,vec=4,stages=3,unroll=1,layout=0,"
                   f"splits={splits}")
    tiles = [(64, 32, 2, 2), (32, 32, 2, 2)] if m * n >= 256 * 1024 else []
    for tm, tn, wm, wn in tiles + [(16, 32, 1, 2), (16, 16, 1, 1)]:
        for tk in (32, 16, 8, 4):
            yield (f"tile_m={tm},tile_n={tn},tile_k={tk},waves_m={wm},waves_n={wn},vec={vec},stages=2,unroll=1,"
                   f"layout=0")


def _attention_texts(case):
    s, d = case["s"], case["d"]
    if not case["causal"] and s >= 2048 and d == 128:
        yield "block_m=128,block_n=64,waves=4,mfma=16,stages=4,vec=8,unroll=2,order=1,occ=2,splits=2,chunk=0"
    bn = 32 if d == 128 else 64
    for order in ((2, 1) if case["causal"] and d == 128 else (1,)):
        for bm, w in ((64, 4), (32, 2), (16, 1)):
            yield (f"block_m={bm},block_n={bn},waves={w},mfma=16,stages=4,vec=8,unroll=1,order={order},occ=4,"
                   f"splits=2,chunk=0")
            yield (f"block_m={bm},block_n=32,waves={w},mfma=16,stages=4,vec=8,unroll=1,order={order},occ=1,"
                   f"splits=1,chunk=0")


def _mlp_texts(case):
    t = case["t"]
    rows = next(r for r in (16, 32, 64, 128, 256) if t <= r or r == 256)
    if t >= 1024:
        ups = [_block("up.", 256, 128, 32, 2, 4, 1, 1) + f",up.tail={tail}" for tail in (1, 0)]
        ups += [_block("up.", 128, 64, 64, 2, 2, 1, 1)]
        downs = [_block("down.", 256, 256, 32, 2, 4, 1, 1) + f",down.split={sp}" for sp in (2, 1)]
        downs += [_block("down.", 128, 128, 64, 2, 2, 1, 1), _block("down.", 128, 64, 64, 2, 2, 1, 1)]
    elif t > 64:
        ups = [_block("up.", 128, 128, 64, 2, 4, 1, 1), _block("up.", 128, 64, 64, 2, 2, 1, 1)]
        downs = [_block("down.", 128, 128, 64, 2, 4, 1, 1) + f",down.split={sp}" for sp in (4, 2, 1)]
        downs += [_block("down.", 128, 64, 64, 2, 2, 1, 1)]
    else:
        ups = [_block("up.", rows, 64, tk, 1, 4, 1, 1) for tk in (128, 64)]
        downs = [_block("down.", rows, 64, tk, 1, 4, 1, 1) + f",down.split={sp}"
                 for sp in (4, 2, 1) for tk in (128, 64)]
    for u in ups:
        for d in downs:
            yield u + "," + d + ",fuse=1"


def _moe_texts(case):
    per = case["t"] * case["topk"] / case["e"]
    if per > 128:
        for u in (_block("up.", 256, 128, 32, 2, 4, 2, 2), _block("up.", 128, 64, 64, 2, 2, 2, 1)):
            for d in (_block("down.", 256, 256, 32, 2, 4, 2, 1), _block("down.", 128, 128, 64, 2, 2, 2, 1)):
                yield u + "," + d + ",fuse=1,up.skip=1,down.skip=1"
    for rows in (16, 32, 64, 128):
        if per <= rows or rows == 128:
            for tk in (128, 64):
                u = _block("up.", rows, 32, tk, 1, 2, 2, 1) if rows <= 32 else _block("up.", rows, 64, tk, 2, 2, 2, 1)
                d = _block("down.", rows, 64, tk, 1, 4, 1, 1) if rows <= 32 else _block("down.", rows, 64, tk, 2, 2, 2, 1)
                yield u + "," + d + ",fuse=1,up.skip=0,down.skip=0"


def _conv_texts(case):
    pix = case["n"] * case["h"] * case["w"]
    blocks = [(256, 256, 32, 2, 4, 1, 1), (128, 128, 64, 2, 4, 1, 2), (64, 160, 64, 2, 2, 2, 1), (64, 64, 64, 2, 2, 1, 1)]
    for least in (200, 0):          # first the largest tile that still gives most CUs a workgroup
        for b in blocks if least else blocks[::-1]:
            if -(-pix // b[0]) * (case["k"] // b[1]) >= least:
                yield _block("", *b) + ",fuse=1"
    for tm, tn in ((32, 64), (16, 64), (16, 32)):
        yield _block("", tm, tn, 64, 1, 2, 1, 1) + ",fuse=1"


_TEXTS = {"gemm_f32": _gemm_texts, "attention": _attention_texts, "gated_mlp": _mlp_texts, "moe": _moe_texts,
          "conv": _conv_texts}


def _schedule(op, case):
    for text in _TEXTS[case["op"]](case):
        s = op.from_string(text)
        if s.validate() == "":
            return s
    raise ValueError(f"no legal schedule for {case}")


# ---------------------------------------------------------------------------
# Inputs, a pass, the work and the exact result
# ---------------------------------------------------------------------------

def _inputs(case, seed):
    """Device inputs of a case in the order and layout rc_launch takes: bf16
    weights stored [N][K] (fp32: [K][N]), distributions as in
    paper_2506_01374_amd.inputs."""
    g = torch.Generator(device="cuda").manual_seed(1000003 * (int(seed) + 1))
    dev = "cuda"

    def normal(*shape, sigma=1.0):
        x = torch.empty(shape, dtype=torch.bfloat16, device=dev)
        flat = x.view(-1)
        for i in range(0, flat.numel(), 1 << 26):     # in pieces: no large fp32 copy
            n = min(1 << 26, flat.numel() - i)
            flat[i:i + n] = torch.randn(n, generator=g, device=dev).mul_(sigma)
        return x

    op = case["op"]
    if op == "gemm_f32":
        m, n, k = case["m"], case["n"], case["k"]
        return [torch.rand(a, b, generator=g, device=dev).mul_(2).sub_(1) for a, b in ((m, k), (k, n))]
    if op == "attention":
        shape = (case["b"], case["h"], case["s"], case["d"])
        return [normal(*shape) for _ in range(3)]
    if op == "gated_mlp":
        t, hd, i = case["t"], case["hd"], case["i"]
        return [normal(t, hd)] + [normal(a, b, sigma=0.02) for a, b in ((i, hd), (i, hd), (hd, i))]
    if op == "moe":
        t, hd, e, i, topk = (case[k] for k in ("t", "hd", "e", "i", "topk"))
        p = torch.softmax(torch.randn(t, e, generator=g, device=dev, dtype=torch.float64), dim=1)
        w, ids = torch.topk(p, topk, dim=1)
        return [normal(t, hd), ids.to(torch.int32).contiguous(), w.to(torch.float32).contiguous(),
                normal(e, i, hd, sigma=0.02), normal(e, i, hd, sigma=0.02), normal(e, hd, i, sigma=0.02)]
    n, h, w, c, k, r = (case[x] for x in ("n", "h", "w", "c", "k", "r"))
    return [normal(n, h, w, c), normal(k, r, r, c, sigma=1.0 / math.sqrt(r * r * c)),
            torch.randn(k, generator=g, device=dev)]


def _out_shape(case):
    op = case["op"]
    if op == "gemm_f32":
        return (case["m"], case["n"])
    if op == "attention":
        return (case["b"], case["h"], case["s"], case["d"])
    if op in ("gated_mlp", "moe"):
        return (case["t"], case["hd"])
    return (case["n"], case["h"], case["w"], case["k"])


def prepare(case, seed):
    op = _op(case)
    plan = rc.Plan(op, _schedule(op, case))
    dtype = torch.float32 if case["op"] == "gemm_f32" else torch.bfloat16
    out = torch.empty(_out_shape(case), dtype=dtype, device="cuda")
    return {"plan": plan, "inputs": _inputs(case, seed), "out": out, "workspace": plan.workspace()}


def run(state):
    state["plan"].launch(state["inputs"], state["out"], state["workspace"])
    return state["out"]


def work(case):
    op = case["op"]
    if op == "moe":
        # an expert that no row reaches need not be read
        t, hd, e, i, topk = (case[k] for k in ("t", "hd", "e", "i", "topk"))
        rows = t * topk
        live = e * (1.0 - (1.0 - topk / e) ** t)
        return {"bytes": 2.0 * (2 * t * hd + 3 * live * hd * i) + 8.0 * rows, "flops": 6.0 * rows * hd * i}
    o = _op(case)
    return {"bytes": o.bytes(), "flops": o.flops()}


def tolerance(case):
    # about four times the distance of the path from 64 bits
    return _TOLERANCE[case["op"]]


_TOLERANCE = {"gemm_f32": {"rel": 4e-6, "max": 4e-5}, "attention": {"rel": 1e-2, "max": 6e-2},
              "gated_mlp": {"rel": 1e-2, "max": 6e-2}, "moe": {"rel": 1e-2, "max": 6e-2},
              "conv": {"rel": 7e-3, "max": 4e-2}}


def exact(case, seed):
    ins = _inputs(case, seed)
    op = case["op"]
    if op == "gemm_f32":
        return ins[0].double() @ ins[1].double()
    if op == "attention":
        q, k, v = (x.flatten(0, 1) for x in ins)
        out = torch.empty(q.shape, dtype=torch.float64, device="cuda")
        s, d = case["s"], case["d"]
        hidden = torch.ones(s, s, dtype=torch.bool, device="cuda").triu(1) if case["causal"] else None
        for i in range(q.shape[0]):
            x = q[i].double() @ k[i].double().t().contiguous() / math.sqrt(d)
            if hidden is not None:
                x.masked_fill_(hidden, -math.inf)
            out[i] = torch.softmax(x, dim=1) @ v[i].double()
        return out.view(_out_shape(case))
    if op == "gated_mlp":
        return _gated(ins[0].double(), *ins[1:])
    if op == "moe":
        x, ids, w, wg, wu, wd = ins
        out = torch.zeros(x.shape, dtype=torch.float64, device="cuda")
        for e in range(case["e"]):
            rows, slots = (ids == e).nonzero(as_tuple=True)
            if rows.numel():
                out.index_add_(0, rows, _gated(x[rows].double(), wg[e], wu[e], wd[e]) * w[rows, slots].double()[:, None])
        return out
    x, w, bias = (t.double() for t in ins)
    n, h, wd, r = case["n"], case["h"], case["w"], case["r"]
    p = r // 2
    xp = torch.nn.functional.pad(x, (0, 0, p, p, p, p))
    out = bias.expand(n * h * wd, -1).clone()
    for i in range(r):
        for j in range(r):
            out += xp[:, i:i + h, j:j + wd, :].reshape(n * h * wd, -1) @ w[:, i, j, :].t().contiguous()
    if case["act"]:
        out = torch.nn.functional.silu(out)
    return out.view(_out_shape(case))


def _gated(x, wg, wu, wd):
    """SiLU(x Wg) (x Wu) Wd in 64 bits; weights stored [N][K]."""
    h = torch.nn.functional.silu(x @ wg.double().t()) * (x @ wu.double().t())
    return h @ wd.double().t()
