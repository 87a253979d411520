"""Timed cases of the framework's main paths, through its public entry points.

Each case is a dict of plain values; `prepare` makes what a program holds
before the call (operands on the GPU, descriptors, one library context for
the process), `run` makes one call and returns everything it computed, and
`exact` gives the same outputs from plain torch in FP64.

The sizes are those of the repository's own workloads: triads of 2^20 to 2^28
elements, square GEMMs of 512 to 8192 in the three dtypes, BF16 GEMVs of 4096
to 16384, Llama-3.1-8B decode shapes, per-tensor quantisation of the GEMM
operands, bursts of the serving loop's request mix, and a sensitivity cell.

Outputs: a triad's are exact in FP32, so its checksums come back with it; a
GEMM's or GEMV's checksum is a digest of rounded values that are returned
whole.  BF16 outputs, which the library returns as 16-bit codes, come back
viewed as BF16.
"""
import math
import random

import torch

from paper_2501_16909_amd import coloc

LLAMA = dict(hidden=4096, n_q=32, n_kv=8, head_dim=128, ffn=14336, eps=1e-5, rope_base=500000.0)
SMALL = dict(hidden=512, n_q=4, n_kv=2, head_dim=128, ffn=1032, eps=1e-5, rope_base=500000.0)

_CTX = None


def _ctx():
    """One library context for the process, as a program keeps it."""
    global _CTX
    if _CTX is None:
        _CTX = coloc.Context(0)
    return _CTX


def listed():
    return [
        # the smallest call of the suite: launch latency, stamps and checksum around 12 MB of traffic
        dict(name="triad_1m", op="triad", n=(1 << 20) + 333, passes=1, in_kernel=False),
        # the serving mix's largest streaming request: HBM-bound, far beyond the Infinity Cache
        dict(name="triad_256m", op="triad", n=1 << 28, passes=1, in_kernel=False),
        # the serving mix's smallest GEMM: far fewer tiles than CUs
        dict(name="gemm_bf16_512", op="gemm", dtype="bf16", m=512, n=512, k=512),
        # a mid-sized FP32 GEMM with ragged edges
        dict(name="gemm_f32_1416", op="gemm", dtype="f32", m=1416, n=1402, k=1416),
        # the sensitivity sweep's compute victim
        dict(name="gemm_bf16_4096", op="gemm", dtype="bf16", m=4096, n=4096, k=4096),
        # the precision workload's largest rate
        dict(name="gemm_fp8_8192", op="gemm", dtype="fp8", m=8192, n=8192, k=8192),
        # the sensitivity sweep's memory-bound victim: weights rotated over three copies, so each run is cold
        dict(name="gemv_8192", op="gemv", n=8192, k=8192, copies=3),
        # one token of the Llama-shaped decoder, replayed as a graph
        dict(name="decode_8b", op="decode", model="llama", layers=32, vocab=128256, batch=1, ctx=4096, pos=4095,
             graph=True),
        # decode attention of a full batch of ragged contexts
        dict(name="attention_b8", op="attention", batch=8, n_q=32, n_kv=8, head_dim=128, ctx=8064, pos=8063,
             noalloc=True),
        # per-tensor quantisation of one precision-workload operand
        dict(name="quantize_fp8_8192", op="quantize", dtype="fp8", n=8192 * 8192),
        # sixteen requests of the serving mix that arrive together
        dict(name="serve_burst", op="serve", requests=16, slots=4, budget=8 << 30, mix=119),
        # one cell of a sensitivity sweep: GEMV beside the HBM stressor on half the CUs
        dict(name="sensitivity_gemv", op="sensitivity", n=8192, k=8192, resource="hbm", intensity=0.5, reps=10),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    op = rng.choice(["triad", "triad", "gemm", "gemm", "gemm", "gemm", "gemv", "gemv", "rows", "decode", "decode",
                     "attention", "attention", "quantize", "quantize", "checksum", "serve", "serve"])
    if op == "triad":
        in_kernel = rng.random() < 0.2
        n = int(_log(rng, 1 << 20, 1 << 24 if in_kernel else 1 << 28))
        passes = rng.choice([2, 4, 8]) if in_kernel else (rng.choice([1, 1, 2]) if n < 1 << 26 else 1)
        return dict(op="triad", n=n, passes=passes, in_kernel=in_kernel)
    if op == "gemm":
        dtype = rng.choice(["bf16", "bf16", "fp8", "f32"])
        unit = {"bf16": 8, "fp8": 16, "f32": 4}[dtype]
        top = 4096 if dtype == "f32" else 8192
        m = int(_log(rng, 512, top))
        shape = rng.choice(["square", "square", "aligned", "ragged"])
        n, k = m, m
        if shape == "aligned":                     # the serving mix's sizes
            m = n = k = max(512, m // 128 * 128)
        elif shape == "ragged":
            n, k = (max(64, min(top, int(m * rng.uniform(0.5, 2.0)))) for _ in range(2))
        return dict(op="gemm", dtype=dtype, m=m, n=n, k=max(unit, k // unit * unit))
    if op == "gemv":
        n = int(_log(rng, 4096, 16384))
        k = n if rng.random() < 0.5 else int(_log(rng, 4096, 16384))
        return dict(op="gemv", n=n, k=k // 8 * 8, copies=rng.choice([1, 2, 3]))
    if op == "rows":
        return dict(op="rows", rows=int(_log(rng, 512, 28672)), k=int(_log(rng, 512, 14336)) // 8 * 8,
                    batch=rng.randint(1, 8), res=rng.random() < 0.5)
    if op == "decode":
        model = rng.choice(["llama", "llama", "small"])
        ctx = int(_log(rng, 128, 4096))
        return dict(op="decode", model=model, layers=rng.randint(1, 4),
                    vocab=rng.choice([0, 1000, 32000, 128256] if model == "llama" else [0, 1000]),
                    batch=rng.randint(1, 8), ctx=ctx, pos=rng.randint(ctx // 2, ctx - 1),
                    graph=rng.random() < 0.5)
    if op == "attention":
        n_q, n_kv, d = rng.choice([(32, 8, 128), (32, 8, 128), (16, 8, 256), (4, 1, 256), (32, 32, 128), (16, 1, 128)])
        batch = rng.randint(1, 8)
        ctx = int(_log(rng, 128, 8064))
        return dict(op="attention", batch=batch, n_q=n_q, n_kv=n_kv, head_dim=d, ctx=ctx,
                    pos=rng.randint(ctx // 2, ctx - 1),
                    noalloc=rng.random() < 0.5 and batch * n_q * -(-ctx // 64) * (d + 2) * 4 <= coloc.NOALLOC_PART_BYTES)
    if op == "quantize":
        return dict(op="quantize", dtype=rng.choice(["fp8", "bf16"]), n=int(_log(rng, 1 << 18, 1 << 26)))
    if op == "checksum":
        return dict(op="checksum", n=int(_log(rng, 1 << 18, 1 << 28)))
    while True:                                    # no burst beyond the largest listed case
        case = dict(op="serve", requests=rng.randint(2, 12), slots=rng.randint(1, 4),
                    budget=rng.choice([3, 4, 8]) << 30, mix=rng.randint(100, 1 << 20))
        if work(case)["bytes"] <= 10e9:
            return case


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _uniform(g, *shape):
    return torch.rand(shape, generator=g, device="cuda") * 2.0 - 1.0


def _normal(g, *shape, sigma=1.0):
    return torch.randn(shape, generator=g, device="cuda").mul_(sigma)


def _bf16(x):
    return x.to(torch.bfloat16).view(torch.int16)


def _operand(g, rows, k, dtype):
    """(operand as the library takes it, its values in FP32, scale)."""
    x = _normal(g, rows, k)
    if dtype == "f32":
        return x, x, 1.0
    if dtype == "bf16":
        q = x.to(torch.bfloat16)
        return q.view(torch.int16), q, 1.0
    amax = x.abs().max()
    q = (x * (448.0 / amax)).to(torch.float8_e4m3fn)
    return q.view(torch.uint8), q, float(amax / 448.0)


def _requests(case, seed):
    """A burst of the serving mix: BF16 GEMM 512-8192, BF16 GEMV 4096-16384,
    FP32 triad 2^20-2^28, all log-uniform and a third each; the shapes come
    from the case, the inputs' seeds from `seed`."""
    reqs = [dict(q, arrival_s=0.0, seed=int(seed) * 1000 + 10 * i) for i, q in enumerate(_shapes(case))]
    for q in reqs:
        out = q["m"] * q["n"] if q["kind"] == "gemm" else q["n"]
        q["out_copy"] = torch.empty(out, dtype=torch.float32, device="cuda")
    return reqs


def _positions(case):
    """Ragged contexts: sequence b ends earlier than sequence 0."""
    return [max(0, case["pos"] - (case["ctx"] // 4) * (b % 4)) for b in range(case["batch"])]


def prepare(case, seed):
    ctx = _ctx()
    op, g = case["op"], _gen(seed)
    s = dict(case=case, ctx=ctx)
    if op == "triad":
        s["b"], s["c"] = _uniform(g, case["n"]), _uniform(g, case["n"])
        s["out"] = torch.empty_like(s["b"])
        s["desc"] = ctx.triad_desc(s["b"], s["c"], s["out"], case["passes"], case["in_kernel"])
    elif op == "gemm":
        m, n, k, dt = case["m"], case["n"], case["k"], case["dtype"]
        a, s["va"], s["sa"] = _operand(g, m, k, dt)
        b, s["vb"], s["sb"] = _operand(g, n, k, dt)
        s["out"] = torch.empty((m, n), dtype=torch.float32, device="cuda")
        s["desc"] = ctx.gemm_desc(a, b, s["out"], dt, m, n, k, s["sa"], s["sb"])
    elif op in ("gemv", "sensitivity"):
        n, k, copies = case["n"], case["k"], case.get("copies", 3)
        w = _bf16(_normal(g, n, k, sigma=0.02))
        s["w"] = w.unsqueeze(0).expand(copies, n, k).contiguous()
        s["x"] = _bf16(_normal(g, k))
        s["out"] = torch.empty(n, dtype=torch.float32, device="cuda")
        s["desc"] = ctx.gemv_desc(s["w"], s["x"], s["out"], n, k, copies)
        if op == "sensitivity":
            e = 1 << 26                            # 256 MiB an array: the three pass the Infinity Cache
            sb, sc = _uniform(g, e), _uniform(g, e)
            s["opts"] = dict(src0=sb, src1=sc, dst=torch.empty_like(sb), n=e)
            s["ws"] = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    elif op == "rows":
        s["w"] = _bf16(_normal(g, case["rows"], case["k"], sigma=0.02))
        s["v"] = _bf16(_normal(g, case["batch"], case["k"]))
        s["res"] = _normal(g, case["batch"], case["rows"]) if case["res"] else None
        s["out"] = torch.empty((case["batch"], case["rows"]), dtype=torch.float32, device="cuda")
    elif op == "decode":
        cfg = dict(LLAMA if case["model"] == "llama" else SMALL, layers=case["layers"], vocab=case["vocab"],
                   batch=case["batch"], max_ctx=case["ctx"])
        s["model"] = coloc.DecodeModel(ctx, cfg, _positions(case), int(seed) * 4096,
                                       flags=coloc.DECODE_GRAPH if case["graph"] else 0)
    elif op == "attention":
        b, d = case["batch"], case["head_dim"]
        s["q"] = _uniform(g, b, case["n_q"], d) * 4.0
        s["k"] = _bf16(_uniform(g, b, case["n_kv"], case["ctx"], d))
        s["v"] = _bf16(_uniform(g, b, case["n_kv"], case["ctx"], d))
        s["out"] = torch.empty((b, case["n_q"] * d), dtype=torch.int16, device="cuda")
    elif op in ("quantize", "checksum"):
        s["x"] = _normal(g, case["n"])
    elif op == "serve":
        s["requests"] = _requests(case, seed)
    torch.cuda.synchronize()
    return s


# --------------------------------------------------------------------- run
def run(state):
    case, ctx, op = state["case"], state["ctx"], state["case"]["op"]
    if op == "triad":
        r = ctx.victim_run(state["desc"])
        return dict(a=state["out"], checksum=r.checksum_bits, sum=r.sum_f64)
    if op in ("gemm", "gemv"):
        ctx.victim_run(state["desc"])
        return state["out"]
    if op == "rows":
        return ctx.gemv_bf16_rows(state["w"], state["v"], res=state["res"], out=state["out"])
    if op == "decode":
        m = state["model"]
        ctx.decode_step(m)
        out = dict(x=m.x_out, k_cache=m.k_cache.view(torch.bfloat16), v_cache=m.v_cache.view(torch.bfloat16))
        if case["vocab"]:
            out["logits"] = m.logits
        return out
    if op == "attention":
        args = (state["q"], state["k"], state["v"], _positions(case), case["n_q"], case["n_kv"], case["head_dim"],
                case["ctx"], state["out"])
        (ctx.attention_decode_noalloc if case["noalloc"] else ctx.attention_decode)(*args)
        return state["out"].view(torch.bfloat16)
    if op == "quantize":
        codes, scale = ctx.quantize(state["x"], case["dtype"])
        return dict(codes=codes, scale=scale)
    if op == "checksum":
        bits, total = ctx.checksum(state["x"])
        return dict(bits=bits, sum=total)
    if op == "serve":
        done = ctx.serve(state["requests"], policy="naive", hbm_budget=case["budget"], slots=case["slots"])
        return dict(status=[r["status"] for r in done], out=[q["out_copy"] for q in state["requests"]])
    cell, = ctx.measure_sensitivity(state["desc"], [case["resource"]], [state["opts"]], [case["intensity"]],
                                    reps=case["reps"], warmups=2, deadline_ms=200, ws=state["ws"])
    return dict(y=state["out"], ncu=cell["ncu"], output_equal=cell["output_equal"], reps=cell["reps"])


# -------------------------------------------------------------------- work
def _victim_work(kind, q):
    """Operands read once, the output written once and read once more for its checksum."""
    if kind == "triad":
        return q["n"] * 16, 2 * q["n"]
    if kind == "gemm":
        e = {"f32": 4, "bf16": 2, "fp8": 1}[q["dtype"]]
        return (q["m"] + q["n"]) * q["k"] * e + 8 * q["m"] * q["n"], 2 * q["m"] * q["n"] * q["k"]
    return 2 * q["n"] * q["k"] + 2 * q["k"] + 8 * q["n"], 2 * q["n"] * q["k"]


def work(case):
    op = case["op"]
    if op in ("triad", "gemm", "gemv"):
        b, f = _victim_work(op, case)
        if op == "triad":                          # every sweep streams the arrays, unless one launch keeps them near
            extra = 0 if case["in_kernel"] else (case["passes"] - 1) * 12 * case["n"]
            b, f = b + extra, f * case["passes"]
        return dict(bytes=b, flops=f)
    if op == "rows":
        b = 2 * case["rows"] * case["k"] + 2 * case["batch"] * case["k"] + 4 * case["batch"] * case["rows"] * (
            2 if case["res"] else 1)
        return dict(bytes=b, flops=2 * case["rows"] * case["k"] * case["batch"])
    if op == "decode":
        c = LLAMA if case["model"] == "llama" else SMALL
        hid, d = c["hidden"], c["head_dim"]
        w = case["layers"] * hid * ((2 * c["n_q"] + 2 * c["n_kv"]) * d + 3 * c["ffn"]) + case["vocab"] * hid
        att = sum(p + 1 for p in _positions(case)) * case["layers"] * d
        return dict(bytes=2 * w + 4 * att * c["n_kv"] + 4 * case["batch"] * (2 * hid + 2 * case["vocab"]),
                    flops=2 * w * case["batch"] + 4 * att * c["n_q"])
    if op == "attention":
        att = sum(p + 1 for p in _positions(case)) * case["head_dim"]
        return dict(bytes=4 * att * case["n_kv"] + 6 * case["batch"] * case["n_q"] * case["head_dim"],
                    flops=4 * att * case["n_q"])
    if op == "quantize":                           # FP8 reads the input for its maximum and again to convert it
        return dict(bytes=case["n"] * (9 if case["dtype"] == "fp8" else 6), flops=2 * case["n"])
    if op == "checksum":
        return dict(bytes=4 * case["n"], flops=case["n"])
    if op == "serve":                              # inputs drawn (written) on the device, then each request's own work
        b = f = 0
        for q in _shapes(case):
            wb, wf = _victim_work(q["kind"], q)
            inputs = {"triad": 8 * q["n"], "gemm": 2 * (q.get("m", 0) + q["n"]) * q.get("k", 0),
                      "gemv": 2 * q["n"] * q.get("k", 0)}[q["kind"]]
            b, f = b + wb + inputs + 8 * (q.get("m", 1) * q["n"] if q["kind"] == "gemm" else q["n"]), f + wf
        return dict(bytes=b, flops=f)
    runs = 2 * case["reps"] + 2
    b, f = _victim_work("gemv", case)
    return dict(bytes=runs * b, flops=runs * f)


def _shapes(case):
    rng = random.Random(case["mix"])
    out = []
    for i in range(case["requests"]):
        if i % 3 == 0:
            s = round(_log(rng, 512, 8192) / 128) * 128
            out.append(dict(kind="gemm", dtype="bf16", m=s, n=s, k=s))
        elif i % 3 == 1:
            s = round(_log(rng, 4096, 16384) / 8) * 8
            out.append(dict(kind="gemv", dtype="bf16", n=s, k=s))
        else:
            out.append(dict(kind="triad", n=int(_log(rng, 1 << 20, 1 << 28))))
    rng.shuffle(out)
    return out


# ------------------------------------------------------------------- exact
def _q(x):
    return x.float().to(torch.bfloat16).double()


def _norm(x, g, eps):
    return _q(x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * g)


def _rope(x, pos, base):
    """x (heads, d): pair i of a head turns by pos * base^(-2i/d)."""
    h = x.shape[-1] // 2
    ang = pos * base ** (-2.0 * torch.arange(h, dtype=torch.float64, device=x.device) / (2 * h))
    a, b = x[..., :h], x[..., h:]
    return torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], -1)


def _attend(q, k, v):
    """q (n_q, d), k and v (n_kv, t, d)."""
    group = q.shape[0] // k.shape[0]
    out = []
    for h in range(k.shape[0]):
        p = torch.softmax(q[h * group:(h + 1) * group] @ k[h].T / math.sqrt(q.shape[1]), -1)
        out.append(p @ v[h])
    return torch.cat(out)


def _decode_exact(case, model):
    """The decode step in FP64, rounded to BF16 where the model stores BF16.
    `model` is read for its inputs only."""
    cfg, lay = model.cfg, model.layout
    hid, nq, nkv, d, f = cfg["hidden"], cfg["n_q"], cfg["n_kv"], cfg["head_dim"], cfg["ffn"]
    batch, ctx = case["batch"], case["ctx"]
    arena = model.weights.view(torch.bfloat16)
    caches = [c.view(torch.bfloat16).view(case["layers"], batch, nkv, ctx, d) for c in (model.k_cache, model.v_cache)]

    def tensor(name, layer, *shape):
        off = int(getattr(lay, name) + layer * lay.layer_stride)
        return arena[off:off + math.prod(shape)].view(*shape).double()

    x = model.x_in.double()
    for l in range(case["layers"]):
        y = _norm(x, tensor("g_attn", l, hid), cfg["eps"])
        qkv = (y @ tensor("w_qkv", l, (nq + 2 * nkv) * d, hid).T).view(batch, nq + 2 * nkv, d)
        att = torch.empty(batch, nq * d, dtype=torch.float64, device=x.device)
        for b, p in enumerate(_positions(case)):
            k, v = (c[l, b, :, :p + 1].double() for c in caches)
            k[:, p] = _q(_rope(qkv[b, nq:nq + nkv], p, cfg["rope_base"]))
            v[:, p] = _q(qkv[b, nq + nkv:])
            att[b] = _q(_attend(_rope(qkv[b, :nq], p, cfg["rope_base"]), k, v)).reshape(-1)
        x = x + att @ tensor("w_o", l, hid, nq * d).T
        gu = _norm(x, tensor("g_mlp", l, hid), cfg["eps"]) @ tensor("w_gu", l, 2 * f, hid).T
        h = _q(gu[:, :f] * torch.sigmoid(gu[:, :f]) * gu[:, f:])
        x = x + h @ tensor("w_down", l, hid, f).T
    out = dict(x=x, k_cache=None, v_cache=None)
    if case["vocab"]:
        y = _norm(x, arena[int(lay.g_final):int(lay.g_final) + hid].double(), cfg["eps"])
        off = int(lay.w_lm)
        out["logits"] = torch.cat([y @ w.double().T for w in
                                   arena[off:off + case["vocab"] * hid].view(case["vocab"], hid).split(16384)], -1)
    return out


def exact(case, seed):
    op = case["op"]
    if op == "serve":          # the loop draws its inputs itself
        return None
    s = prepare(case, seed)
    if op == "triad":
        # the output is FP32 by definition (two roundings), and its sum is over those FP32 values
        a = s["b"] + 3.0 * s["c"]
        return dict(a=a.double(), checksum=None, sum=float(a.double().sum()))
    if op == "gemm":
        return s["sa"] * s["sb"] * (s["va"].float().double() @ s["vb"].float().double().T)
    if op in ("gemv", "sensitivity"):
        y = s["w"][0].view(torch.bfloat16).double() @ s["x"].view(torch.bfloat16).double()
        return y if op == "gemv" else dict(y=y, ncu=None, output_equal=None, reps=None)
    if op == "rows":
        y = s["v"].view(torch.bfloat16).double() @ s["w"].view(torch.bfloat16).double().T
        return y if s["res"] is None else y + s["res"].double()
    if op == "decode":
        return _decode_exact(case, s["model"])
    if op == "attention":
        kc, vc = s["k"].view(torch.bfloat16), s["v"].view(torch.bfloat16)
        return torch.stack([_attend(s["q"][b].double(), kc[b, :, :p + 1].double(), vc[b, :, :p + 1].double()).reshape(-1)
                            for b, p in enumerate(_positions(case))])
    if op == "quantize":
        return dict(codes=None, scale=float(s["x"].abs().max().double() / 448.0) if case["dtype"] == "fp8" else 1.0)
    return dict(bits=None, sum=float(s["x"].double().sum()))
