"""The work that users of this library have it do, as a set of measurable cases.

Every case runs through the package's Python entry points (`laq`, `decode`).
Decode-time cases replay a HIP graph that `prepare` captured, as a serving loop
does; the one-linear, quantize and pack cases are ordinary eager calls.

Shapes are those of `inputs.py` (Qwen3-4B and Qwen3-32B decoder layers, the
1024 x 1024 single linear) and generic ones.  Weights and activations follow
`inputs.py`'s distributions (N(0, 0.02) with 1 % x10 outliers; N(0, 1)).
"""
import math

import torch

from paper_2605_08755_amd import decode, laq

DEV = "cuda:0"
GROUP = 128
HEAD = 128
EPS = 1e-6

# Decoder shapes: hidden, query heads, key/value heads, MLP width, vocabulary.
SHAPES = {
    "4b": {"hidden": 2560, "heads": 32, "kv_heads": 8, "mlp": 9728},
    "32b": {"hidden": 5120, "heads": 64, "kv_heads": 8, "mlp": 25600},
}
VOCAB = 151936


def listed():
    return [
        # One small linear called eagerly from Python: the latency of a call.
        {"name": "single_w3_m1", "kind": "linear", "bits": 3, "M": 1, "N": 1024, "K": 1024, "copies": 1,
         "graph": False},
        # The linears of one decode step at batch 1: 36 Qwen3-4B layers of
        # q|k|v, o, gate|up, down (the benchmark's headline workload).
        {"name": "stack4b_w3_m1", "kind": "stack", "model": "4b", "bits": 3, "M": 1, "layers": 36,
         "grouped": False},
        # The same at batch 4 in 4 bits, with separate q, k, v and gate, up
        # weights that one grouped launch each serves.
        {"name": "grouped4b_w4_m4", "kind": "stack", "model": "4b", "bits": 4, "M": 4, "layers": 12,
         "grouped": True},
        # Large layers at the largest batch: 8 Qwen3-32B layers, 16 rows.
        {"name": "stack32b_w3_m16", "kind": "stack", "model": "32b", "bits": 3, "M": 16, "layers": 8,
         "grouped": False},
        # Odd sizes: 7 rows, an output count that fills no tile, 25 groups.
        {"name": "ragged_w4_m7", "kind": "linear", "bits": 4, "M": 7, "N": 3001, "K": 3200, "copies": 24,
         "graph": True},
        # The LM head (hidden 2560 -> 151936 logits) for eight sequences.
        {"name": "head_w3_m8", "kind": "linear", "bits": 3, "M": 8, "N": VOCAB, "K": 2560, "copies": 1,
         "graph": False},
        # The MLP blocks of 12 layers for a batch of 12 tokens: residual add +
        # RMSNorm, gate|up, SiLU-and-multiply, down.
        {"name": "mlp4b_w3_m12", "kind": "mlp", "bits": 3, "M": 12, "D": 2560, "I": 9728, "layers": 12},
        # A whole batch-1 decode step: 12 Qwen3-4B layers at context 1024 and
        # the LM head, with the fused norm, SiLU and residual linears.
        {"name": "decode4b_w3_ctx1024", "kind": "decode", "model": "4b", "bits": 3, "layers": 12, "ctx": 1024},
        # One token's attention at a short context, 64 query heads (the 32B
        # layer), 36 layers: many small launches.
        {"name": "attention_ctx300", "kind": "attention", "heads": 64, "kv_heads": 8, "ctx": 300, "layers": 36},
        # One token's attention over a long context, four 4B layers.
        {"name": "attention_ctx32768", "kind": "attention", "heads": 32, "kv_heads": 8, "ctx": 32768, "layers": 4},
        # Quantizing a large matrix when a model is loaded (32B gate|up).
        {"name": "quantize_w3_gateup32b", "kind": "quantize", "bits": 3, "N": 51200, "K": 5120},
        # Packing trained parameters of a mid-sized matrix, 4 bits, odd sizes.
        {"name": "pack_w4_odd", "kind": "pack", "bits": 4, "N": 6007, "K": 3712},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _groups(rng, lo, hi):
    """A multiple of 128 between lo and hi groups, odd group counts included."""
    return GROUP * max(1, _log_int(rng, lo, hi))


def draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "stack", "mlp", "decode", "attention", "attention", "quantize",
                       "pack"])
    bits = rng.choice([3, 3, 4])
    if kind == "linear":
        K = _groups(rng, 4, 224)
        N = _log_int(rng, 256, min(VOCAB, 3 * 10**8 // K))
        copies = max(1, min(24, 3 * 10**8 // (N * K)))
        return {"kind": kind, "bits": bits, "M": rng.randint(1, 16), "N": N, "K": K, "copies": copies,
                "graph": copies > 1}
    if kind == "stack":
        model = rng.choice(["4b", "32b"])
        layers = rng.randint(4, 24) if model == "4b" else rng.randint(2, 6)
        return {"kind": kind, "model": model, "bits": bits, "M": rng.randint(1, 16), "layers": layers,
                "grouped": rng.random() < 0.3}
    if kind == "mlp":
        D, I = _groups(rng, 6, 40), _groups(rng, 12, 200)
        layers = max(1, min(12, 4 * 10**8 // (D * I)))
        return {"kind": kind, "bits": bits, "M": rng.randint(2, 16), "D": D, "I": I, "layers": layers}
    if kind == "decode":
        model = rng.choice(["4b", "32b"])
        layers = rng.randint(2, 12) if model == "4b" else rng.randint(1, 3)
        return {"kind": kind, "model": model, "bits": bits, "layers": layers, "ctx": _log_int(rng, 20, 8192)}
    if kind == "attention":
        kv = rng.choice([1, 2, 4, 8])
        ctx = _log_int(rng, 16, 40960)
        layers = max(1, min(36, 2**20 // (kv * ctx)))
        return {"kind": kind, "heads": kv * rng.choice([1, 2, 4, 8]), "kv_heads": kv, "ctx": ctx, "layers": layers}
    K = _groups(rng, 4, 200)
    N = _log_int(rng, 256, min(51200, 26 * 10**7 // K))
    return {"kind": kind, "bits": bits, "N": N, "K": K}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1009 + 17)
    return g


def _weights(g, N, K):
    w = torch.randn((N, K), generator=g, device=DEV, dtype=torch.float32).mul_(0.02)
    return torch.where(torch.rand((N, K), generator=g, device=DEV) < 0.01, w * 10, w).to(torch.float16)


def _acts(g, *shape):
    return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32).to(torch.float16)


def _norm_weight(g, n):
    return (1.0 + 0.1 * torch.randn((n,), generator=g, device=DEV)).to(torch.float16)


def _linear_inputs(case, seed):
    """(w, x) of each copy."""
    g = _gen(seed)
    for _ in range(case["copies"]):
        w = _weights(g, case["N"], case["K"])
        yield w, _acts(g, case["M"], case["K"])


def _stack_shapes(case):
    """Calls of one layer: (row counts of the weights that share x, K)."""
    s = SHAPES[case["model"]]
    D, q, kv, I = s["hidden"], s["heads"] * HEAD, s["kv_heads"] * HEAD, s["mlp"]
    return [((q, kv, kv), D), ((D,), q), ((I, I), D), ((D,), I)]


def _stack_inputs(case, seed):
    """(weights, x) of each call: the weights separate, in order."""
    g = _gen(seed)
    for _ in range(case["layers"]):
        for Ns, K in _stack_shapes(case):
            ws = [_weights(g, N, K) for N in Ns]
            yield ws, _acts(g, case["M"], K)


def _mlp_inputs(case, seed):
    """The embedding rows, then (norm weight, gate|up, down) of each layer."""
    g = _gen(seed)
    D, I = case["D"], case["I"]
    yield torch.randn((case["M"], D), generator=g, device=DEV, dtype=torch.float32)
    for _ in range(case["layers"]):
        nw = _norm_weight(g, D)
        gu = _weights(g, 2 * I, D)
        yield nw, gu, _weights(g, D, I)


def _s_max(ctx):
    return (ctx + 255) // 256 * 256


def _attention_inputs(case, seed):
    """(qkv, q norm, k norm, caches [2][Hkv][S_max][128]) of each layer."""
    g = _gen(seed)
    Hq, Hkv = case["heads"], case["kv_heads"]
    for _ in range(case["layers"]):
        qkv = _acts(g, (Hq + 2 * Hkv) * HEAD)
        qn, kn = _norm_weight(g, HEAD), _norm_weight(g, HEAD)
        yield qkv, qn, kn, _acts(g, 2, Hkv, _s_max(case["ctx"]), HEAD)


def _decode_inputs(case, seed):
    """The embedding, then per layer the norms, the cache and the four weights
    (gate and up rows interleaved), then the final norm and the head."""
    g = _gen(seed)
    s = SHAPES[case["model"]]
    D, Hq, Hkv, I = s["hidden"], s["heads"], s["kv_heads"], s["mlp"]
    yield torch.randn((1, D), generator=g, device=DEV, dtype=torch.float32)
    for _ in range(case["layers"]):
        norms = (_norm_weight(g, D), _norm_weight(g, D), _norm_weight(g, HEAD), _norm_weight(g, HEAD))
        cache = _acts(g, 2, Hkv, _s_max(case["ctx"]), HEAD)
        ws = [_weights(g, (Hq + 2 * Hkv) * HEAD, D), _weights(g, D, Hq * HEAD), _weights(g, 2 * I, D),
              _weights(g, D, I)]
        yield norms, cache, ws
    yield _norm_weight(g, D), _weights(g, VOCAB, D)


def _capture(fn):
    """fn's launches as a HIP graph, after one eager pass."""
    fn()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        fn()
    return graph


def _decode_callables(packed, bits):
    """A layer's four callables for decode.DecodeStep: the norms inside q|k|v
    and gate|up, SiLU inside gate|up, o and down adding to the residual."""
    def with_norm(p, swiglu):
        def f(x, out):
            return laq.linear_swiglu(x, *p, bits, out=out) if swiglu else laq.linear(x, *p, bits, out=out)
        f.swiglu = swiglu
        f.norm_linear = lambda res, delta, w, eps, res_out, out: laq.add_rmsnorm_linear(
            res, delta, w, eps, *p, bits, swiglu=swiglu, out=out, residual_out=res_out)
        return f

    def with_residual(p):
        def f(x, out):
            return laq.linear(x, *p, bits, out=out)
        f.residual_linear = lambda x, r_in, r_out, out: laq.linear_residual(x, *p, r_in, r_out, bits,
                                                                            write_out=False)
        return f

    qkv, o, gu, down = packed
    return with_norm(qkv, False), with_residual(o), with_norm(gu, True), with_residual(down)


def prepare(case, seed):
    kind, st = case["kind"], {"case": case}
    if kind == "linear":
        bits = case["bits"]
        calls = [(x, laq.quantize(w, bits)) for w, x in _linear_inputs(case, seed)]
        st["calls"] = calls
        if case["graph"]:
            ys = [torch.empty((case["M"], case["N"]), dtype=torch.float16, device=DEV) for _ in calls]

            def fn():
                for (x, p), y in zip(calls, ys):
                    laq.linear(x, *p, bits, out=y)
            st["graph"], st["out"] = _capture(fn), ys
    elif kind == "stack":
        bits, calls, outs = case["bits"], [], []
        M, per = case["M"], _stack_shapes(case)
        # one output tensor per call of a layer and weight, all layers in it
        for Ns, _ in per:
            for N in (Ns if case["grouped"] else (sum(Ns),)):
                outs.append(torch.empty((case["layers"], M, N), dtype=torch.float16, device=DEV))
        slots = [len(Ns) if case["grouped"] else 1 for Ns, _ in per]
        for i, (ws, x) in enumerate(_stack_inputs(case, seed)):
            layer, j = divmod(i, len(per))
            first = sum(slots[:j])
            ys = [outs[first + k][layer] for k in range(slots[j])]
            ws = ws if case["grouped"] else [torch.cat(ws)]
            calls.append(([(x,) + laq.quantize(w, bits) for w in ws], ys))

        def fn():
            for group, ys in calls:
                if len(group) == 1:
                    laq.linear(*group[0], bits, out=ys[0])
                else:
                    laq.linear_group(group, bits, outs=ys)
        st["calls"], st["graph"], st["out"] = calls, _capture(fn), outs
    elif kind == "mlp":
        bits, D, I, M = case["bits"], case["D"], case["I"], case["M"]
        it = _mlp_inputs(case, seed)
        x0 = next(it)
        layers = [(nw, laq.quantize(gu, bits), laq.quantize(dn, bits)) for nw, gu, dn in it]
        res = torch.empty_like(x0)
        h, y = (torch.empty((M, D), dtype=torch.float16, device=DEV) for _ in range(2))
        gu, m = (torch.empty((M, n), dtype=torch.float16, device=DEV) for n in (2 * I, I))

        def fn():
            res.copy_(x0)
            delta = None
            for nw, pgu, pdn in layers:
                laq.add_rmsnorm(res, delta, nw, EPS, out=h)
                laq.linear(h, *pgu, bits, out=gu)
                laq.silu_mul(gu, out=m)
                delta = laq.linear(m, *pdn, bits, out=y)
        st["keep"], st["graph"], st["out"] = (x0, layers, h, gu, m), _capture(fn), [res, y]
    elif kind == "attention":
        Hq, Hkv, pos = case["heads"], case["kv_heads"], case["ctx"] - 1
        layers = list(_attention_inputs(case, seed))
        cs = decode.rope_table(_s_max(case["ctx"]), 1e6, DEV)
        out = torch.empty((len(layers), Hq, HEAD), dtype=torch.float16, device=DEV)
        ws = torch.empty(laq.attention_qkv_workspace_bytes(Hq, Hkv, _s_max(case["ctx"])), dtype=torch.uint8,
                         device=DEV)

        def fn():
            for l, (qkv, qn, kn, c) in enumerate(layers):
                laq.decode_attention_qkv(qkv, qn, kn, cs, pos, Hq, Hkv, EPS, c[0], c[1], out=out[l], workspace=ws)
        rows = [c[:, :, pos] for _, _, _, c in layers]  # the rows appended to the caches
        st["keep"], st["graph"], st["out"] = (layers, cs, ws), _capture(fn), [out] + rows
    elif kind == "decode":
        bits, s = case["bits"], SHAPES[case["model"]]
        shape = dict(s, layers=case["layers"], eps=EPS, rope_theta=1e6, vocab=VOCAB)
        it = _decode_inputs(case, seed)
        x0 = next(it)
        norms, caches, linears = [], [], []
        for _ in range(case["layers"]):
            n, c, ws = next(it)
            norms.append(n)
            caches.append(c)
            linears.append(_decode_callables([laq.quantize(w, bits) for w in ws], bits))
        final_norm, head = next(it)
        head = laq.quantize(head, bits)
        step = decode.DecodeStep(shape, linears, norms, final_norm, [c[0] for c in caches], [c[1] for c in caches],
                                 DEV, lm_head=lambda x, out: laq.linear(x, *head, bits, out=out))
        step.x0.copy_(x0)
        pos = case["ctx"] - 1
        graph = _capture(lambda: step.run(pos))
        st["keep"], st["graph"] = step, graph
        st["out"] = [step.logits, step.residual] + [c[:, :, pos] for c in caches]
    else:
        w = _weights(_gen(seed), case["N"], case["K"])
        st["w"] = w
        if kind == "pack":
            # parameters as training leaves them: near min-max, not equal to it
            s, z = _min_max(w, case["bits"])
            st["s"], st["z"] = (s.float() * 0.9).clamp_min(2.0**-24).to(torch.float16), z
    torch.cuda.synchronize()
    return st


def run(st):
    case = st["case"]
    if "graph" in st:
        st["graph"].replay()
        return st["out"]
    if case["kind"] == "linear":
        return [laq.linear(x, *p, case["bits"]) for x, p in st["calls"]]
    if case["kind"] == "quantize":
        return laq.quantize(st["w"], case["bits"])
    return laq.pack(st["w"], st["s"], st["z"], case["bits"])


# ---------------------------------------------------------------------------
# work
# ---------------------------------------------------------------------------
def _weight_bytes(N, K, bits):
    return N * K * bits / 8 + N * (K // GROUP) * 3


def _linear_bytes(M, N, K, bits):
    return _weight_bytes(N, K, bits) + 2 * M * (N + K)


def _attention_work(Hq, Hkv, L):
    return 2 * 2 * Hkv * L * HEAD + 2 * (2 * Hq + 2 * Hkv) * HEAD, 4 * Hq * L * HEAD


def work(case):
    kind, bits = case["kind"], case.get("bits", 0)
    if kind == "linear":
        M, N, K, n = case["M"], case["N"], case["K"], case["copies"]
        return {"bytes": n * _linear_bytes(M, N, K, bits), "flops": n * 2.0 * M * N * K}
    if kind == "stack":
        M, n = case["M"], case["layers"]
        shapes = [(sum(Ns), K) for Ns, K in _stack_shapes(case)]
        return {"bytes": n * sum(_linear_bytes(M, N, K, bits) for N, K in shapes),
                "flops": n * sum(2.0 * M * N * K for N, K in shapes)}
    if kind == "mlp":
        M, D, I, n = case["M"], case["D"], case["I"], case["layers"]
        # the block's weights; the residual rows in and out and the last
        # layer's output (what lies between stays on the chip at best)
        return {"bytes": n * (_weight_bytes(2 * I, D, bits) + _weight_bytes(D, I, bits)) + 10 * M * D,
                "flops": n * 6.0 * M * D * I}
    if kind == "attention":
        b, f = _attention_work(case["heads"], case["kv_heads"], case["ctx"])
        return {"bytes": case["layers"] * b, "flops": float(case["layers"] * f)}
    if kind == "decode":
        s, n = SHAPES[case["model"]], case["layers"]
        shapes = [(sum(Ns), K) for Ns, K in _stack_shapes(case)]
        b, f = _attention_work(s["heads"], s["kv_heads"], case["ctx"])
        head = (VOCAB, s["hidden"])
        return {"bytes": n * (sum(_weight_bytes(N, K, bits) for N, K in shapes) + b) + _weight_bytes(*head, bits)
                + 2 * VOCAB + 8 * s["hidden"],
                "flops": n * (sum(2.0 * N * K for N, K in shapes) + f) + 2.0 * head[0] * head[1]}
    N, K = case["N"], case["K"]
    # per weight: a subtraction or comparison, a division, a rounding, a clip
    return {"bytes": 2.0 * N * K + _weight_bytes(N, K, bits), "flops": 4.0 * N * K}


# fp16 outputs of fp32 sums: the rounding alone is 2.1e-4 of the result's norm
# (measured against 64 bits); chains of several such roundings add up: 3e-4 in
# attention (q), 2.6e-3 over 12 MLP layers, 1.9e-3 over a 12-layer decode
# step.  The bounds are about four times what was measured.
def tolerance(case):
    if case["kind"] in ("quantize", "pack"):
        return "exact"  # codes, scales and zero points are defined bit by bit
    return {"linear": {"rel": 8e-4, "max": 8e-3}, "stack": {"rel": 8e-4, "max": 8e-3},
            "attention": {"rel": 1.2e-3, "max": 1.2e-2}, "mlp": {"rel": 1e-2, "max": 1e-1},
            "decode": {"rel": 8e-3, "max": 8e-2}}[case["kind"]]


# ---------------------------------------------------------------------------
# the same results in 64 bits, in plain torch
# ---------------------------------------------------------------------------
def _min_max(w, bits):
    """Eq. 1's parameters of every group: fp16 scales, uint8 zero points, by
    fp32 arithmetic (a quotient of floats rounded from a double is the
    correctly rounded one)."""
    qmax = 2**bits - 1
    v = w.view(w.shape[0], -1, GROUP)
    lo = v.amin(-1).float().clamp_max(0)
    hi = v.amax(-1).float().clamp_min(0)
    s = ((hi - lo).double() / qmax).float().to(torch.float16)
    s = torch.where(s == 0, torch.full_like(s, 2.0**-24), s)
    z = torch.round((-lo.double() / s.double()).float()).clamp(0, qmax)
    return s, z.to(torch.uint8)


def _w_hat(w, bits):
    """The dequantized weights s (q - z), fp64."""
    qmax = 2**bits - 1
    s, z = _min_max(w, bits)
    v = w.view(w.shape[0], -1, GROUP).double()
    s, z = s.double().unsqueeze(-1), z.double().unsqueeze(-1)
    q = (torch.round((v / s).float().double()) + z).clamp(0, qmax)
    return (s * (q - z)).view(w.shape)


def _mul(x, w, bits):
    """x w_hat^T in fp64, by rows of w in pieces of bounded size."""
    step = max(1, 2**27 // w.shape[1])
    return torch.cat([x.double() @ _w_hat(w[i:i + step], bits).t() for i in range(0, w.shape[0], step)], dim=1)


def _rms(x, w):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * w.double()


def _silu(g):
    return g / (1 + torch.exp(-g))


def _attend(qkv, qn, kn, cache, cs, pos, Hq, Hkv):
    """(out [Hq][128], appended rows [2][Hkv][128]); cs: cos, sin of pos."""
    c, s = cs
    q, k, v = qkv.double().view(-1, HEAD).split([Hq, Hkv, Hkv])

    def rot(x, w):
        x = _rms(x, w)
        a, b = x[:, :64], x[:, 64:]
        return torch.cat([a * c - b * s, b * c + a * s], dim=1)
    q, k = rot(q, qn), rot(k, kn)
    out = []
    for h in range(Hkv):  # one key/value head at a time
        ks = torch.cat([cache[0, h, :pos].double(), k[h:h + 1]])
        vs = torch.cat([cache[1, h, :pos].double(), v[h:h + 1]])
        R = Hq // Hkv
        p = torch.softmax(q[h * R:(h + 1) * R] @ ks.t() / math.sqrt(HEAD), dim=-1)
        out.append(p @ vs)
    return torch.cat(out), torch.stack([k, v])


def _rope_row(pos):
    a = pos * torch.pow(torch.tensor(1e6, dtype=torch.float64, device=DEV),
                        -2.0 * torch.arange(64, dtype=torch.float64, device=DEV) / HEAD)
    return torch.cos(a), torch.sin(a)


def exact(case, seed):
    kind, bits = case["kind"], case.get("bits", 0)
    if kind == "linear":
        return [_mul(x, w, bits) for w, x in _linear_inputs(case, seed)]
    if kind == "stack":
        per = len(_stack_shapes(case))
        cols = [[] for _ in range(per)]
        for i, (ws, x) in enumerate(_stack_inputs(case, seed)):
            ys = [_mul(x, w, bits) for w in ws]
            cols[i % per].append(ys if case["grouped"] else [torch.cat(ys, dim=1)])
        return [torch.stack([layer[k] for layer in col]) for col in cols for k in range(len(col[0]))]
    if kind == "mlp":
        it = _mlp_inputs(case, seed)
        res = next(it).double()
        y = None
        I = case["I"]
        for nw, gu, dn in it:
            if y is not None:
                res = res + y
            a = _mul(_rms(res, nw), gu, bits)
            y = _mul(_silu(a[:, :I]) * a[:, I:], dn, bits)
        return [res, y]
    if kind == "attention":
        pos = case["ctx"] - 1
        got = [_attend(qkv, qn, kn, c, _rope_row(pos), pos, case["heads"], case["kv_heads"])
               for qkv, qn, kn, c in _attention_inputs(case, seed)]
        return [torch.stack([o for o, _ in got])] + [r for _, r in got]
    if kind == "decode":
        s, pos = SHAPES[case["model"]], case["ctx"] - 1
        it = _decode_inputs(case, seed)
        res, rows = next(it).double(), []
        for _ in range(case["layers"]):
            (w_in, w_post, qn, kn), cache, (qkv, o, gu, dn) = next(it)
            a = _mul(_rms(res, w_in), qkv, bits)
            a, r = _attend(a[0], qn, kn, cache, _rope_row(pos), pos, s["heads"], s["kv_heads"])
            rows.append(r)
            res = res + _mul(a.reshape(1, -1), o, bits)
            a = _mul(_rms(res, w_post), gu, bits)
            res = res + _mul(_silu(a[:, 0::2]) * a[:, 1::2], dn, bits)
        final_norm, head = next(it)
        return [_mul(_rms(res, final_norm), head, bits), res] + rows
    if kind == "quantize":
        return [None, _min_max(_weights(_gen(seed), case["N"], case["K"]), bits)[0].double(), None]
    return None  # packed words only
