"""What the speed of this library is measured on.

A case is one call (or the short chain of calls) a program that serves or prefills a
Switch-Transformer-shaped mixture-of-experts model makes through the C ABI's binding:

  kind "step"   pgmoe_stack_step over `L` pre-gated MoE blocks of `T` tokens: gate, token grouping,
                expert FFN, weighted combine and residual.  L = 1 is one MoE block by itself.
                store "hbm": experts resident; "host": experts in pinned host memory, migrated.
  kind "ffn"    pgmoe_expert_ffn alone on rows that are already grouped.
  kind "gate"   pgmoe_pregate_topk alone, with or without the full softmax.
  kind "group"  pgmoe_permute followed by pgmoe_combine: what a program with experts of its own uses.

Shapes: Switch-Base (d_model 768, d_ff 3072, 8 / 64 / 128 / 256 experts) and Switch-Large (1024,
4096, 128 experts), the small and wide neighbours (512, 2048) and (2048, 8192) the library is also
built for, and the tiny float32 stack (64, 256) the repository checks itself on.

Expert weights are drawn directly as blobs: the blob is a permutation of the two matrices
(documented in pgmoe.h), so independent normal values make the same distribution either way.
`exact` undoes the permutation.
"""
import math

import torch

from paper_2308_12066_amd import binding as B

DIMS = ((64, 256), (512, 2048), (768, 3072), (1024, 4096), (2048, 8192))


def listed():
    return [
        # one token through the six MoE blocks of Switch-Base-8's encoder or decoder: latency
        _step("decode_base8_t1", 768, 3072, 8, 1, 6, 1),
        # the same with the experts in host memory, the design point of the method
        _step("decode_base8_t1_host", 768, 3072, 8, 1, 6, 1, store="host"),
        # a small serving batch on Switch-Base-64, popular and unpopular experts
        _step("decode_base64_t16", 768, 3072, 64, 1, 6, 16, zipf=1.1),
        # a serving batch on Switch-Large-128, two experts per token
        _step("decode_large128_t64_top2", 1024, 4096, 128, 2, 2, 64, zipf=1.1),
        # the float32 stack: the smallest one, and the shape and precision of the published Switch-Base-8
        _step("step_tiny_f32", 64, 256, 8, 1, 2, 32, dtype="f32"),
        _step("block_base8_t100_f32", 768, 3072, 8, 1, 1, 100, dtype="f32"),
        # prefill of 8 sequences of 512 tokens: 32 rows per expert, bound by the weights
        _step("prefill_base128_t4096", 768, 3072, 128, 1, 1, 4096),
        # a ragged prefill with some ninety rows per expert, two experts per token
        _step("prefill_base64_t3001_top2", 768, 3072, 64, 2, 1, 3001, zipf=1.1),
        # prefill of 8 sequences of 512 tokens on 8 experts: bound by the matrix cores
        _step("prefill_base8_t4096", 768, 3072, 8, 1, 1, 4096),
        # a large prefill on Switch-Large-128, two experts per token
        _step("prefill_large128_t16384_top2", 1024, 4096, 128, 2, 1, 16384),
        # the gate by itself over a prefill batch, with the probabilities of every expert
        {"name": "gate_large128_t4096", "kind": "gate", "dtype": "bf16", "d": 1024, "E": 128, "k": 2, "T": 4096, "zipf": 1.1, "probs": True},
        # grouping and combining around experts of the caller's own
        {"name": "group_combine_t8191_top2", "kind": "group", "dtype": "bf16", "d": 768, "E": 64, "k": 2, "T": 8191, "zipf": 1.1},
    ]


def _step(name, d, f, E, k, L, T, dtype="bf16", zipf=0.0, store="hbm"):
    return {"name": name, "kind": "step", "dtype": dtype, "d": d, "f": f, "E": E, "k": k, "L": L, "T": T, "zipf": zipf, "store": store}


def draw(rng):
    def log_int(lo, hi):
        return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    zipf = rng.choice((0.0, 1.1))
    what = rng.choice(("decode", "decode", "prefill", "prefill", "prefill", "ffn", "f32", "host", "gate", "group"))
    if what == "f32":
        d, f = rng.choice(DIMS[:4])
        return _pure(_step("", d, f, rng.choice((8, 16, 64)), rng.choice((1, 2)), 1, log_int(1, 128), dtype="f32", zipf=zipf))
    if what == "gate":
        d = rng.choice((512, 768, 1024, 2048))
        return {"kind": "gate", "dtype": rng.choice(("bf16", "bf16", "f32")), "d": d, "E": rng.choice((8, 64, 128, 256)),
                "k": rng.choice((1, 2)), "T": log_int(1, 8192), "zipf": zipf, "probs": rng.choice((True, False))}
    if what == "group":
        return {"kind": "group", "dtype": rng.choice(("bf16", "bf16", "f32")), "d": rng.choice((512, 768, 1024, 2048)),
                "E": rng.choice((8, 64, 128, 256)), "k": rng.choice((1, 2, 4)), "T": log_int(8, 16384), "zipf": zipf}
    if what == "host":
        d, f = rng.choice(DIMS[1:4])
        return _pure(_step("", d, f, 8, 1, rng.choice((2, 4, 6)), log_int(1, 8), zipf=zipf, store="host"))
    while True:
        d, f = rng.choice(DIMS[1:])
        E, k = rng.choice((8, 16, 32, 64, 128, 256)), rng.choice((1, 1, 2))
        T = log_int(1, 128) if what == "decode" else log_int(129, 16384)
        L = rng.choice((2, 6)) if what == "decode" else 1
        if E * L * 4 * d * f > 3.3e9 or 4.0 * T * k * d * f > 5.5e11:  # at most the largest listed case's weights and products
            continue
        if what == "ffn":
            return {"kind": "ffn", "dtype": "bf16", "d": d, "f": f, "E": E, "rows": min(T, 8192), "zipf": zipf}
        return _pure(_step("", d, f, E, k, L, T, zipf=zipf))


def _pure(c):
    del c["name"]
    return c


# ----------------------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(1_000_003 * int(seed) + 17)


def _dt(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _normal(case, g, shape, scale):
    return torch.randn(shape, generator=g, device="cuda", dtype=_dt(case)).mul_(scale)


def _zipf_bias(case, g):
    """Logit bias that makes the experts' popularity roughly Zipf-shaped, in an order of its own; None without a skew."""
    E = case["E"]
    if not case["zipf"]:
        return None
    q = torch.arange(1, E + 1, dtype=torch.float64, device="cuda") ** -case["zipf"]
    perm = torch.randperm(E, generator=g, device="cuda")
    scale = 0.75 * E ** -0.08  # fitted: the most popular expert wins as often as its Zipf share says, over normal logits
    return (scale * 0.02 * math.sqrt(case["d"]) * torch.log(q / q.sum())[perm]).float()


def _blobs(case, g, n_blocks):
    """The packed experts [n_blocks, E, 2*d*f] in HBM: W1 and W2 ~ N(0, 0.02)."""
    out = torch.empty((n_blocks, case["E"], 2 * case["d"] * case["f"]), dtype=_dt(case), device="cuda")
    for b in range(n_blocks):
        out[b].normal_(0.0, 0.02, generator=g)
    return out


def _routing(case, g, T, k):
    """Top-k routing [T, k] as a gate over skewed logits would give it, and probabilities."""
    z = torch.randn((T, case["E"]), generator=g, device="cuda") * (0.02 * math.sqrt(case["d"]))
    bias = _zipf_bias(case, g)
    z = z if bias is None else z + bias
    p, idx = torch.softmax(z, dim=1).topk(k, dim=1)
    return idx.to(torch.int32).contiguous(), p.float().contiguous()


def _tensors(case, seed):
    """Everything that is drawn: made from the seed alone, in a fixed order."""
    g = _gen(seed)
    t = {}
    if case["kind"] == "step":
        L, d, E = case["L"], case["d"], case["E"]
        t["blobs"] = _blobs(case, g, L)
        t["gate_w"] = [_normal(case, g, (d, E), 0.02) for _ in range(L)]
        t["gate_b"] = [_zipf_bias(case, g) for _ in range(L)]
        t["x0"] = _normal(case, g, (case["T"], d), 1.0)
    elif case["kind"] == "ffn":
        t["blobs"] = _blobs(case, g, 1)
        idx, _ = _routing(case, g, case["rows"], 1)
        counts = torch.bincount(idx.view(-1), minlength=case["E"])
        t["offsets"] = torch.cat([counts.new_zeros(1), counts.cumsum(0)]).to(torch.int32)
        t["x"] = _normal(case, g, (case["rows"], case["d"]), 1.0)
    elif case["kind"] == "gate":
        t["w"] = _normal(case, g, (case["d"], case["E"]), 0.02)
        t["b"] = _zipf_bias(case, g)
        t["x"] = _normal(case, g, (case["T"], case["d"]), 1.0)
    else:
        T, k, d = case["T"], case["k"], case["d"]
        t["x"] = _normal(case, g, (T, d), 1.0)
        t["idx"], t["prob"] = _routing(case, g, T, k)
        t["y_perm"] = _normal(case, g, (T * k, d), 0.4)
    return t


def _context(case, max_tokens, k, L, f):
    flags = B.FLAG_FETCH_AUTO if case.get("store") == "host" else 0
    return B.Context(B.make_config(case["d"], f, case["E"], k, L, max_tokens, B.F32 if case["dtype"] == "f32" else B.BF16, flags=flags))


def prepare(case, seed):
    t = _tensors(case, seed)
    dt, dev = _dt(case), "cuda"
    i32 = dict(dtype=torch.int32, device=dev)
    s = {"case": case, "t": t, "stream": torch.cuda.Stream()}
    if case["kind"] == "step":
        T, d, k, E, L = case["T"], case["d"], case["k"], case["E"], case["L"]
        ctx = s["ctx"] = _context(case, T, k, L, case["f"])
        s["copy"] = torch.cuda.Stream()
        expert = t["blobs"][0, 0].numel() * t["blobs"].element_size()
        if case["store"] == "host":
            # two streams that share a hardware queue would serialise the migration: take another, as the repository's harness does
            for _ in range(8):
                if not ctx.check_streams(s["stream"], s["copy"]) & B.STREAMS_COMPUTE_COPY:
                    break
                s["copy"] = torch.cuda.Stream()
            s["store"] = torch.empty(t["blobs"].shape, dtype=dt, pin_memory=True)
            s["store"].copy_(t["blobs"])
            del t["blobs"]
            ctx.register_host_experts(s["store"], expert, expert * E)
        else:
            ctx.register_resident_experts(t["blobs"], expert, expert * E)
        s["x"] = torch.zeros((L + 1, T, d), dtype=dt, device=dev)
        s["x"][0] = t["x0"]
        s["y"] = torch.zeros((L, T, d), dtype=dt, device=dev)
        s["idx"] = torch.zeros((L, T, k), **i32)
        s["prob"] = torch.zeros((L, T, k), dtype=torch.float32, device=dev)
        s["bufs"] = ctx.make_step_buffers(t["gate_w"], t["gate_b"], s["x"], s["y"], s["idx"], s["prob"], torch.zeros((L, T * k), **i32),
                                          torch.zeros((L, E + 1), **i32), torch.zeros((T * k, d), dtype=dt, device=dev),
                                          torch.zeros((T * k, d), dtype=dt, device=dev),
                                          torch.zeros(ctx.workspace_bytes, dtype=torch.uint8, device=dev))
    elif case["kind"] == "ffn":
        ctx = s["ctx"] = _context(case, case["rows"], 1, 1, case["f"])
        expert = t["blobs"][0, 0].numel() * t["blobs"].element_size()
        ctx.register_resident_experts(t["blobs"], expert, expert * case["E"])
        s["y"] = torch.zeros((case["rows"], case["d"]), dtype=dt, device=dev)
        s["ws"] = torch.zeros(ctx.workspace_bytes, dtype=torch.uint8, device=dev)
    else:
        T, k = case["T"], case["k"]
        s["ctx"] = _context(case, T, k, 1, 64)
        if case["kind"] == "gate":
            s["idx"] = torch.zeros((T, k), **i32)
            s["prob"] = torch.zeros((T, k), dtype=torch.float32, device=dev)
            s["probs"] = torch.zeros((T, case["E"]), dtype=torch.float32, device=dev) if case["probs"] else None
        else:
            s["x_perm"] = torch.zeros((T * k, case["d"]), dtype=dt, device=dev)
            s["row_of"] = torch.zeros((T * k,), **i32)
            s["offsets"] = torch.zeros((case["E"] + 1,), **i32)
            s["y"] = torch.zeros((T, case["d"]), dtype=dt, device=dev)
            s["x_next"] = torch.zeros((T, case["d"]), dtype=dt, device=dev)
    torch.cuda.synchronize()
    return s


def run(s):
    case, t, ctx = s["case"], s["t"], s["ctx"]
    if case["kind"] == "step":
        ctx.stack_step(s["bufs"], case["T"], s["stream"], s["copy"])
        return {"x": [s["x"][i + 1] for i in range(case["L"])], "y": [s["y"][i] for i in range(case["L"])], "idx": s["idx"], "prob": s["prob"]}
    if case["kind"] == "ffn":
        ctx.expert_ffn(0, t["x"], t["offsets"], case["rows"], s["y"], s["ws"], s["stream"])
        return s["y"]
    if case["kind"] == "gate":
        ctx.pregate_topk(t["x"], t["w"], t["b"], case["T"], s["idx"], s["prob"], s["probs"], s["stream"])
        return {"idx": s["idx"], "prob": s["prob"], "probs": s["probs"]}
    ctx.permute(t["x"], t["idx"], case["T"], s["x_perm"], s["row_of"], s["offsets"], s["stream"])
    ctx.combine(t["y_perm"], s["row_of"], t["prob"], case["T"], s["y"], t["x"], s["x_next"], s["stream"])
    return {"x_perm": s["x_perm"], "row_of": s["row_of"], "offsets": s["offsets"], "y": s["y"], "x_next": s["x_next"]}


# ----------------------------------------------------------------------------- what a pass cannot do without
def _distinct(case, entries):
    """Expected number of distinct experts among `entries` selections."""
    E = case["E"]
    w = [(e + 1.0) ** -case["zipf"] for e in range(E)]
    total = sum(w)
    return sum(1.0 - (1.0 - v / total) ** entries for v in w)


def work(case):
    el = 4 if case["dtype"] == "f32" else 2
    d, E = case["d"], case["E"]
    if case["kind"] == "gate":
        T = case["T"]
        return {"bytes": el * (T * d + d * E) + 8 * T * case["k"] + (4 * T * E if case["probs"] else 0), "flops": 2 * T * d * E}
    if case["kind"] == "group":
        T, k = case["T"], case["k"]
        # x is read by both calls, y_perm by the second; x_perm, y and x_next are written
        return {"bytes": el * d * (2 * T + T * k + T * k + 2 * T) + 4 * T * k * 5, "flops": 2 * T * k * d}
    f = case["f"]
    expert = 2 * d * f * el
    if case["kind"] == "ffn":
        return {"bytes": _distinct(case, case["rows"]) * expert + 2 * el * case["rows"] * d, "flops": 4 * case["rows"] * d * f}
    T, k, L = case["T"], case["k"], case["L"]
    return {"bytes": L * (_distinct(case, T * k) * expert + el * (d * E + 3 * T * d) + 8 * T * k), "flops": L * (4 * T * k * d * f + 2 * T * d * E)}


def tolerance(case):
    """bf16 results carry one rounding of the hidden activation (averaged over d_ff products) and one of the result; float32 ones
    their sums' order.  Routing may differ where two logits are equal to the last bits, in a chain of several blocks also where
    a rounding of a hidden state tips them."""
    if case["kind"] == "group":
        return {"rel": 8e-3, "max": 2e-2} if case["dtype"] == "bf16" else {"rel": 1e-6, "max": 1e-5}
    if case["kind"] == "gate":
        return {"rel": 1e-5, "differ": 2e-3}
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "differ": 2e-3}
    if case["kind"] == "ffn":
        return {"rel": 1.2e-2}
    return {"rel": 1.2e-2, "differ": 2e-3 if case["L"] <= 2 else 5e-2}


# ----------------------------------------------------------------------------- the same in 64 bits
def _matrices(case, blob):
    """(W1 [d, f], W2 [f, d]) in 64 bits out of one packed expert."""
    d, f = case["d"], case["f"]
    a, b = blob[: d * f].double(), blob[d * f:].double()
    if case["dtype"] == "f32":
        return a.view(d, f), b.view(f, d)
    # tiles of 32 (k) x 16 (n): inside, [k group of 8][n][k within the group]; W1 n-tile major, W2 k-tile major
    w1 = a.view(f // 16, d // 32, 4, 16, 8).permute(1, 2, 4, 0, 3).reshape(d, f)
    w2 = b.view(f // 32, d // 16, 4, 16, 8).permute(0, 2, 4, 1, 3).reshape(f, d)
    return w1, w2


def _gate64(x, w, b, k):
    z = x.double() @ w.double()
    z = z if b is None else z + b.double()
    p = torch.softmax(z, dim=1)
    idx = z.topk(k, dim=1).indices
    return idx, p.gather(1, idx), p


def _block64(case, blobs, x, idx, prob):
    y = torch.zeros_like(x)
    for e in range(case["E"]):
        for j in range(case["k"]):
            rows = (idx[:, j] == e).nonzero().view(-1)
            if rows.numel():
                w1, w2 = _matrices(case, blobs[e])
                y[rows] += prob[rows, j: j + 1] * (torch.relu(x[rows] @ w1) @ w2)
    return y


def exact(case, seed):
    t = _tensors(case, seed)
    if case["kind"] == "gate":
        idx, p, probs = _gate64(t["x"], t["w"], t["b"], case["k"])
        return {"idx": idx.int(), "prob": p, "probs": probs if case["probs"] else None}
    if case["kind"] == "ffn":
        y = torch.zeros((case["rows"], case["d"]), dtype=torch.float64, device="cuda")
        offs = t["offsets"].tolist()
        for e in range(case["E"]):
            lo, hi = offs[e], offs[e + 1]
            if hi > lo:
                w1, w2 = _matrices(case, t["blobs"][0, e])
                y[lo:hi] = torch.relu(t["x"][lo:hi].double() @ w1) @ w2
        return y
    if case["kind"] == "group":
        T, k = case["T"], case["k"]
        e = t["idx"].view(-1).long()
        order = torch.sort(e, stable=True).indices
        row_of = torch.empty_like(order)
        row_of[order] = torch.arange(T * k, device="cuda")
        counts = torch.bincount(e, minlength=case["E"])
        x = t["x"].double()
        y = (t["prob"].double().unsqueeze(2) * t["y_perm"].double()[row_of].view(T, k, -1)).sum(1)
        return {"x_perm": x[order // k], "row_of": row_of.int(), "offsets": torch.cat([counts.new_zeros(1), counts.cumsum(0)]).int(),
                "y": y, "x_next": x + y}
    # Pre-gated stack: block 0 is routed by its own gate and block 1 by the pre-gate on the same input, so both routings and the two
    # blocks' outputs follow from the input.  Later blocks are routed from hidden states the library stores in 16 bits, where a
    # rounding may tip a choice between two experts: no such value.
    L = case["L"]
    known = min(L, 2)
    x = t["x0"].double()
    route = [_gate64(t["x0"], t["gate_w"][i], t["gate_b"][i], case["k"])[:2] for i in range(known)]
    xs, ys = [], []
    for i in range(known):
        y = _block64(case, t["blobs"][i], x, *route[i])
        x = x + y
        xs.append(x)
        ys.append(y)
    rest = [None] * (L - known)
    return {"x": xs + rest, "y": ys + rest, "idx": torch.stack([r[0] for r in route]).int() if known == L else None,
            "prob": torch.stack([r[1] for r in route]) if known == L else None}
