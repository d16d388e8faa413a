"""Performance cases of the R-Sparse linear layer: what a decoder has this library do, through its public calls.

A case is one block (or a stack of blocks with weights of their own, so that weights come from HBM as they do in a
decoder that walks its layers) at one batch size.  Calls are issued as a decoder issues them: q/k/v grouped on their
shared input, then o; gate and up together, then down.  Weights, factors and tokens are synthetic: i.i.d. Gaussian
weights and factors with the entry scales of a power-law spectrum, heavy-tailed tokens with a few outlier channels,
silu(g) * u at the down projection.  Thresholds are calibrated for the case's channel sparsity on separate tokens.
"""
import math

import numpy as np
import torch

import paper_2504_19449_amd as rs

F16, BF16, F32 = rs.F16, rs.BF16, rs.F32
TORCH = {F16: torch.float16, BF16: torch.bfloat16, F32: torch.float32}
CODE = {"f16": F16, "bf16": BF16, "f32": F32}
CALIB_TOKENS = 16


# ---------------------------------------------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------------------------------------------
def _case(**kw):
    c = dict(part="attn", call="rsparse", d_model=4096, d_kv=4096, d_ff=11008, rank=256, rank_kv=256, dtype="bf16", out="same",
             batch=1, mask_mode=0, cmp_mode=0, sparsity=0.5, topk=False, bias=False, strip_cols=0, rowmajor=0, channel_major=0,
             q4_group=0, stack=1, graph=False)
    unknown = set(kw) - set(c) - {"name"}
    assert not unknown, unknown
    c.update(kw)
    return c


def listed():
    return [
        # one token, one 4096 x 4096 projection, one call: the smallest call of a decode step, all latency
        _case(name="o_4096_b1", part="o", dtype="f16", rank=256),
        # one token, the attention projections of 4096-wide layers packed in strips, replayed from a captured graph
        _case(name="attn_4096_strip_graph_b1", part="attn", dtype="f16", rank=256, strip_cols=128, stack=4, graph=True),
        # one token, the MLP of a 4096 / 11008 decoder layer
        _case(name="mlp_11008_b1", part="mlp", rank=512, channel_major=1, stack=4),
        # one token, all seven linears of an 8192 / 28672 decoder layer: the largest
        _case(name="block_28672_b1", part="block", d_model=8192, d_kv=1024, d_ff=28672, rank=1024, rank_kv=1024, channel_major=1),
        # one token, fixed-count activation with a static bias and fp32 outputs, sizes off every power of two
        _case(name="mlp_topk_bias_b1", part="mlp_gated", d_model=5128, d_ff=13832, rank=328, dtype="f16", out="f32", topk=True,
              bias=True, stack=2),
        # four tokens (small-batch decode or a few speculated tokens), library's choice of the mask
        _case(name="mlp_14336_b4", part="mlp", d_ff=14336, rank=256, batch=4, mask_mode=2, channel_major=1, stack=2),
        # eight tokens, grouped-query attention projections, row-major copy kept
        _case(name="attn_gqa_b8", part="attn", d_kv=1024, rank=256, rank_kv=128, batch=8, rowmajor=1, stack=4),
        # twelve tokens on layers that keep only the column-major weights
        _case(name="mlp_11008_colmajor_b12", part="mlp", dtype="f16", rank=512, batch=12, stack=1),
        # 32 tokens, the largest batch of one call (a short prefill, or many sequences), unrounded outputs
        _case(name="o_8192_b32", part="o", d_model=8192, rank=1024, batch=32, rowmajor=1, out="f32", stack=2),
        # the dense product that the per-layer plan falls back to at 16 tokens
        _case(name="mlp_14336_dense_b16", part="mlp_split", call="dense", d_ff=14336, rank=256, batch=16, rowmajor=1, stack=2),
        # 4-bit weights, one token
        _case(name="mlp_q4_b1", part="mlp_split", rank=512, q4_group=128, stack=2),
        # 4-bit weights, sixteen tokens
        _case(name="mlp_q4_b16", part="mlp_split", rank=512, q4_group=128, batch=16, stack=2),
    ]


def _size(rng, lo, hi):
    """A multiple of 8, spread over the logarithm of the range; one in three is a multiple of 256."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    step = 256 if rng.random() < 0.34 else 8
    return max(lo, v // step * step)


def draw(rng):
    kind = rng.choice(["b1", "b1", "strip", "block", "topk", "small", "rowmajor", "rowmajor", "colmajor", "dense", "q4", "q4"])
    # the weights of one linear: at most 2^27; 2^25 where a pass re-reads them or works on more than their bytes
    most = 1 << (25 if kind in ("colmajor", "q4") else 26 if kind in ("block", "dense", "rowmajor") else 27)
    d_model = _size(rng, 1024, 8192 if kind not in ("colmajor", "q4") else 4096)
    d_ff = _size(rng, d_model, max(d_model, min(28672, 7 * d_model // 2, most // d_model)))
    d_kv = _size(rng, 512, d_model)
    frac = rng.choice([1 / 32, 1 / 16, 1 / 8])
    rank = max(8, int(d_model * frac) // 8 * 8)
    kw = dict(d_model=d_model, d_ff=d_ff, d_kv=d_kv, rank=rank, rank_kv=min(rank, d_kv // 2 // 8 * 8), dtype=rng.choice(["f16", "bf16"]),
              out=rng.choice(["same", "same", "f32"]), sparsity=rng.choice([0.4, 0.5, 0.6, 0.7]))
    if kind == "b1":
        kw.update(part=rng.choice(["o", "attn", "mlp", "mlp_split"]), channel_major=rng.choice([0, 1]), cmp_mode=rng.choice([0, 0, 1]))
    elif kind == "strip":
        kw.update(part=rng.choice(["o", "attn"]), strip_cols=rng.choice([64, 128, 256]), graph=rng.random() < 0.5, stack=2)
    elif kind == "block":
        kw.update(part="block", channel_major=1, batch=rng.choice([1, 1, 2]))
    elif kind == "topk":
        kw.update(part=rng.choice(["mlp_split", "mlp_gated", "o"]), topk=True, bias=rng.random() < 0.5, batch=rng.choice([1, 1, 2, 4]))
    elif kind == "small":
        kw.update(part=rng.choice(["attn", "mlp", "mlp_split"]), batch=rng.randint(2, 4), mask_mode=rng.choice([0, 1, 2]),
                  channel_major=rng.choice([0, 1]))
    elif kind == "rowmajor":
        kw.update(part=rng.choice(["o", "attn", "mlp", "mlp_split"]), batch=rng.randint(5, 32), rowmajor=1,
                  mask_mode=rng.choice([0, 0, 1, 2]), bias=rng.random() < 0.2)
    elif kind == "colmajor":
        kw.update(part=rng.choice(["o", "attn", "mlp_split"]), batch=rng.randint(5, 32), mask_mode=rng.choice([0, 0, 2]))
    elif kind == "dense":
        kw.update(part=rng.choice(["o", "attn", "mlp_split"]), call="dense", batch=rng.choice([1, 2, 4, 8, 16, 32]), rowmajor=1)
    else:
        kw.update(part=rng.choice(["o", "mlp", "mlp_split"]), q4_group=rng.choice([64, 128]), batch=rng.choice([1, 1, 2, 4, 8, 16, 32]))
        kw["d_model"] = d_model // 256 * 256
        kw["d_ff"] = max(256, d_ff // 256 * 256)
        kw["rank"] = max(8, int(kw["d_model"] * frac) // 8 * 8)
    if kw["part"] == "mlp":
        kw["out"] = "same"        # the pair call stores round(silu(g) * u)
    return _case(**kw)


# ---------------------------------------------------------------------------------------------------------------
# what a case consists of: calls, each with its linears
# ---------------------------------------------------------------------------------------------------------------
def _calls(c):
    """[(kind, input kind, [(d_in, d_out, rank), ...])]: the calls of one block."""
    dm, kv, ff, r, rk = c["d_model"], c["d_kv"], c["d_ff"], c["rank"], c["rank_kv"]
    qkv = ("group", "dmodel", [(dm, dm, r), (dm, kv, rk), (dm, kv, rk)])
    o = ("linear", "dmodel", [(dm, dm, r)])
    up2 = [(dm, ff, r), (dm, ff, r)]
    down = ("linear", "down", [(ff, dm, r)])
    return {"o": [o],
            "attn": [qkv, o],
            "mlp": [("gate_up", "dmodel", up2), down],
            "mlp_split": [("group", "dmodel", up2), down],
            "mlp_gated": [("group", "dmodel", up2), ("gated", "pair", [(ff, dm, r)])],
            "block": [qkv, o, ("group", "dmodel", up2), down]}[c["part"]]


def _out_dtype(c):
    return CODE[c["dtype"]] if c["out"] == "same" else CODE[c["out"]]


def _gen(seed, *what):
    g = torch.Generator(device="cuda")
    h = int(seed) & 0xFFFFFFFF
    for v in what:
        h = (h * 1000003 + int(v) + 0x9E3779B9) & 0x7FFFFFFFFFFF
    g.manual_seed(h)
    return g


def _laplace(n, d, g):
    u = torch.rand((n, d), generator=g, device="cuda", dtype=torch.float64) - 0.5
    return -torch.sign(u) * torch.log1p(-2.0 * u.abs().clamp(max=0.5 - 1e-9))


def _tokens(kind, d, n, seed, block, ci, dt):
    """CALIB_TOKENS calibration tokens and n tokens of one call's input (and, for the gated call, the operands)."""
    total = CALIB_TOKENS + n
    g = _gen(seed, 1, block, ci)
    if kind == "dmodel":
        scale = torch.exp(0.5 * torch.randn(d, generator=g, device="cuda", dtype=torch.float64))
        scale[torch.randperm(d, generator=g, device="cuda")[:8]] *= 20.0
        x = (_laplace(total, d, g) * scale).to(dt)
        return x[:CALIB_TOKENS], x[CALIB_TOKENS:].contiguous(), None
    a = torch.randn((total, d), generator=g, device="cuda").to(dt)
    u = torch.randn((total, d), generator=g, device="cuda").to(dt)
    x = (a.double() / (1.0 + torch.exp(-a.double())) * u.double()).to(dt)
    pair = (a[CALIB_TOKENS:].contiguous(), u[CALIB_TOKENS:].contiguous()) if kind == "pair" else None
    return x[:CALIB_TOKENS], x[CALIB_TOKENS:].contiguous(), pair


def _tau(calib, s):
    """The calibrated threshold: the order statistic floor(s n) of the pooled magnitudes."""
    a = torch.sort(calib.abs().double().reshape(-1)).values
    return float(a[min(int(math.floor(s * a.numel())), a.numel() - 1)])


def _linear(c, d_in, d_out, r, seed, block, ci, li):
    """Weights and factors of one linear, on the GPU."""
    dt = TORCH[CODE[c["dtype"]]]
    g = _gen(seed, 2, block, ci, li)
    p = min(d_in, d_out)
    sig = 0.5 * torch.arange(1, p + 1, device="cuda", dtype=torch.float32) ** -0.6
    rms = float(torch.sqrt((sig.double() ** 2).sum() / (d_in * d_out)))
    w = {}
    if c["q4_group"]:
        G = d_in // c["q4_group"]
        w["Q"] = torch.randint(0, 16, (d_out, d_in), generator=g, device="cuda", dtype=torch.uint8)
        w["S"] = ((0.75 + 0.5 * torch.rand((d_out, G), generator=g, device="cuda")) * (rms / 4.6)).to(dt)
        w["Z"] = torch.randint(5, 11, (d_out, G), generator=g, device="cuda", dtype=torch.uint8)
    else:
        w["W"] = torch.empty((d_out, d_in), device="cuda", dtype=dt).normal_(0.0, rms, generator=g)
    w["U"] = torch.empty((d_out, r), device="cuda", dtype=dt).normal_(0.0, 1.0 / math.sqrt(d_out), generator=g)
    w["SV"] = (torch.randn((r, d_in), generator=g, device="cuda") * (sig[:r, None] / math.sqrt(d_in))).to(dt)
    w["bias"] = torch.randn(d_out, generator=g, device="cuda") * 0.1 if c["bias"] else None
    return w


def _bits(t):
    return t.view(torch.int16).cpu().numpy().view(np.uint16)


def _inputs(c, seed):
    """Per block and call: (kind, [linears' operands], tau, tokens, gate/up operands or None)."""
    dt = TORCH[CODE[c["dtype"]]]
    for block in range(c["stack"]):
        for ci, (kind, src, linears) in enumerate(_calls(c)):
            calib, x, pair = _tokens(src, linears[0][0], c["batch"], seed, block, ci, dt)
            ops = (_linear(c, d_in, d_out, r, seed, block, ci, li) for li, (d_in, d_out, r) in enumerate(linears))
            yield kind, linears, ops, _tau(calib, c["sparsity"]), x, pair


# ---------------------------------------------------------------------------------------------------------------
# what a program has in hand, and one pass
# ---------------------------------------------------------------------------------------------------------------
def _handle(c, d_in, d_out, r, tau, w):
    cfg = rs.make_config(d_in, d_out, r, tau, CODE[c["dtype"]], max_batch=c["batch"], out_dtype=_out_dtype(c), cmp_mode=c["cmp_mode"],
                         batch_mask_mode=c["mask_mode"], dense_rowmajor=c["rowmajor"], strip_cols=c["strip_cols"],
                         topk=int((1.0 - c["sparsity"]) * d_in) if c["topk"] else 0, lowrank_channel_major=c["channel_major"])
    U, SV = (_bits(w["U"]), _bits(w["SV"])) if r else (None, None)
    if c["q4_group"]:
        layer = rs.rsparse_prepare_q4(cfg, w["Q"].cpu().numpy(), _bits(w["S"]), w["Z"].cpu().numpy(), c["q4_group"], U, SV)
    else:
        layer = rs.rsparse_prepare_factors(cfg, _bits(w["W"]), U, SV)
    if w["bias"] is not None:
        rs.rsparse_set_bias(layer, w["bias"].cpu().numpy())
    return layer


def prepare(case, seed):
    c = case
    steps, outs = [], []
    odt = TORCH[_out_dtype(c)]
    for kind, linears, ops, tau, x, pair in _inputs(c, seed):
        layers = [_handle(c, *shape, tau, w) for shape, w in zip(linears, ops)]
        n_out = 1 if kind == "gate_up" else len(linears)
        ys = [torch.zeros((c["batch"], linears[i][1]), dtype=odt, device="cuda") for i in range(n_out)]
        steps.append((kind, layers, x, pair, ys))
        outs += ys
    state = {"case": c, "steps": steps, "outs": outs, "graph": None}
    if c["graph"]:
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            _issue(state)
        state["graph"] = graph
    return state


def _issue(state):
    c = state["case"]
    s = torch.cuda.current_stream().cuda_stream
    B = c["batch"]
    dense = c["call"] == "dense"
    for kind, layers, x, pair, ys in state["steps"]:
        if kind == "gate_up":
            rs.rsparse_mlp_gate_up(layers[0], layers[1], x.data_ptr(), B, ys[0].data_ptr(), s)
        elif kind == "gated":
            rs.rsparse_linear_gated(layers[0], pair[0].data_ptr(), pair[1].data_ptr(), B, ys[0].data_ptr(), s)
        elif len(layers) > 1:
            (rs.rsparse_dense_ref_group if dense else rs.rsparse_linear_group)(layers, x.data_ptr(), B, [y.data_ptr() for y in ys], s)
        else:
            (rs.rsparse_dense_ref if dense else rs.rsparse_linear)(layers[0], x.data_ptr(), B, ys[0].data_ptr(), s)


def run(state):
    if state["graph"] is not None:
        state["graph"].replay()
    else:
        _issue(state)
    return state["outs"]


# ---------------------------------------------------------------------------------------------------------------
# what a pass cannot do without, how close results have to be, and the results in 64 bits
# ---------------------------------------------------------------------------------------------------------------
def work(case):
    """Kept columns of W once (the union over the tokens; all of W where the call is dense), both factors (of S_r V_r^T
    the columns of channels that some token drops), tokens and outputs once."""
    c = case
    B, keep = c["batch"], 1.0 - c["sparsity"]
    union = c["mask_mode"] == 1 or (c["mask_mode"] == 2 and B >= 4)
    read = 1.0 - (1.0 - keep) ** B                       # channels that some token keeps
    drop = (1.0 - read) if union else 1.0 - keep ** B    # channels that some token drops
    eo = 4 if c["out"] == "f32" else 2
    nbytes = flops = 0.0
    for kind, _, linears in _calls(c):
        nbytes += 2.0 * B * linears[0][0] * (2 if kind == "gated" else 1)
        for i, (d_in, d_out, r) in enumerate(linears):
            share = 1.0 if c["call"] == "dense" else read
            if c["q4_group"]:
                nbytes += share * d_in * d_out / 2 + 2.5 * d_out * (d_in // c["q4_group"])
            else:
                nbytes += 2.0 * share * d_in * d_out
            own = 1.0 if c["call"] == "dense" else (read if union else keep)
            flops += 2.0 * B * own * d_in * d_out
            if c["call"] != "dense":
                nbytes += 2.0 * r * (d_out + drop * d_in)
                flops += 2.0 * B * r * (d_out + (1.0 - own) * d_in)
            if not (kind == "gate_up" and i > 0):
                nbytes += eo * B * d_out
    return {"bytes": c["stack"] * nbytes, "flops": c["stack"] * flops}


def tolerance(case):
    """16-bit outputs: one rounding of the result (2^-9 and 2^-12 relative at most, measured 1.7e-3 and 2.1e-4 from the
    64-bit result), times three to four; fp32 outputs: sums of up to 3e4 terms in 32 bits, and t in two 16-bit halves on
    the matrix cores."""
    if case["out"] == "f32":
        return {"rel": 1e-5}
    return {"rel": 8e-4 if case["dtype"] == "f16" else 6e-3}


def _masks(c, x, tau):
    """Kept channels per token, x [B, d] in 64 bits."""
    if c["topk"]:
        k = int((1.0 - c["sparsity"]) * x.shape[1])
        order = torch.sort(-x.abs(), dim=1, stable=True).indices[:, :k]
        m = torch.zeros_like(x, dtype=torch.bool).scatter_(1, order, True)
    else:
        t = float(np.float32(tau))
        m = x.abs() > t if c["cmp_mode"] == 1 else x.abs() >= t
    if c["mask_mode"] == 1 or (c["mask_mode"] == 2 and x.shape[0] >= 4):
        m = m.any(dim=0, keepdim=True).expand_as(m)
    return m


def exact(case, seed):
    c = case
    dt = TORCH[CODE[c["dtype"]]]
    outs = []
    for kind, linears, ops, tau, x16, _ in _inputs(c, seed):
        x = x16.double()
        m = _masks(c, x, tau)
        ys = []
        for w in ops:
            if c["q4_group"]:
                g = c["q4_group"]
                W = w["S"].double().repeat_interleave(g, 1) * (w["Q"].double() - w["Z"].double().repeat_interleave(g, 1))
            else:
                W = w["W"].double()
            if c["call"] == "dense":
                y = x @ W.T
            else:
                xs, xd = torch.where(m, x, 0.0), torch.where(m, 0.0, x)
                y = xs @ W.T
                if w["U"].shape[1]:
                    y = y + (xd @ w["SV"].double().T) @ w["U"].double().T
                if w["bias"] is not None:
                    y = y + w["bias"].double()
            del W
            ys.append(y)
        if kind == "gate_up":
            g, u = ys[0].to(dt).double(), ys[1].to(dt).double()
            ys = [g / (1.0 + torch.exp(-g)) * u]
        outs += ys
    return outs
