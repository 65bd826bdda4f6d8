"""The performance cases of the library: what a serving program has it do, through its public entry points.

A case is a dict of plain values.  `kind` "verify" is one verification pass of one MoE layer (or of a stack
of `layers` layers replayed from one HIP graph): route the T draft tokens, then moe_verify_layer.  `kind`
"route" is the router from hidden states with the expert union, and `kind` "pack" the conversion of a
layer's weights to the streaming layout when a model is loaded.

Shapes are the benchmark's three layers (DeepSeek-V3.1, Qwen3-235B and GPT-OSS-120B shaped) and generic ones.
All inputs are seeded synthetic draws of the distributions the benchmark uses.
"""
import math
import zlib

import numpy as np
import torch

import paper_2607_12696_amd as moe

DEV = "cuda:0"

SHAPES = {
    "qwen": dict(d=4096, d_ff=1536, E=128, k=8, fmt=0, score=0, shared=False, oai=False),
    "ds": dict(d=7168, d_ff=2048, E=256, k=8, fmt=1, score=1, shared=True, oai=False),
    "gpt": dict(d=2880, d_ff=2880, E=128, k=4, fmt=2, score=0, shared=False, oai=True),
}


def _verify(shape, T, routing, U=0, router="logits", call="buffers", mx=False, layers=1, **more):
    return dict(SHAPES[shape], kind="verify", T=T, routing=routing, U=U, router=router, call=call, mx=mx, layers=layers,
                **more)


def listed():
    return [
        # Plain decoding of one token on a GPT-OSS layer (its biased, clamped experts): the smallest pass.
        dict(_verify("gpt", 1, "scattered", call="step"), name="gpt_t1"),
        # The paper's operating point of four verified tokens, as a serving loop runs it: the router and the
        # experts of a stack of layers captured once and replayed.
        dict(_verify("gpt", 4, "scattered", router="hidden", call="graph", layers=8), name="gpt_t4_stack8"),
        # A 64-token draft tree on a GPT-OSS layer.
        dict(_verify("gpt", 64, "tree"), name="gpt_t64_tree"),
        # A batch of drafts with the opt-in MX FP8 activations.
        dict(_verify("gpt", 300, "scattered", mx=True), name="gpt_t300_mx"),
        # Four verified tokens on a Qwen layer in bf16, through the one-call step.
        dict(_verify("qwen", 4, "tree", call="step"), name="qwen_t4_tree"),
        # A ragged draft tree on a Qwen layer.
        dict(_verify("qwen", 37, "tree"), name="qwen_t37_tree"),
        # Four verified tokens on a DeepSeek layer: the paper's 31 distinct experts.
        dict(_verify("ds", 4, "exact", U=31), name="ds_t4_u31"),
        # The 16 tokens that the selector keeps of a draft tree, through the one-call step.
        dict(_verify("ds", 16, "tree", call="step"), name="ds_t16_tree"),
        # The benchmark's headline: 64 draft tokens on exactly 32 distinct experts.
        dict(_verify("ds", 64, "exact", U=32), name="ds_t64_u32"),
        # A batch of drafts under DeepSeek's own group-limited routing: nearly every expert of the layer.
        dict(_verify("ds", 200, "scattered", router="grouped"), name="ds_t200_grouped"),
        # The router alone: logits, top-k and expert union of 64 hidden states.
        dict(SHAPES["ds"], kind="route", T=64, name="route_t64"),
        # Loading a quarter of a DeepSeek layer's experts (one GPU's share of four).
        dict(SHAPES["ds"], kind="pack", experts=64, name="pack_ds_e64"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def _any_shape(rng):
    """One of the benchmark's layers, or a generic one (odd widths, expert counts and top-k)."""
    name = rng.choice(["qwen", "ds", "gpt", "generic"])
    if name != "generic":
        return dict(SHAPES[name])
    fmt = rng.choice([0, 1, 2])
    unit = 128 if fmt == 1 else 32
    E = rng.randint(12, 200)
    return dict(d=unit * rng.randint(768 // unit, 6144 // unit), d_ff=unit * rng.randint(512 // unit, 3072 // unit), E=E,
                k=rng.randint(1, 8), fmt=fmt, score=rng.choice([0, 1]), shared=rng.random() < 0.3, oai=rng.random() < 0.3)


def draw(rng):
    c = _any_shape(rng)
    pick = rng.random()
    if pick < 0.12:
        return dict(c, kind="route", T=_log_int(rng, 1, 512))
    if pick < 0.24:
        return dict(c, kind="pack", experts=_log_int(rng, 1, min(c["E"], 64)))
    T = _log_int(rng, 1, 200 if c["fmt"] == 1 else 512)
    routing = rng.choice(["scattered", "tree", "exact"])
    most = min(c["E"], T * c["k"])
    U = rng.randint(c["k"], most) if routing == "exact" else 0
    router = "logits"
    if routing == "scattered":
        router = rng.choice(["logits", "hidden", "grouped"])
        if router == "grouped" and (c["E"] % 8 or c["k"] > c["E"] // 2):
            router = "hidden"
    call = rng.choice(["step", "buffers", "graph"]) if router == "logits" else rng.choice(["buffers", "graph"])
    return dict(c, kind="verify", T=T, routing=routing, U=U, router=router, call=call, mx=c["fmt"] == 2 and rng.random() < 0.4,
                layers=2 if call == "graph" and T <= 16 else 1)


# ----------------------------------------------------------------------------- inputs

def _gen(seed, tag):
    g = torch.Generator(device=DEV)
    g.manual_seed((seed << 32) | zlib.crc32(tag.encode()))
    return g


def _matrix(fmt, n, N, K, seed, tag):
    """Stacked weights [n, N, K] in the interchange layout and their scales."""
    g = _gen(seed, tag)
    if fmt == 0:
        return torch.empty(n, N, K, dtype=torch.bfloat16, device=DEV).normal_(0.0, 0.02, generator=g), None
    if fmt == 1:  # blocks of N(0, 0.02 * 2^u), codes up to about 448 in each block
        q = torch.empty(n, N, K, dtype=torch.uint8, device=DEV)
        for e in range(0, n, 8):
            part = q[e:e + 8]
            v = torch.empty(part.shape, dtype=torch.bfloat16, device=DEV).normal_(0.0, 112.0, generator=g)
            part.copy_(v.clamp_(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8))
        u = torch.randint(-2, 3, (n, N // 128, K // 128), generator=g, device=DEV).float()
        return q, 0.02 / 112.0 * torch.exp2(u)
    q = torch.randint(0, 256, (n, N, K // 2), generator=g, device=DEV, dtype=torch.uint8)
    return q, torch.randint(119, 122, (n, N, K // 32), generator=g, device=DEV, dtype=torch.uint8)


def _raw_layer(c, seed, layer, n):
    """A layer's weights in the interchange layout, the keys that pack_layer takes."""
    out = dict(fmt=c["fmt"], d=c["d"], d_ff=c["d_ff"], E=n)
    for pre, count in (("", n), ("sh_", 1)):
        if pre and not c["shared"]:
            continue
        for name, N, K in (("gate", c["d_ff"], c["d"]), ("up", c["d_ff"], c["d"]), ("down", c["d"], c["d_ff"])):
            w, s = _matrix(c["fmt"], count, N, K, seed, "%s%s/%d" % (pre, name, layer))
            out[pre + name] = w
            if s is not None:
                out[pre + "s_" + name] = s
    if c["oai"]:
        out.update(act=moe.MOE_ACT_SWIGLU_OAI, alpha=1.702, limit=7.0)
        for name, N in (("b_gate", c["d_ff"]), ("b_up", c["d_ff"]), ("b_down", c["d"])):
            out[name] = torch.randn(n, N, generator=_gen(seed, "%s/%d" % (name, layer)), device=DEV) * 0.5
    if c.get("mx"):
        out["act_fmt"] = moe.MOE_ACTQ_MXFP8
    return out


def _routes(c, seed, layer):
    """Expert lists [T, k] of a "tree" (children reuse their parent's experts) or an "exact" routing."""
    rng = np.random.default_rng([seed, layer, 7])
    T, E, k = c["T"], c["E"], c["k"]
    if c["routing"] == "exact":
        return rng.permutation(E)[:c["U"]][(np.arange(T)[:, None] * k + np.arange(k)) % c["U"]]
    out = np.zeros((T, k), np.int64)
    for t in range(T):
        order = rng.permutation(E)
        if t:
            keep = rng.permutation(out[(t - 1) // 2])[rng.random(k) < (0.7 if c["shared"] else 0.8)]
            order = np.concatenate([keep, order[~np.isin(order, keep)]])
        out[t] = rng.permutation(order[:k])
    return out


def _logits(c, seed, layer):
    """fp32 router logits [T, E]: N(0, 1), or such that each token's top-k is its list of _routes."""
    rng = np.random.default_rng([seed, layer, 8])
    lg = rng.standard_normal((c["T"], c["E"]))
    if c["routing"] != "scattered":
        r = _routes(c, seed, layer)
        lg = np.clip(lg, -4.0, 4.0)
        noise = np.clip(rng.standard_normal(r.shape) * 0.01, -0.05, 0.05)
        np.put_along_axis(lg, r, 9.0 - 0.25 * np.arange(c["k"]) + noise, axis=1)
    return torch.from_numpy(lg.astype(np.float32)).to(DEV)


def _inputs(c, seed, layer):
    """x and what the router reads: logits, or a router matrix, and the group-limited rule's bias."""
    x = torch.randn(c["T"], c["d"], generator=_gen(seed, "x/%d" % layer), device=DEV).to(torch.bfloat16)
    out = {"x": x}
    if c["kind"] == "route" or c["router"] == "hidden":
        w = torch.randn(c["E"], c["d"], generator=_gen(seed, "router/%d" % layer), device=DEV) * 0.02
        out["w_router"] = w.to(torch.bfloat16)
    else:
        out["logits"] = _logits(c, seed, layer)
        if c["router"] == "grouped":
            out["bias"] = (torch.rand(c["E"], generator=_gen(seed, "bias/%d" % layer), device=DEV) * 2 - 1) * 0.1
    return out


def _routing_buffers(c):
    T, k, E = c["T"], c["k"], c["E"]
    i32 = dict(dtype=torch.int32, device=DEV)
    return moe.Routing(T, k, E, torch.empty(T, k, **i32), torch.empty(T, k, dtype=torch.float32, device=DEV),
                       torch.empty(E, **i32), torch.empty(E, **i32), torch.empty(1, **i32), torch.empty(E + 1, **i32),
                       torch.empty(T * k, **i32))


def prepare(case, seed):
    c = case
    if c["kind"] == "pack":
        return {"case": c, "raw": _raw_layer(c, seed, 0, c["experts"])}
    if c["kind"] == "route":
        st = dict(_inputs(c, seed, 0), case=c, r=_routing_buffers(c))
        st["lg"] = torch.empty(c["T"], c["E"], dtype=torch.float32, device=DEV)
        st["ws"] = torch.empty(moe.moe_router_workspace_size(c["T"], c["d"], c["E"]), dtype=torch.uint8, device=DEV)
        return st
    layers = []
    for n in range(c["layers"]):
        la = dict(_inputs(c, seed, n), w=moe.pack_layer(_raw_layer(c, seed, n, c["E"])), r=_routing_buffers(c))
        la["y"] = torch.empty_like(la["x"])
        layers.append(la)
    st = {"case": c, "layers": layers}
    st["ws"] = torch.empty(moe.moe_verify_workspace_size(layers[0]["w"], c["T"], c["k"]), dtype=torch.uint8, device=DEV)
    if c["router"] == "hidden":
        st["rws"] = torch.empty(moe.moe_router_workspace_size(c["T"], c["d"], c["E"]), dtype=torch.uint8, device=DEV)
    if c["call"] == "graph":
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _pass(st)
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        st["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(st["graph"]):
            st["out"] = _pass(st)
    return st


def _outputs(y, r):
    return {"y": y, "idx": r.topk_idx, "w": r.topk_w, "counts": r.counts, "union": r.union_ids, "n": r.n_unique,
            "offsets": r.offsets, "perm": r.perm}


def _pass(st):
    c, out = st["case"], []
    for la in st["layers"]:
        r = la["r"]
        if c["call"] == "step":
            y, r = moe.moe_verify_step(la["x"], la["logits"], la["w"], c["k"], c["score"], workspace=st["ws"])
            out.append(_outputs(y, r))
            continue
        if c["router"] == "hidden":
            moe.moe_route_topk_hidden(la["x"], la["w_router"], c["k"], c["score"], workspace=st["rws"], topk_idx=r.topk_idx,
                                      topk_w=r.topk_w)
        elif c["router"] == "grouped":
            moe.moe_route_topk_grouped(la["logits"], la["bias"], c["k"], 8, 4, 2.5, topk_idx=r.topk_idx, topk_w=r.topk_w)
        else:
            moe.moe_route_topk(la["logits"], c["k"], c["score"], topk_idx=r.topk_idx, topk_w=r.topk_w)
        out.append(_outputs(moe.moe_verify_layer(la["x"], la["w"], r, y=la["y"], workspace=st["ws"]), r))
    return out


def run(state):
    c = state["case"]
    if c["kind"] == "pack":
        return {k: v for k, v in moe.pack_layer(state["raw"]).items() if isinstance(v, torch.Tensor)}
    if c["kind"] == "route":
        r = state["r"]
        moe.moe_route_topk_hidden(state["x"], state["w_router"], c["k"], c["score"], logits=state["lg"], workspace=state["ws"],
                                  topk_idx=r.topk_idx, topk_w=r.topk_w)
        moe.moe_expert_union(r.topk_idx, c["E"], out=r)
        return dict(_outputs(None, r), logits=state["lg"])
    if c["call"] == "graph":
        state["graph"].replay()
        return state["out"]
    return _pass(state)


# ----------------------------------------------------------------------------- work, tolerance, exact

def _expert_bytes(c):
    n = 3 * c["d"] * c["d_ff"]
    return 2 * n if c["fmt"] == 0 else n + 4 * (n // 16384) if c["fmt"] == 1 else n // 2 + n // 32


def work(case):
    c = case
    T = c.get("T", 0)
    if c["kind"] == "pack":
        return {"bytes": 2 * (c["experts"] + c["shared"]) * _expert_bytes(c), "flops": 0}
    router = 2 * (T + c["E"]) * c["d"]
    ints = 4 * (3 * T * c["k"] + 3 * c["E"] + 2)
    if c["kind"] == "route":
        return {"bytes": router + 4 * T * c["E"] + ints, "flops": 2 * T * c["E"] * c["d"]}
    if c["routing"] == "exact":
        U = c["U"]
    elif c["routing"] == "tree":
        U = len(np.unique(_routes(c, 1, 0)))
    elif c["router"] == "grouped":  # biased scores within the best half of the groups: counted on a draw
        rng = np.random.default_rng(1)
        s = 1 / (1 + np.exp(-rng.standard_normal((T, c["E"])))) + rng.uniform(-0.1, 0.1, c["E"])
        grp = np.sort(s.reshape(T, 8, -1), -1)[:, :, -2:].sum(-1)
        s[np.repeat(grp < np.sort(grp, -1)[:, 4:5], c["E"] // 8, 1)] = -1
        U = len(np.unique(np.argsort(-s, 1)[:, :c["k"]]))
    else:
        U = round(c["E"] * (1 - (1 - c["k"] / c["E"]) ** T))
    n_bias = U * (2 * c["d_ff"] + c["d"]) * 4 if c["oai"] else 0
    scores = router - 2 * T * c["d"] if c["router"] == "hidden" else 4 * T * c["E"]
    flops = 6 * T * (c["k"] + c["shared"]) * c["d"] * c["d_ff"] + (2 * T * c["E"] * c["d"] if c["router"] == "hidden" else 0)
    return {"bytes": c["layers"] * ((U + c["shared"]) * _expert_bytes(c) + n_bias + 4 * T * c["d"] + scores + ints),
            "flops": c["layers"] * flops}


def tolerance(case):
    # About four times the distance from exact(): 1.6e-7 (router logits and gates, fp32 sums), 2.4e-3 with at
    # most 1.0e-2 of a single value (bf16 intermediate and output), 1.7e-3 with 1.6e-2 (MX FP8 activations,
    # whose codes can flip at rounding boundaries).
    if case["kind"] == "pack":
        return "exact"
    if case["kind"] == "route":
        return {"rel": 1e-6, "max": 5e-6}
    return {"rel": 8e-3, "max": 0.065} if case["mx"] else {"rel": 1e-2, "max": 0.04}


_FP4 = [0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0, -0.0, -0.5, -1.0, -1.5, -2.0, -3.0, -4.0, -6.0]


def _decode(fmt, w, s, K):
    """One expert's matrix [N, K] in 64 bits."""
    if fmt == 0:
        return w.double()
    if fmt == 1:
        return w.view(torch.float8_e4m3fn).double() * s.double().repeat_interleave(128, 0).repeat_interleave(128, 1)
    codes = torch.stack([w & 15, w >> 4], -1).reshape(w.shape[0], K).long()
    v = torch.tensor(_FP4, dtype=torch.float64, device=DEV)[codes]
    return v * torch.exp2(s.double() - 127.0).repeat_interleave(32, 1)


def _mx_quant(v):
    """OCP MX FP8 of each 32-element block of the rows of v, in 64 bits."""
    b = v.reshape(v.shape[0], -1, 32)
    amax = b.abs().amax(-1, keepdim=True)
    e = torch.where(amax > 0, torch.floor(torch.log2(amax.clamp_min(1e-300))) - 8, torch.full_like(amax, -127.0)).clamp(-127, 127)
    u = b / torch.exp2(e)
    a = u.abs().clamp_max(448.0)
    step = torch.exp2(torch.floor(torch.log2(a.clamp_min(2.0 ** -6))) - 3)
    return (torch.copysign(torch.round(a / step) * step, u).clamp(-448, 448) * torch.exp2(e)).reshape(v.shape)


def _gates(score, l):
    g = torch.softmax(l, -1) if score == 0 else torch.sigmoid(l)
    return g / g.sum(-1, keepdim=True)


def _exact_route(c, st):
    """(logits, idx, w) in 64 bits."""
    if "w_router" in st:
        lg = st["x"].double() @ st["w_router"].double().t().contiguous()
    else:
        lg = st["logits"].double()
    if c.get("router") == "grouped":
        s = torch.sigmoid(lg)
        ch = s + st["bias"].double()
        grp = ch.reshape(c["T"], 8, -1).topk(2, -1).values.sum(-1)
        ok = torch.zeros_like(grp, dtype=torch.bool).scatter_(1, grp.topk(4, -1).indices, True)
        ch = ch.masked_fill(~ok.repeat_interleave(c["E"] // 8, 1), -math.inf)
        idx = ch.topk(c["k"], -1).indices
        g = s.gather(1, idx)
        return lg, idx, 2.5 * g / g.sum(-1, keepdim=True)
    l, idx = torch.sort(lg, dim=-1, descending=True, stable=True)
    return lg, idx[:, :c["k"]], _gates(c["score"], l[:, :c["k"]])


def _exact_layer(c, st, raw):
    _, idx, w = _exact_route(c, st)
    q = _mx_quant if c["mx"] else (lambda v: v)
    x = q(st["x"].double())
    y = torch.zeros(c["T"], c["d"], dtype=torch.float64, device=DEV)

    def ffn(pre, e, rows, bias):
        m = [_decode(c["fmt"], raw[pre + n][e], raw[pre + "s_" + n][e] if c["fmt"] else None, K)
             for n, K in (("gate", c["d"]), ("up", c["d"]), ("down", c["d_ff"]))]
        g, u = rows @ m[0].t().contiguous(), rows @ m[1].t().contiguous()
        if bias:
            g, u = g + raw["b_gate"][e].double(), u + raw["b_up"][e].double()
        if c["oai"]:
            g, u = g.clamp_max(7.0), u.clamp(-7.0, 7.0)
            h = g * torch.sigmoid(float(np.float32(1.702)) * g) * (u + 1)
        else:
            h = g * torch.sigmoid(g) * u
        o = q(h) @ m[2].t().contiguous()
        return o + raw["b_down"][e].double() if bias else o

    for e in torch.unique(idx).tolist():
        t, j = torch.nonzero(idx == e, as_tuple=True)
        y.index_add_(0, t, w[t, j][:, None] * ffn("", e, x[t], c["oai"]))
    if c["shared"]:
        y += ffn("sh_", 0, x, False)
    return y, w


def exact(case, seed):
    c = case
    none = {k: None for k in ("y", "idx", "w", "counts", "union", "n", "offsets", "perm")}
    if c["kind"] == "pack":
        return None
    if c["kind"] == "route":
        lg, _, w = _exact_route(c, _inputs(c, seed, 0))
        return dict(none, w=w, logits=lg)
    out = []
    for n in range(c["layers"]):
        y, w = _exact_layer(c, _inputs(c, seed, n), _raw_layer(c, seed, n, c["E"]))
        out.append(dict(none, y=y, w=w))
    return out
