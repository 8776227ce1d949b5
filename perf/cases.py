"""The work a user of this framework has it do, as cases that can be timed and compared.

Almost everything a serving program asks for is one MoE layer forward (``MoELayer.forward``): block-routed, token-routed
or Alg. 1 with a Top-P coreset, over one small block (a decode step of one sequence) up to thousands of tokens (many
sequences, or a prompt), in bf16 or fp32.  Loading a model packs every layer's expert weights once (``pack_weights``).
``listed`` holds one case of each kind; ``draw`` gives more of the same ranges.  Sizes are those of the repository's
workload presets (dmoe_synth) or generic.

A forward case:
  layers  consecutive layers of one pass, each with its own weights and hidden states (a decode step runs through many
          layers, so one layer's experts never wait in the last-level cache for the next pass)
  graph   the pass is captured once in a HIP graph and replayed, as a decode loop does; without it the pass is called
  dtype, H, E, I, I_s, k, nb, bs, routing, p: the layer (nb blocks of bs tokens, top-k of E experts, I_s: shared expert)
  bias    "zipf": router bias -1.1 ln(rank), skewed expert popularity
  x       "corr": tokens of one block share a direction; else independent N(0, 1)
  resid   each layer's call also writes the next layer's input, residual + output
"""
import math

import torch

from paper_2605_30876_amd.layer import MoELayer, pack_weights

DEV = "cuda"


def _fwd(name, dtype, H, E, I, I_s, k, nb, bs, routing, *, layers=1, graph=False, p=0.6, bias="none", x="iid", resid=False):
    return {"name": name, "kind": "forward", "dtype": dtype, "H": H, "E": E, "I": I, "I_s": I_s, "k": k, "nb": nb,
            "bs": bs, "routing": routing, "p": p, "bias": bias, "x": x, "layers": layers, "graph": graph, "resid": resid}


def listed():
    return [
        # the smallest call: a tiny fp32 layer, one block of 8 tokens (launches and latency only)
        _fwd("tiny_f32_block", "f32", 256, 16, 128, 0, 2, 1, 8, "block", graph=True),
        # fp32 in earnest: a mid-sized layer checked or served at full precision, two blocks, each token its own experts
        _fwd("mid_f32_token", "f32", 1024, 32, 512, 512, 4, 2, 32, "token"),
        # a ragged small bf16 layer: blocks of 24, top-6 of 48 experts
        _fwd("ragged_b5x24_block", "bf16", 768, 48, 384, 256, 6, 5, 24, "block", graph=True),
        # a decode step of one sequence through eight block-routed layers, with the residual stream
        _fwd("decode_b1_block_x8", "bf16", 2048, 256, 512, 512, 8, 1, 32, "block", layers=8, graph=True, resid=True),
        # one decode layer of one sequence with the two other routings
        _fwd("decode_b1_topp", "bf16", 2048, 256, 512, 512, 8, 1, 32, "topp", graph=True),
        _fwd("decode_b1_token", "bf16", 2048, 256, 512, 512, 8, 1, 32, "token", graph=True),
        # sixteen sequences decoded together
        _fwd("decode_b16_block", "bf16", 2048, 256, 512, 512, 8, 16, 32, "block"),
        _fwd("decode_b16_topp", "bf16", 2048, 256, 512, 512, 8, 16, 32, "topp"),
        # a wide layer with popular experts, eight sequences: few experts with many rows, and many experts
        _fwd("large_zipf_b8_block", "bf16", 4096, 256, 1536, 1536, 8, 8, 32, "block", bias="zipf"),
        _fwd("large_zipf_b8_token", "bf16", 4096, 256, 1536, 1536, 8, 8, 32, "token", bias="zipf"),
        # 64 sequences of 64 correlated tokens: the compute-heavy end (prompts, large batches)
        _fwd("corr_b64x64_block", "bf16", 2048, 256, 512, 512, 8, 64, 64, "block", x="corr"),
        # loading a model: one layer's expert weights into the packed layout
        {"name": "pack_decode_layer", "kind": "pack", "dtype": "bf16", "H": 2048, "E": 256, "I": 512, "I_s": 512},
    ]


# ---- draws ------------------------------------------------------------------

_MAX_WEIGHT_BYTES = 3 * 257 * 4096 * 1536 * 2       # the largest listed layer's experts
_MAX_FLOPS = 4096 * 6.0 * 2048 * 512 * 9            # the largest listed forward's
_MAX_F32_FLOPS = 64 * 6.0 * 1024 * 512 * 5 * 2      # fp32 draws stay near the listed fp32 layer


def _log_int(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def _weight_bytes(c):
    return 3 * c["H"] * (c["E"] * c["I"] + c["I_s"]) * (4 if c["dtype"] == "f32" else 2)


def _flops(c):
    T = c["nb"] * c["bs"]
    return c["layers"] * T * (6.0 * c["H"] * (c["k"] * c["I"] + c["I_s"]) + 2.0 * c["H"] * c["E"])


def draw(rng):
    if rng.random() < 0.08:
        while True:
            f32 = rng.random() < 0.3
            step = 4 if f32 else 128
            c = {"kind": "pack", "dtype": "f32" if f32 else "bf16", "H": _log_int(rng, 256, 4096, step),
                 "E": _log_int(rng, 8, 256), "I": _log_int(rng, 128, 1536, step), "I_s": 0}
            c["I_s"] = c["I"] if rng.random() < 0.5 else 0
            if _weight_bytes(c) <= 3 * 257 * 2048 * 512 * 2:
                return c
    while True:
        f32 = rng.random() < 0.2
        routing = rng.choice(["block", "block", "token", "topp"])
        E = _log_int(rng, 16, 256, rng.choice([1, 4, 16]))
        k = min(rng.choice([2, 4, 6, 8, 8, 8]), E)
        bs = rng.choice([32, 32, 8, 16, 24, 64, _log_int(rng, 4, 64)])
        nb = 1 if rng.random() < 0.35 else _log_int(rng, 2, 64)
        if f32:
            H, I = _log_int(rng, 96, 1024, 4), _log_int(rng, 40, 512, 8)
        else:
            H, I = _log_int(rng, 256, 4096, 128), _log_int(rng, 128, 1536, 128)
        c = _fwd("", "f32" if f32 else "bf16", H, E, I, rng.choice([0, I, I]), k, nb, bs, routing,
                 p=rng.choice([0.4, 0.6, 0.6, 0.8]), bias=rng.choice(["none", "none", "zipf"]),
                 x=rng.choice(["iid", "iid", "corr"]), graph=nb * bs <= 256)
        del c["name"]
        small = _weight_bytes(c) * 4 < 2 * _MAX_WEIGHT_BYTES and nb == 1
        if small and rng.random() < 0.5:
            c["layers"] = 4
        c["resid"] = rng.random() < 0.3
        if c["layers"] * _weight_bytes(c) <= _MAX_WEIGHT_BYTES and _flops(c) <= (_MAX_F32_FLOPS if f32 else _MAX_FLOPS):
            return c


# ---- inputs -----------------------------------------------------------------

def _gen(seed, *key):
    g = torch.Generator(device=DEV)
    v = seed
    for x in key:
        v = (v * 1000003 + x + 12345) & 0x7FFFFFFFFFFF
    g.manual_seed(v)
    return g


def _dtype(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


def _normal(shape, std, c, g):
    return torch.empty(shape, dtype=_dtype(c), device=DEV).normal_(0.0, std, generator=g)


def _experts(c, seed, layer):
    """Unpacked expert weights of one layer, N(0, 0.02^2)."""
    H, E, I, I_s = c["H"], c["E"], c["I"], c["I_s"]
    g = _gen(seed, layer, 1)
    w = {"w_gate": _normal((E, I, H), 0.02, c, g), "w_up": _normal((E, I, H), 0.02, c, g),
         "w_down": _normal((E, H, I), 0.02, c, g)}
    if I_s:
        w.update(ws_gate=_normal((I_s, H), 0.02, c, g), ws_up=_normal((I_s, H), 0.02, c, g),
                 ws_down=_normal((H, I_s), 0.02, c, g))
    return w


def _router(c, seed, layer):
    """Router weights, bias, hidden states and the residual of one layer."""
    g = _gen(seed, layer, 2)
    T = c["nb"] * c["bs"]
    wr = _normal((c["E"], c["H"]), 0.02, c, g)
    bias = None
    if c["bias"] == "zipf":
        ranks = torch.randperm(c["E"], generator=g, device=DEV).double() + 1.0
        bias = (-1.1 * torch.log(ranks)).float()
    if c["x"] == "corr":
        u = torch.randn((c["nb"], 1, c["H"]), generator=g, device=DEV)
        x = (u + 0.5 * torch.randn((c["nb"], c["bs"], c["H"]), generator=g, device=DEV)).reshape(T, c["H"]).to(_dtype(c))
    else:
        x = _normal((T, c["H"]), 1.0, c, g)
    return wr, bias, x


def prepare(case, seed):
    c = case
    if c["kind"] == "pack":
        w = _experts(c, seed, 0)
        w["w_router"] = _normal((c["E"], c["H"]), 0.02, c, _gen(seed, 0, 2))
        return {"case": c, "w": w}
    ws, ms, xs, outs = [], [], [], []
    for l in range(c["layers"]):
        w = _experts(c, seed, l)
        wr, bias, x = _router(c, seed, l)
        w.update(w_router=wr, bias=bias)
        ws.append(pack_weights(w))
        xs.append(x)
        outs.append(torch.empty_like(x) if c["resid"] else None)
        ms.append(MoELayer(c["H"], c["E"], c["I"], c["I_s"], c["k"], c["nb"], c["bs"], dtype=_dtype(c), device=DEV,
                           top_p=c["p"]))
        del w
    s = {"case": c, "w": ws, "m": ms, "x": xs, "out": outs, "graph": None}
    if c["graph"]:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _forward(s)
        torch.cuda.current_stream().wait_stream(side)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            s["result"] = _forward(s)
        s["graph"] = g
    return s


def _forward(s):
    c = s["case"]
    got = []
    for m, w, x, out in zip(s["m"], s["w"], s["x"], s["out"]):
        y = m.forward(x, w, c["routing"], residual=(x, out) if out is not None else None)
        got.append({"y": y, "weights": m.combine_w, "experts": m.experts(c["routing"])})
        if out is not None:
            got[-1]["next"] = out
    return got


def run(state):
    if state["case"]["kind"] == "pack":
        p = pack_weights(state["w"])
        return {n: p[n] for n in ("w13", "w2", "ws13", "ws2") if n in p}
    if state["graph"] is not None:
        state["graph"].replay()
        return state["result"]
    return _forward(state)


# ---- the definition in plain torch ------------------------------------------

def _topk(p, k):
    """Indices of the k largest, the lower index first among equals."""
    return torch.sort(p, dim=-1, descending=True, stable=True).indices[..., :k]


def _route(c, wr, bias, x, dtype):
    """Each token's experts [T, k] and weights [T, k]."""
    T, E, k, nb, bs = c["nb"] * c["bs"], c["E"], c["k"], c["nb"], c["bs"]
    z = x.to(dtype) @ wr.to(dtype).t()
    if bias is not None:
        z = z + bias.to(dtype)
    prob = torch.softmax(z, dim=-1)
    if c["routing"] == "block":
        sel = _topk(prob.view(nb, bs, E).mean(1), k)[:, None, :].expand(nb, bs, k).reshape(T, k)
    else:
        sel = _topk(prob, k)
        if c["routing"] == "topp":
            own = torch.zeros_like(prob).scatter_(1, sel, prob.gather(1, sel))
            score = own.view(nb, bs, E).sum(1)
            score = score / score.sum(-1, keepdim=True)
            order = _topk(score, E)
            mass = score.gather(1, order).cumsum(-1)
            n = ((mass < c["p"]).sum(-1) + 1).clamp(min=k, max=E)
            rank = torch.empty_like(order).scatter_(1, order, torch.arange(E, device=x.device).expand(nb, E).contiguous())
            inside = (rank < n[:, None])[:, None, :].expand(nb, bs, E).reshape(T, E)
            sel = _topk(prob.masked_fill(~inside, -1.0), k)
    w = prob.gather(1, sel)
    return sel, w / w.sum(-1, keepdim=True)


def _swiglu(x, g, u, d):
    a = x @ g.double().t()
    return (a / (1.0 + torch.exp(-a)) * (x @ u.double().t())) @ d.double().t()


def exact(case, seed):
    c = case
    if c["kind"] == "pack":
        return None  # a permutation of whole values
    got = []
    for l in range(c["layers"]):
        w = _experts(c, seed, l)
        wr, bias, x = _router(c, seed, l)
        sel, cw = _route(c, wr, bias, x, torch.float64)
        xd = x.double()
        y = _swiglu(xd, w["ws_gate"], w["ws_up"], w["ws_down"]) if c["I_s"] else torch.zeros_like(xd)
        for e in torch.unique(sel).tolist():
            t, j = torch.nonzero(sel == e, as_tuple=True)
            y.index_add_(0, t, cw[t, j, None] * _swiglu(xd[t], w["w_gate"][e], w["w_up"][e], w["w_down"][e]))
        got.append({"y": y, "weights": cw, "experts": None})
        if c["resid"]:
            got[-1]["next"] = xd + y
        del w
    return got


_UNIQUE = {}


def work(case):
    c = case
    eb = 4 if c["dtype"] == "f32" else 2
    if c["kind"] == "pack":
        return {"bytes": 2.0 * _weight_bytes(c), "flops": 0.0}
    key = str(sorted((k, v) for k, v in c.items() if k != "name"))
    if key not in _UNIQUE:  # distinct experts of a forward, from one draw of its inputs
        wr, bias, x = _router(c, 1, 0)
        _UNIQUE[key] = int(torch.unique(_route(c, wr, bias, x, torch.float32)[0]).numel())
    T = c["nb"] * c["bs"]
    per = 3 * c["H"] * (_UNIQUE[key] * c["I"] + c["I_s"]) * eb + c["E"] * c["H"] * eb
    per += T * c["H"] * (eb + 4) + T * c["k"] * 8                       # x in, y (fp32) out, weights and experts out
    if c["resid"]:
        per += T * c["H"] * eb                                          # the next input (the residual is x itself)
    return {"bytes": float(c["layers"] * per), "flops": _flops(c)}


def tolerance(case):
    if case["kind"] == "pack":
        return "exact"
    # differ: exact near-ties in a top-k (scores equal to 7 digits) may fall either way
    # rel: four times the present path's distance from exact() (fp32: up to 8e-7; bf16 layers, whose SwiGLU activations
    # are rounded to bf16 between the two products: 1.6e-3 to 1.8e-3)
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 1e-3, "differ": 1e-3}
    return {"rel": 7e-3, "max": 0.5, "differ": 1e-3}
