"""The work a decode program has this library do, as cases that can be timed.

A decode program loads its layers once (packs the signs of ``W_gate``,
transposes ``W_down``, quantizes for INT8) and then runs the MLP of every
layer once per token step: the fused call (predict and MLP in one), the
decoder-block call (RMSNorm and residual fused as well), or the MLP over rows
that it chose itself (a mask, or a predictor's list).  A step works on 1 to 8
tokens.

* ``form``   : ``fused``, ``block``, ``mask`` (``sparse_mlp`` over a caller's
  mask), ``list`` (``predict``, then ``sparse_mlp`` over its list) or ``load``
  (what is done once per layer at load).
* ``weights``: ``fp16`` or ``int8``; ``gated`` False is the MLP without W_up.
* ``d``, ``k``: model and hidden dimension; ``b`` tokens; ``s`` the share of
  rows that are inactive for one token; ``alpha`` the predictor's
  conservativeness.
* ``layers`` : layers of one pass.  Every layer has weights of its own, so that
  a pass meets its bytes in HBM and not in a cache, as in a model.
* ``graph``  : the pass is replayed from a HIP graph that holds one call per
  layer (what a decode loop does, as the calls take 10-60 us each); without
  it the calls are made from Python (prefill of a cache of graphs, loading,
  callers with other work between the calls).

Every tensor is drawn from the case's seed.  The gate rows are planted as in
ReLU-fied models: each row is active for a share ``1 - s`` of the tokens, and
its signs agree with a token's more often than not exactly where it is active
for it.
"""

import math

import torch

import paper_2411_12692_amd as si

DEV = "cuda"
EPS = 1e-5


def _case(name, form, d, k, b=1, s=0.9, alpha=1.0, weights="fp16", gated=True, layers=1, graph=False):
    return {"name": name, "form": form, "weights": weights, "gated": gated, "d": d, "k": k, "b": b, "s": s,
            "alpha": alpha, "layers": layers, "graph": graph}


def listed():
    return [
        # the smallest call: a single small layer called from Python, where the
        # call's own cost counts
        _case("small-1tok", "fused", 512, 1376),
        # decoding one sequence: the 7B- and 13B-shaped stacks
        _case("7b-1tok", "fused", 4096, 11008, layers=16, graph=True),
        _case("13b-1tok", "fused", 5120, 13824, s=0.88, alpha=1.02, layers=12, graph=True),
        # the same with INT8 weights
        _case("7b-int8-1tok", "fused", 4096, 11008, weights="int8", layers=16, graph=True),
        # the MLP half of the decoder layer in one call
        _case("7b-block-1tok", "block", 4096, 11008, alpha=1.01, layers=16, graph=True),
        # a few sequences at once, rows chosen by the caller
        _case("7b-mask-4tok", "mask", 4096, 11008, b=4, layers=8, graph=True),
        # the largest batch, fp16 and INT8
        _case("7b-8tok", "fused", 4096, 11008, b=8, layers=8, graph=True),
        _case("7b-int8-8tok", "fused", 4096, 11008, b=8, weights="int8", layers=8, graph=True),
        # a large non-gated layer
        _case("relu-large-6tok", "fused", 7168, 28672, b=6, gated=False, layers=2, graph=True),
        # the two-step form at a ragged size, called from Python
        _case("list-ragged-3tok", "list", 2944, 7777, b=3, s=0.85, alpha=1.03, layers=2),
        # loading one layer
        _case("load-7b", "load", 4096, 11008),
        _case("load-7b-int8", "load", 4096, 11008, weights="int8"),
    ]


def draw(rng):
    def log(lo, hi):
        return math.exp(rng.uniform(math.log(lo), math.log(hi)))

    form = rng.choices(["fused", "block", "mask", "list", "load"], [5, 2, 2, 2, 2])[0]
    weights = "fp16" if form in ("block", "list") else rng.choices(["fp16", "int8"], [2, 1])[0]
    d = 128 * max(4, min(56, round(log(512, 7168) / 128)))
    # a pass of the largest listed layer is the most a drawn one costs
    k = max(512, min(28672, round(log(1024, 28672))))
    if rng.random() < 0.5:
        k = max(512, k // 64 * 64)  # the usual hidden sizes are multiples of 64
    if form == "load":
        k = min(k, 11008 * 4096 // d)
        return {k_: v for k_, v in _case("", form, d, k, weights=weights, gated=rng.random() < 0.8).items()
                if k_ != "name"}
    c = _case("", form, d, k, b=rng.choice([1, 1, 1, 2, 3, 4, 5, 6, 7, 8]), s=round(rng.uniform(0.8, 0.97), 3),
              alpha=rng.choice([1.0, 1.0, 1.01, 1.02, 1.03]), weights=weights, gated=rng.random() < 0.8,
              graph=form != "list" and rng.random() < 0.75)
    most = 8 * 11008 * 4096  # weights' elements per matrix in one pass
    c["layers"] = rng.randint(1, max(1, min(12, most // (d * k)))) if c["graph"] else 1
    del c["name"]
    return c


# ---- inputs ---------------------------------------------------------------

def _generator(seed, layer):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1009 + layer) % (1 << 62))
    return g


def _normal(g, shape, std):
    return torch.randn(*shape, generator=g, device=DEV).mul_(std)


def _draw_layer(case, seed, layer):
    """What one layer is made of: tokens ``x`` ``[b][d]`` fp16 (decoder-block
    form: ``h`` and ``norm_w`` in float32, ``x`` having their signs), the
    fp16 weights and the rows active per token ``[b][k]``."""
    d, k, b = case["d"], case["k"], case["b"]
    g = _generator(seed, layer)
    x = _normal(g, (b, d), 1.0)
    n_act = max(1, k - int(math.floor(case["s"] * k + 0.5)))
    active = torch.zeros(b, k, dtype=torch.bool, device=DEV)
    for t in range(b):
        active[t, torch.randperm(k, generator=g, device=DEV)[:n_act]] = True
    # every element of a row follows one token of the batch: its sign
    # disagrees with that token's with probability 1/2 + e where the row is
    # inactive for it and 1/2 - e where it is active (0.6 / 0.4 per token up
    # to 4 tokens)
    e = 0.1 * min(b, 4)
    neg = x < 0
    if b == 1:
        p = torch.where(active[0], 0.5 - e, 0.5 + e)
        flip = torch.rand(k, d, generator=g, device=DEV) < p[:, None]
        sign_neg = neg ^ flip
    else:
        tok = torch.randint(0, b, (k, d), generator=g, device=DEV, dtype=torch.int32)
        coin = torch.rand(k, d, generator=g, device=DEV)
        sign_neg = torch.zeros(k, d, dtype=torch.bool, device=DEV)
        for t in range(b):
            p = torch.where(active[t], 0.5 - e, 0.5 + e)
            sign_neg |= (tok == t) & (neg[t][None, :] ^ (coin < p[:, None]))
        del tok, coin
    w = _normal(g, (k, d), 0.02).abs_()
    w_gate = torch.where(sign_neg, -w, w).to(torch.float16)
    del w, sign_neg
    w_up = _normal(g, (k, d), 0.02).to(torch.float16) if case["gated"] else None
    w_down = _normal(g, (d, k), 0.02).to(torch.float16)
    norm_w = 1.0 + _normal(g, (d,), 0.1)
    h = x * 2.0
    if case["form"] == "block":
        h = h * torch.where(norm_w < 0, -1.0, 1.0)
    return {"x": x.to(torch.float16), "h": h, "norm_w": norm_w, "w_gate": w_gate, "w_up": w_up, "w_down": w_down,
            "active": active}


def prepare(case, seed):
    state = {"case": case, "layers": [], "graph": None}
    if case["form"] == "load":
        lay = _draw_layer(case, seed, 0)
        state["layers"].append((lay["w_gate"], lay["w_up"], lay["w_down"]))
        return state
    b, d = case["b"], case["d"]
    for i in range(case["layers"]):
        lay = _draw_layer(case, seed, i)
        make = si.Int8MLPLayer if case["weights"] == "int8" else si.MLPLayer
        mlp = make(lay["w_gate"], lay["w_up"], lay["w_down"], max_batch=b)
        entry = {"mlp": mlp, "y": torch.empty(b, d, dtype=torch.float32, device=DEV)}
        if case["form"] == "block":
            entry.update(h=lay["h"], norm_w=lay["norm_w"])
        else:
            entry["x"] = lay["x"]
        if case["form"] == "mask":
            entry["mask"] = lay["active"].any(dim=0).to(torch.uint8)
        state["layers"].append(entry)
        del lay
    if case["graph"]:
        # the decode loop's graph: one call per layer, captured once
        stream = torch.cuda.Stream()
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            _calls(state)
        torch.cuda.current_stream().wait_stream(stream)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            state["out"] = _calls(state)
        state["graph"] = graph
    return state


# ---- one pass -------------------------------------------------------------

def _calls(state):
    case = state["case"]
    form, alpha = case["form"], case["alpha"]
    out = []
    for e in state["layers"]:
        mlp = e["mlp"]
        if form == "fused":
            out.append(mlp(e["x"], alpha, y=e["y"]))
        elif form == "block":
            out.append(mlp.block(e["h"], e["norm_w"], EPS, alpha, y=e["y"]))
        elif form == "mask":
            out.append(mlp.sparse_mlp(e["x"], mask=e["mask"]))
        else:
            mask, idx, n = mlp.predict(e["x"], alpha)
            out.append({"mask": mask, "n": n, "y": mlp.sparse_mlp(e["x"], active_idx=idx, n_active=n)})
    return out


def run(state):
    if state["graph"] is not None:
        state["graph"].replay()
        return state["out"]
    case = state["case"]
    if case["form"] != "load":
        return _calls(state)
    w_gate, w_up, w_down = state["layers"][0]
    if case["weights"] == "int8":
        mlp = si.Int8MLPLayer(w_gate, w_up, w_down)
        got = {"q_gate": mlp.q_gate, "s_gate": mlp.s_gate, "q_down_t": mlp.q_down_t, "s_down": mlp.s_down,
               "signs": mlp.signs}
        if w_up is not None:
            got.update(q_up=mlp.q_up, s_up=mlp.s_up)
        return got
    mlp = si.MLPLayer(w_gate, w_up, w_down)
    return {"signs": mlp.signs, "w_down_t": mlp.w_down_t}


# ---- what a pass cannot do without ----------------------------------------

def work(case):
    d, k, b = case["d"], case["k"], case["b"]
    signs = k * d / 8
    if case["form"] == "load":
        if case["weights"] == "int8":
            mats = 3 if case["gated"] else 2
            return {"bytes": mats * k * d * 3 + signs + 4 * (k * (mats - 1) + d), "flops": mats * k * d * 2}
        return {"bytes": 2 * k * d + signs + 4 * k * d, "flops": k * d}
    size = 1 if case["weights"] == "int8" else 2
    mats = 3 if case["gated"] else 2
    rows = k * (1.0 - case["s"] ** b)  # active for some token of the batch
    per = mats * rows * d * size + 4 * d * b + (8 * d if case["form"] == "block" and b == 1 else 0)
    per += (4 * d * b + 4 * d) if case["form"] == "block" else 2 * d * b
    if case["weights"] == "int8":
        per += 4 * (mats - 1) * rows + 4 * d
    if case["form"] == "mask":
        per += k
    else:
        per += signs
    if case["form"] == "list":
        per += k + 4 * rows
    return {"bytes": case["layers"] * per, "flops": case["layers"] * mats * rows * d * b * 2}


def tolerance(case):
    # loading moves and rounds single values: the same everywhere
    if case["form"] == "load":
        return "exact"
    # the decoder-block form rounds x to fp16 after an fp32 RMSNorm: another
    # order of its sum moves some elements by one fp16 unit (2^-11 of the
    # element, in a few of them; up to 1e-5 of y seen, where few rows are kept)
    if case["form"] == "block":
        return {"rel": 4e-5, "max": 4e-4}
    # exact products (fp16, or INT8 turned into fp16) summed in fp32: 2e-7 from
    # the 64-bit sums, and 1e-6 at most between two passes (the order of the
    # adds into y is not fixed)
    return {"rel": 1e-6, "max": 1e-5}


# ---- the same in 64 bits ---------------------------------------------------

def _quantize(w):
    w = w.float()
    scale = (w.abs().amax(dim=1).double() / 127.0).float()  # (a division by a number is a product with its inverse in fp32)
    safe = torch.where(scale > 0, scale, torch.ones_like(scale))
    q = torch.round(w / safe[:, None]).clamp_(-127, 127)
    return torch.where(scale[:, None] > 0, q, torch.zeros_like(q)), scale


def _kept(w_gate_negative, x, alpha):
    """Eq. (2): a row is kept if for some token not alpha * N_pos < N_neg."""
    d = x.shape[1]
    one = torch.ones((), device=DEV)
    sx = torch.where(x.view(torch.int16) < 0, -one, one)
    sw = torch.where(w_gate_negative, -one, one)
    n_neg = ((d - sw @ sx.t()) / 2).round().double()
    a = float(torch.tensor(alpha, dtype=torch.float32))
    return (~(a * (d - n_neg) < n_neg)).any(dim=1)


def exact(case, seed):
    if case["form"] == "load":
        if case["weights"] != "int8":
            return None
        lay = _draw_layer(case, seed, 0)
        got = {"q_gate": None, "q_down_t": None, "signs": None,
               "s_gate": lay["w_gate"].double().abs().amax(dim=1) / 127.0,
               "s_down": lay["w_down"].double().abs().amax(dim=1) / 127.0}
        if lay["w_up"] is not None:
            got.update(q_up=None, s_up=lay["w_up"].double().abs().amax(dim=1) / 127.0)
        return got
    out = []
    for i in range(case["layers"]):
        lay = _draw_layer(case, seed, i)
        x = lay["x"]
        if case["form"] == "block":
            h = lay["h"].double()
            x = (h / torch.sqrt(h.square().mean(dim=1, keepdim=True) + EPS) * lay["norm_w"].double()).to(torch.float16)
        if case["weights"] == "int8":
            mats = [None if m is None else _quantize(m) for m in (lay["w_gate"], lay["w_up"], lay["w_down"])]
            negative = mats[0][0] < 0
        else:
            mats = [None if m is None else (m, None) for m in (lay["w_gate"], lay["w_up"], lay["w_down"])]
            negative = mats[0][0].view(torch.int16) < 0
        if case["form"] == "mask":
            keep = lay["active"].any(dim=0)
        else:
            keep = _kept(negative, x, case["alpha"])
        rows = keep.nonzero().flatten()

        def some(m):  # the kept rows of W_gate or W_up in 64 bits
            v = m[0][rows].double()
            return v if m[1] is None else v * m[1][rows].double()[:, None]

        xt = x.double().t().contiguous()
        h3 = (some(mats[0]) @ xt).clamp_(min=0.0)
        if mats[1] is not None:
            h3 = h3 * (some(mats[1]) @ xt)
        down = mats[2][0][:, rows].double()
        if mats[2][1] is not None:
            down = down * mats[2][1].double()[:, None]
        y = (down @ h3).t().contiguous()
        if case["form"] == "block":
            y = y + lay["h"].double()
        if case["form"] == "list":
            out.append({"mask": None, "n": None, "y": y})
        else:
            out.append(y)
        del lay, mats, down, h3, negative
    return out
