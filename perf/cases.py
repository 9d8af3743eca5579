"""The work the library's speed is measured on.

Each case is one pass of a user's program through the public entry points:
a training step (forward, back-propagation through time and every gradient)
of one layer (`Layer`) or of a stack (`Stack`), or a forward call of a
serving loop (`lstm_forward_noalloc`).  The sizes are those of the networks
the library is built for (GNMT's 1024-wide stacks, BigLSTM's 8192 cells with
a 1024-wide projection, the tiny fp32 layer) and generic ones between them:
other widths, ragged batches, fp32 storage, narrower projections.

A case is a dict of
  kind     "layer", "stack" or "serve"
  T, B     time steps, batch rows
  I, H, Hp input width, cells, projection width (0: none) of the layer; a
           stack's first layer (its other layers take the layer below)
  dtype    "bf16" or "f32"
  states   layer: initial states given, and gradients for the final ones
  reverse  layer: the sequence visited from the end (a bidirectional layer's
           second direction, whose rows interleave with the first one's:
           y has twice the row stride)
  micro    layer: mini-batches of one step, accumulated into one gradient
  layers   stack: its depth
  bi       stack: a bidirectional first layer, residual sums from the third
           layer on (GNMT's encoder)
  scale    weights and biases are U(-scale, scale)
"""
import math

import torch

from paper_1907_13257_amd import Layer, Stack, StackLayer, lstm355


def _case(name=None, kind="layer", T=1, B=1, I=8, H=8, Hp=0, dtype="bf16", states=False, reverse=False, micro=1,
          layers=1, bi=False, scale=0.1):
    c = dict(kind=kind, T=T, B=B, I=I, H=H, Hp=Hp, dtype=dtype, states=states, reverse=reverse, micro=micro,
             layers=layers, bi=bi, scale=scale)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest training step: a unit-test sized fp32 layer with its states carried
        _case("tiny_f32", T=8, B=4, I=32, H=64, dtype="f32", states=True, scale=0.125),
        # one decoder step of a served 1024-wide layer, states in and out
        _case("decode_t1", kind="serve", T=1, B=16, I=1024, H=1024, states=True),
        # a served half-width encoder layer over a sentence, a few sentences at a time
        _case("encode_h512", kind="serve", T=30, B=4, I=512, H=512),
        # the GNMT stack at the smallest per-worker batch of the batch sweep
        _case("gnmt4_b16", kind="stack", T=50, B=16, I=1024, H=1024, layers=4),
        # the GNMT stack at the per-worker batch of the headline benchmark
        _case("gnmt4_b128", kind="stack", T=50, B=128, I=1024, H=1024, layers=4),
        # GNMT's eight-layer encoder: bidirectional first layer, residual sums
        _case("gnmt8_b256", kind="stack", T=50, B=256, I=1024, H=1024, layers=8, bi=True),
        # one GNMT layer at the largest batch of the sweep
        _case("layer_b512", T=50, B=512, I=1024, H=1024),
        # the reverse direction of a bidirectional layer on a 2048-wide input, a ragged batch, states carried
        _case("layer_reverse_b250", T=50, B=250, I=2048, H=1024, states=True, reverse=True),
        # one BigLSTM layer
        _case("biglstm_layer", T=20, B=128, I=1024, H=8192, Hp=1024, scale=0.05),
        # fp32 storage at GNMT's width
        _case("f32_wide", T=50, B=32, I=1024, H=1024, dtype="f32", scale=0.1),
        # a layer of neither network: odd widths and batch, two mini-batches accumulated
        _case("ragged_bf16", T=35, B=50, I=304, H=648, states=True, micro=2, scale=0.04),
        # a projected layer of ordinary width
        _case("lstmp_mid", T=20, B=64, I=512, H=1024, Hp=512, scale=0.05),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mult8(v):
    return max(8, (v + 4) // 8 * 8)


def draw(rng):
    kind = rng.choice(["stack", "wide", "wide", "any", "any", "f32", "lstmp", "big", "serve"])
    T = rng.randint(8, 50)
    if kind == "stack":
        return _case(kind="stack", T=T, B=_log(rng, 8, 256), I=1024, H=1024, layers=rng.randint(2, 4))
    if kind == "wide":
        H = rng.choice([256, 512, 1024, 1024])
        return _case(T=T, B=_log(rng, 1, 512), I=_mult8(_log(rng, 64, 2048)), H=H, states=rng.random() < 0.5,
                     reverse=rng.random() < 0.5, scale=0.1 * math.sqrt(1024 / H) / 2)
    if kind == "any":
        H = _mult8(_log(rng, 64, 1536))
        return _case(T=T, B=_log(rng, 1, 128), I=_mult8(_log(rng, 32, 1536)), H=H, states=rng.random() < 0.5,
                     reverse=rng.random() < 0.5, micro=rng.randint(1, 2) if H < 700 else 1, scale=1.0 / math.sqrt(H))
    if kind == "f32":
        H = _mult8(_log(rng, 32, 1024))
        return _case(T=rng.randint(5, 30), B=_log(rng, 1, 96), I=_mult8(_log(rng, 32, 1024)), H=H, dtype="f32",
                     states=rng.random() < 0.5, reverse=rng.random() < 0.5, scale=1.0 / math.sqrt(H))
    if kind == "lstmp":
        H = _mult8(_log(rng, 128, 1800))
        return _case(T=rng.randint(5, 30), B=_log(rng, 4, 128), I=_mult8(_log(rng, 64, 1024)), H=H,
                     Hp=_mult8(_log(rng, 64, min(H, 768))), dtype=rng.choice(["bf16", "bf16", "f32"]),
                     states=rng.random() < 0.5, scale=1.0 / math.sqrt(H))
    if kind == "big":
        H = _mult8(_log(rng, 2048, 8192))
        return _case(T=rng.randint(5, 20), B=_log(rng, 16, 128), I=1024, H=H, Hp=_mult8(_log(rng, 256, 1024)),
                     states=rng.random() < 0.5, scale=0.05)
    H = rng.choice([256, 512, 1024, _mult8(_log(rng, 64, 1024))])
    return _case(kind="serve", T=rng.choice([1, 1, _log(rng, 2, 50)]), B=_log(rng, 1, 32),
                 I=_mult8(_log(rng, 64, 1024)), H=H, states=rng.random() < 0.7, scale=1.0 / math.sqrt(H))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _layer_list(case):
    """(I, H, Hp, bidirectional, residual) of each layer."""
    H, Hp = case["H"], case["Hp"]
    Hr = Hp or H
    if case["kind"] != "stack":
        return [(case["I"], H, Hp, False, False)]
    out, width = [], case["I"]
    for l in range(case["layers"]):
        bi = case["bi"] and l == 0
        out.append((width, H, Hp, bi, case["bi"] and l >= 2))
        width = Hr * (2 if bi else 1)
    return out


def _inputs(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    td = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    T, B, a = case["T"], case["B"], case["scale"]

    def uniform(*shape, dtype=td, a=a):
        return ((torch.rand(shape, generator=g, device="cuda") * 2 - 1) * a).to(dtype)

    def normal(*shape, dtype=td):
        return torch.randn(shape, generator=g, device="cuda").to(dtype)

    params = []
    for I, H, Hp, bi, _ in _layer_list(case):
        Hr = Hp or H
        dirs = []
        for _ in range(2 if bi else 1):
            p = dict(W=uniform(4 * H, I), R=uniform(4 * H, Hr), b=uniform(4 * H, dtype=torch.float32))
            if Hp:
                p["P"] = uniform(Hp, H)
            dirs.append(p)
        params.append(dirs)
    H, Hr = case["H"], case["Hp"] or case["H"]
    d = dict(params=params, x=[normal(T, B, case["I"]) for _ in range(case["micro"])],
             h0=None, c0=None, dhT=None, dcT=None)
    if case["states"]:
        d["h0"], d["c0"] = uniform(B, Hr, a=1.0), uniform(B, H, a=1.0, dtype=torch.float32)
    if case["kind"] != "serve":
        # a reverse direction's rows lie in the second half of the bidirectional layer's
        ld = 2 * Hr if case["reverse"] else Hr
        d["dy"] = [normal(T, B, ld)[:, :, ld - Hr:] for _ in range(case["micro"])]
        if case["states"]:
            d["dhT"], d["dcT"] = normal(B, Hr), normal(B, H, dtype=torch.float32)
    return d


def prepare(case, seed):
    d = _inputs(case, seed)
    T, B, I, H, Hp = case["T"], case["B"], case["I"], case["H"], case["Hp"]
    Hr = Hp or H
    td = d["x"][0].dtype
    st = dict(d, kind=case["kind"])
    if case["kind"] == "stack":
        st["stack"] = Stack(T, B, [StackLayer(i, h, hp, bi, res) for i, h, hp, bi, res in _layer_list(case)],
                            case["dtype"])
        st["grads"] = st["stack"].alloc_grads(d["params"])
        return st
    ld = 2 * Hr if case["reverse"] else Hr
    st["layer"] = Layer(T, B, I, H, Hp, case["dtype"], case["reverse"], ldy=ld)
    st["y"] = [torch.zeros((T, B, ld), dtype=td, device="cuda")[:, :, ld - Hr:] for _ in d["x"]]
    st["hT"] = torch.empty((B, Hr), dtype=td, device="cuda")
    st["cT"] = torch.empty((B, H), dtype=torch.float32, device="cuda")
    if case["kind"] == "layer":
        st["dx"] = [torch.empty((T, B, I), dtype=td, device="cuda") for _ in d["x"]]
        st["dh0"] = torch.empty((B, Hr), dtype=td, device="cuda") if case["states"] else None
        st["dc0"] = torch.empty((B, H), dtype=torch.float32, device="cuda") if case["states"] else None
        p = d["params"][0][0]
        st["grads"] = {"d" + k: torch.empty(v.shape, dtype=torch.float32, device="cuda") for k, v in p.items()}
    return st


def run(state):
    s = state
    if s["kind"] == "stack":
        y = s["stack"].forward(s["x"][0], s["params"])
        dx = s["stack"].backward(s["dy"][0], s["params"], s["grads"])
        out = {"y": y, "dx": dx}
        for l, dirs in enumerate(s["grads"]):
            for k, g in enumerate(dirs):
                for n, v in g.items():
                    out["%d.%d.%s" % (l, k, n)] = v
        return out
    lay, p = s["layer"], s["params"][0][0]
    if s["kind"] == "serve":
        lstm355.lstm_forward_noalloc(lay.handle, s["x"][0], s["h0"], s["c0"], p["W"], p["R"], p["b"], p.get("P"),
                                     s["y"][0], s["hT"], s["cT"], lay.reserve)
        return {"y": s["y"][0], "hT": s["hT"], "cT": s["cT"]}
    out = {}
    for m, x in enumerate(s["x"]):
        lay.forward(x, p["W"], p["R"], p["b"], p.get("P"), s["h0"], s["c0"], s["y"][m], s["hT"], s["cT"])
        lay.backward(s["dy"][m], x, p["W"], p["R"], s["y"][m], s["grads"], P=p.get("P"), h0=s["h0"], c0=s["c0"],
                     dhT=s["dhT"], dcT=s["dcT"], dx=s["dx"][m], dh0=s["dh0"], dc0=s["dc0"], accumulate=m > 0)
        out["y%d" % m], out["dx%d" % m] = s["y"][m], s["dx"][m]
    out.update(hT=s["hT"], cT=s["cT"], **s["grads"])   # the states' gradients of the last mini-batch
    if s["dh0"] is not None:
        out.update(dh0=s["dh0"], dc0=s["dc0"])
    return out


# ---------------------------------------------------------------------------
# what a pass cannot do without, and what it should give
# ---------------------------------------------------------------------------
def work(case):
    T, B, m = case["T"], case["B"], case["micro"]
    es = 2 if case["dtype"] == "bf16" else 4
    train = case["kind"] != "serve"
    layers = _layer_list(case)
    flops = nbytes = 0.0
    for I, H, Hp, bi, _ in layers:
        Hr, dirs = Hp or H, 2 if bi else 1
        f = 2.0 * T * B * 4 * H * (I + Hr) + 2.0 * T * B * H * Hp
        flops += dirs * m * f * (3 if train else 1)
        weights = 4 * H * (I + Hr) + Hp * H
        nbytes += dirs * (weights * es + 16 * H)
        if train:
            nbytes += dirs * (weights * 4 + 16 * H)
    Hr0 = layers[-1][2] or layers[-1][1]
    io = T * B * (case["I"] + Hr0 * (2 if layers[-1][3] else 1)) * es
    nbytes += m * io * (2 if train else 1)      # x, y and, in training, dx, dy
    if case["kind"] != "stack":
        st = B * (Hr0 * es + case["H"] * 4)
        nbytes += st * (1 + (1 if case["states"] else 0)) * (2 if train and case["states"] else 1)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times the largest distance from `exact` that the listed and
    some drawn cases show.  bf16: h and the gate gradients are rounded to 8
    bits every step, and a rounding travels through all later steps and
    layers.  fp32: sums of up to 32768 products, and gate functions from the
    hardware's exponential and reciprocal."""
    if case["dtype"] == "f32":
        return {"rel": 6e-6}
    if case["kind"] == "stack":
        return {"rel": 5.5e-2 if case["bi"] else 2.2e-2}
    return {"rel": 1.7e-2 if case["Hp"] else 1.2e-2}


def _cell(z, c):
    i, f, g, o = z.chunk(4, dim=1)
    c = torch.sigmoid(f) * c + torch.sigmoid(i) * torch.tanh(g)
    return torch.sigmoid(o) * torch.tanh(c), c


def _layer64(x, p, h0, c0, reverse):
    T, B = x.shape[0], x.shape[1]
    H = p["b"].numel() // 4
    z = torch.addmm(p["b"], x.reshape(T * B, -1), p["W"].t()).view(T, B, 4 * H)
    h = h0 if h0 is not None else x.new_zeros(B, p["R"].shape[1])
    c = c0 if c0 is not None else x.new_zeros(B, H)
    ys = [None] * T
    for t in (range(T - 1, -1, -1) if reverse else range(T)):
        h, c = _cell(z[t] + h @ p["R"].t(), c)
        if "P" in p:
            h = h @ p["P"].t()
        ys[t] = h
    return torch.stack(ys), h, c


def exact(case, seed):
    d = _inputs(case, seed)
    train = case["kind"] != "serve"

    def f64(v, grad=train):
        return None if v is None else v.double().requires_grad_(grad)

    params = [[{k: f64(v) for k, v in p.items()} for p in dirs] for dirs in d["params"]]
    if case["kind"] == "stack":
        x = f64(d["x"][0])
        cur = x
        for (_, _, _, bi, res), dirs in zip(_layer_list(case), params):
            ys = [_layer64(cur, p, None, None, k == 1)[0] for k, p in enumerate(dirs)]
            y = torch.cat(ys, dim=2) if bi else ys[0]
            cur = y + cur if res else y
        cur.backward(d["dy"][0].double())
        out = {"y": cur.detach(), "dx": x.grad}
        for l, dirs in enumerate(params):
            for k, p in enumerate(dirs):
                for n, v in p.items():
                    out["%d.%d.d%s" % (l, k, n)] = v.grad
        return _ordered(out)
    p = params[0][0]
    if not train:
        y, hT, cT = _layer64(f64(d["x"][0]), p, f64(d["h0"]), f64(d["c0"]), case["reverse"])
        return {"y": y, "hT": hT, "cT": cT}
    out = {}
    for m in range(case["micro"]):
        x, h0, c0 = f64(d["x"][m]), f64(d["h0"]), f64(d["c0"])
        y, hT, cT = _layer64(x, p, h0, c0, case["reverse"])
        loss = (y * d["dy"][m].double()).sum()
        if case["states"]:
            loss = loss + (hT * d["dhT"].double()).sum() + (cT * d["dcT"].double()).sum()
        loss.backward()
        out["y%d" % m], out["dx%d" % m] = y.detach(), x.grad
    out.update(hT=hT.detach(), cT=cT.detach(), **{"d" + k: v.grad for k, v in p.items()})
    if case["states"]:
        out.update(dh0=h0.grad, dc0=c0.grad)
    return out


def _ordered(out):
    """The weight gradients in the order `run` returns them."""
    rank = {"dW": 0, "dR": 1, "db": 2, "dP": 3}
    keys = sorted((k for k in out if "." in k), key=lambda k: (int(k.split(".")[0]), int(k.split(".")[1]),
                                                               rank[k.split(".")[2]]))
    return {"y": out["y"], "dx": out["dx"], **{k: out[k] for k in keys}}
