"""What the framework is timed on: passes through its public entry points as a user's program makes them.

A case is a dict of plain values.  `kind` says which pass it is:

  conv      a stack of convolutions of one shape over packed layers (inference over one pruned layer or head)
  coherent  the same over layers whose patterns are shared in blocks (masks taken over from a parent layer)
  step      selection + packing + the stack: what every round of pruning runs on a layer group
  pyramid   one head's stack applied to every level of a feature pyramid, each level half the one before
  block     a bottleneck block with folded batch-norm, SiLU, shortcut and concatenation, any data type
  detector  the forward of the 57-layer convolution set, wired as a detector with fused output stages, either
            replayed from a HIP graph (batched throughput) or called layer by layer (one frame at a time)
  odd       a 3x3 and a 1x1 layer whose channel counts are no multiples of a matrix tile
  prune     selection and packing of every layer of the convolution set
  usage     selection over random kernels and the usage count behind a reduced dictionary

Sizes are those of the five configurations in workloads.py (single 3x3 layer, 1x1 layer, detection head, 640x640
convolution set) and of the benchmark's sweep over the number of entries per pattern, widened to ranges.
"""
import numpy as np
import torch

from paper_2303_02191_amd import binding as B
from paper_2303_02191_amd import pipeline as pl
from paper_2303_02191_amd import workloads as wl

F32, F16, BF16 = B.F32, B.F16, B.BF16
DTYPES = {"f32": F32, "f16": F16, "bf16": BF16}


# ---------------------------------------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------------------------------------
def listed():
    return [
        # the smallest call: one fp32 layer on one image, where launch and host time count (configuration 1)
        {"name": "layer_f32_n1", "kind": "conv", "dt": "f32", "k": 4, "ks": 3, "ci": 64, "co": 64, "n": 1, "h": 56, "w": 56,
         "stride": 1, "depth": 1},
        # an ordinary memory-bound 1x1 layer (configuration 3)
        {"name": "conv1x1_f16_n8", "kind": "conv", "dt": "f16", "k": 2, "ks": 1, "ci": 256, "co": 256, "n": 8, "h": 80, "w": 80,
         "stride": 1, "depth": 1},
        # dictionaries without a 2-of-4 shape: the 5-entry point of the sweep over k, on the detection head
        {"name": "head_5ep_bf16_n2", "kind": "conv", "dt": "bf16", "k": 5, "ks": 3, "ci": 256, "co": 256, "n": 2, "h": 100,
         "w": 168, "stride": 1, "depth": 4},
        # the detection head pruned and run: the benchmark's default step (configuration 4)
        {"name": "head_step_bf16_n4", "kind": "step", "dt": "bf16", "k": 3, "ks": 3, "ci": 256, "co": 256, "n": 4, "h": 100,
         "w": 168, "stride": 1, "depth": 4},
        # the same head with masks shared in blocks
        {"name": "head_coherent_bf16_n4", "kind": "coherent", "dt": "bf16", "k": 3, "ks": 3, "ci": 256, "co": 256, "n": 4,
         "h": 100, "w": 168, "stride": 1, "depth": 4},
        # the head over all levels of its pyramid, on one image: the levels are ragged and most of them small
        {"name": "pyramid_bf16_n1", "kind": "pyramid", "dt": "bf16", "k": 3, "c": 256, "n": 1, "h": 100, "w": 168, "levels": 5,
         "depth": 4},
        # one block in fp32, the precision models are trained in
        {"name": "block_f32_n4", "kind": "block", "dt": "f32", "k": 3, "c": 128, "n": 4, "h": 80, "w": 80, "reps": 2},
        # batched detector forward (configuration 5's layers)
        {"name": "detector_f16_n16", "kind": "detector", "dt": "f16", "k": 2, "n": 16, "h": 640, "w": 640, "graph": True},
        # one camera frame at a time, called layer by layer
        {"name": "detector_f16_n1", "kind": "detector", "dt": "f16", "k": 3, "n": 1, "h": 640, "w": 640, "graph": False},
        # channel counts between matrix tiles (scaled-width models, class outputs)
        {"name": "odd_channels_f16_n4", "kind": "odd", "dt": "f16", "k": 2, "ci": 48, "mid": 72, "co": 255, "n": 4, "h": 77,
         "w": 91, "stride": 1},
        # pruning a whole model: configuration 5's 57 layers
        {"name": "prune_f16", "kind": "prune", "dt": "f16", "k": 2, "width": 32},
        # usage count over random kernels (2^20 of them, as the benchmark draws)
        {"name": "usage_f32", "kind": "usage", "dt": "f32", "k": 3, "kernels": 1 << 20},
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, spread over its logarithm."""
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["conv", "conv", "conv1x1", "step", "coherent", "pyramid", "block", "detector", "odd", "prune", "usage"])
    dt16 = rng.choice(["f16", "bf16"])
    if kind == "conv1x1":
        ci, co = 32 * rng.choice([1, 2, 3, 4, 6, 8, 12, 16, 32]), 16 * _log(rng, 2, 32)
        h = _log(rng, 10, 160)
        return {"kind": "conv", "dt": dt16, "k": rng.choice([2, 3]), "ks": 1, "ci": ci, "co": co, "n": _log(rng, 1, 8), "h": h,
                "w": max(1, h + rng.randint(-5, 40)), "stride": 1, "depth": 1}
    if kind in ("conv", "step", "coherent"):
        h = _log(rng, 14, 112)
        dt = rng.choice(["f32", dt16, dt16]) if kind == "conv" else dt16
        c = 32 * _log(rng, 1, 4 if dt == "f32" else 8)
        k = rng.choice([2, 3, 3, 4, 5]) if kind == "conv" else rng.choice([2, 3])
        stride = rng.choice([1, 1, 2]) if kind == "conv" else 1
        return {"kind": kind, "dt": dt, "k": k, "ks": 3, "ci": c, "co": 2 * c if stride == 2 else c,
                "n": _log(rng, 1, 4), "h": h, "w": max(1, h + rng.randint(-5, 50)), "stride": stride,
                "depth": 1 if stride == 2 else rng.randint(1, 2 if dt == "f32" else 4)}
    if kind == "pyramid":
        h = _log(rng, 40, 112)
        return {"kind": kind, "dt": dt16, "k": rng.choice([2, 3]), "c": rng.choice([128, 256]), "n": _log(rng, 1, 4), "h": h,
                "w": h + rng.randint(0, 60), "levels": rng.randint(3, 5), "depth": rng.randint(2, 4)}
    if kind == "block":
        c = rng.choice([64, 128, 256, 512])
        h = _log(rng, 20, 10240 // c)
        return {"kind": kind, "dt": rng.choice(["f32", dt16]), "k": rng.choice([2, 3]), "c": c, "n": _log(rng, 1, 8), "h": h,
                "w": h + rng.randint(-3, 20), "reps": rng.randint(1, 3)}
    if kind == "detector":
        return {"kind": kind, "dt": dt16, "k": rng.choice([2, 3]), "n": _log(rng, 1, 16), "h": 32 * rng.randint(10, 20),
                "w": 32 * rng.randint(10, 20), "graph": rng.random() < 0.5}
    if kind == "odd":
        h = _log(rng, 13, 120)
        return {"kind": kind, "dt": rng.choice(["f32", dt16, dt16]), "k": rng.choice([2, 3]), "ci": rng.choice([24, 40, 48, 80]),
                "mid": rng.choice([36, 48, 72, 80]), "co": rng.choice([36, 85, 120, 255]), "n": _log(rng, 1, 4), "h": h,
                "w": max(1, h + rng.randint(-5, 30)), "stride": rng.choice([1, 1, 2])}
    if kind == "prune":
        return {"kind": kind, "dt": rng.choice(["f32", dt16, dt16]), "k": rng.choice([2, 3, 4]), "width": rng.choice([16, 24, 32, 48])}
    return {"kind": kind, "dt": rng.choice(["f32", dt16]), "k": rng.choice([2, 3, 4, 5]), "kernels": _log(rng, 1 << 14, 1 << 20)}


# ---------------------------------------------------------------------------------------------------------
# the wired convolution set: (input, output) of every layer by name; "cat.a:b" is a channel slice of a
# concatenation buffer.  What operations outside this framework would put there (pooled, upsampled and copied
# maps) is part of the inputs.
# ---------------------------------------------------------------------------------------------------------
def _wiring(width):
    """Layers in call order as dicts: ci, co, ks, stride, level (log2 of the down-scaling of the input), x, y, and the
    shortcut; and the concatenation buffers (channels, level)."""
    u = width  # channel widths are multiples of the stem's
    layers, cats = [], {}

    def add(x, y, ci, co, level, ks=1, stride=1, shortcut=None):
        layers.append({"x": x, "y": y, "ci": ci, "co": co, "level": level, "ks": ks, "stride": stride, "shortcut": shortcut})

    def block(tag, x, cin, mid, level, reps, cout, shortcut=True):
        cats[tag] = (2 * mid, level)
        add(x, tag + ".t0", cin, mid, level)
        add(x, "%s:%d" % (tag, mid), cin, mid, level)
        for r in range(reps):
            here, last = "%s.t%d" % (tag, r), r == reps - 1
            add(here, tag + ".m%d" % r, mid, mid, level)
            add(tag + ".m%d" % r, "%s:0" % tag if last else "%s.t%d" % (tag, r + 1), mid, mid, level, 3,
                shortcut=here if shortcut else None)
        add(tag, tag + ".out", 2 * mid, cout, level)

    add("image", "s1", 3, u, 0, 3, 2)
    add("s1", "s2", u, 2 * u, 1, 3, 2)
    block("b2", "s2", 2 * u, u, 2, 1, 2 * u)
    add("b2.out", "s3", 2 * u, 4 * u, 2, 3, 2)
    block("b3", "s3", 4 * u, 2 * u, 3, 2, 4 * u)
    add("b3.out", "s4", 4 * u, 8 * u, 3, 3, 2)
    block("b4", "s4", 8 * u, 4 * u, 4, 3, 8 * u)
    add("b4.out", "s5", 8 * u, 16 * u, 4, 3, 2)
    block("b5", "s5", 16 * u, 8 * u, 5, 1, 16 * u)
    cats["pool"] = (32 * u, 5)
    add("b5.out", "pool:0", 16 * u, 8 * u, 5)
    add("pool", "p5", 32 * u, 16 * u, 5)
    add("p5", "up5", 16 * u, 8 * u, 5)
    cats["join4"] = (16 * u, 4)
    block("h4", "join4", 16 * u, 4 * u, 4, 1, 8 * u, False)
    add("h4.out", "up4", 8 * u, 4 * u, 4)
    cats["join3"] = (8 * u, 3)
    block("h3", "join3", 8 * u, 2 * u, 3, 1, 4 * u, False)
    cats["down4"] = (8 * u, 4)
    add("h3.out", "down4:0", 4 * u, 4 * u, 3, 3, 2)
    block("o4", "down4", 8 * u, 4 * u, 4, 1, 8 * u, False)
    cats["down5"] = (16 * u, 5)
    add("o4.out", "down5:0", 8 * u, 8 * u, 4, 3, 2)
    block("o5", "down5", 16 * u, 8 * u, 5, 1, 16 * u, False)
    return layers, cats


_FORWARD_OUTPUTS = ["up5", "up4", "h3.out", "o4.out", "o5.out"]


# ---------------------------------------------------------------------------------------------------------
# preparation
# ---------------------------------------------------------------------------------------------------------
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(g, shape, dt, std=1.0):
    return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * std).to(pl.TORCH_DTYPE[dt])


def _weights(g, co, ci, ks, dt):
    """Weights that keep the activations of a pruned layer near unit size (the selection keeps the large ones)."""
    return _normal(g, (co, ci, ks, ks), dt, 1.0 / np.sqrt(ci * (3 if ks == 3 else 0.5)))


def _prune_and_pack(ws, dt, k, masks):
    """Packed layers of several weight tensors, with one selection and one packing call."""
    idxs = pl.select_patterns_batch(ws, dt, masks)
    layers = [pl.PackedLayer(w.shape[0], w.shape[1], w.shape[2], k, dt, masks) for w in ws]
    pl.pack_layers(layers, ws, idxs)
    return layers


def _affine(g, co):
    """Folded batch normalisation of one layer."""
    return (torch.rand(co, generator=g, device="cuda") * 0.4 + 0.8, torch.randn(co, generator=g, device="cuda") * 0.1)


def _stack_shapes(case):
    ho, wo = (case["h"] - 1) // case["stride"] + 1, (case["w"] - 1) // case["stride"] + 1
    return ho, wo


def _prepare_stack(case, g):
    dt, k, n = DTYPES[case["dt"]], case["k"], case["n"]
    masks = B.rtoss_pattern_dict(k)
    ws = [_weights(g, case["co"], case["ci"], case["ks"], dt) for _ in range(case["depth"])]
    state = {"x": _normal(g, (n, case["h"], case["w"], case["ci"]), dt), "stride": case["stride"]}
    if case["kind"] == "conv":
        state["layers"] = _prune_and_pack(ws, dt, k, masks)
    elif case["kind"] == "coherent":
        state["layers"] = []
        for w in ws:
            # patterns chosen per run of 8 input channels by the parent and shared down the output channels
            runs = torch.randint(len(masks), (case["ci"] // 8,), generator=g, device="cuda").to(torch.uint8)
            idx = runs.repeat_interleave(8).repeat(case["co"])
            state["layers"].append(pl.CoherentLayer(case["co"], case["ci"], k, dt, masks).pack(w, idx))
    else:
        state.update(ws=ws, dt=dt, masks=masks)
        state["idxs"] = [torch.empty(w.numel() // 9, dtype=torch.uint8, device="cuda") for w in ws]
        state["layers"] = [pl.PackedLayer(case["co"], case["ci"], case["ks"], k, dt, masks) for _ in ws]
    return state


def _prepare_pyramid(case, g):
    dt, c = DTYPES[case["dt"]], case["c"]
    ws = [_weights(g, c, c, 3, dt) for _ in range(case["depth"])]
    layers = _prune_and_pack(ws, dt, case["k"], B.rtoss_pattern_dict(case["k"]))
    return {"layers": layers, "xs": [_normal(g, (case["n"], h, w, c), dt) for h, w in _levels(case)]}


def _levels(case):
    return [((case["h"] - 1 >> l) + 1, (case["w"] - 1 >> l) + 1) for l in range(case["levels"])]


def _prepare_wired(case, g, layers, cats, size_of, inputs, outputs):
    """Packed layers, buffers and call list of a wired set of fused layers."""
    dt, n = DTYPES[case["dt"]], case["n"]
    ws = [_weights(g, L["co"], L["ci"], L["ks"], dt) for L in layers]
    packed = _prune_and_pack(ws, dt, case["k"], B.rtoss_pattern_dict(case["k"]))
    bufs = {name: _normal(g, (n,) + size_of(level) + (c,), dt) for name, (c, level) in dict(cats, **inputs).items()}
    calls = []
    for L, p in zip(layers, packed):
        into = None
        if ":" in L["y"]:
            name, first = L["y"].split(":")
            into = bufs[name][..., int(first): int(first) + L["co"]]
        scale, bias = _affine(g, L["co"])
        calls.append((p, L["x"], L["y"], L["stride"], scale, bias, L["shortcut"], into))
    return {"calls": calls, "bufs": bufs, "outputs": outputs, "graph": None}


def _wired_pass(state):
    maps = dict(state["bufs"])
    for p, x, y, stride, scale, bias, shortcut, into in state["calls"]:
        maps[y] = p.conv_fused(maps[x], stride=stride, scale=scale, bias=bias, act=B.ACT_SILU,
                               residual=maps[shortcut] if shortcut else None, y=into)
    return [maps[name] for name in state["outputs"]]


def _block_layers(case):
    mid = case["c"] // 2
    layers, cats = [], {"cat": (2 * mid, 0)}

    def add(x, y, ci, co, ks=1, shortcut=None):
        layers.append({"x": x, "y": y, "ci": ci, "co": co, "level": 0, "ks": ks, "stride": 1, "shortcut": shortcut})

    add("in", "t0", case["c"], mid)
    add("in", "cat:%d" % mid, case["c"], mid)
    for r in range(case["reps"]):
        add("t%d" % r, "m%d" % r, mid, mid)
        add("m%d" % r, "cat:0" if r == case["reps"] - 1 else "t%d" % (r + 1), mid, mid, 3, "t%d" % r)
    add("cat", "out", 2 * mid, case["c"])
    return layers, cats


def _prepare_detector(case, g):
    layers, cats = _wiring(32)
    size_of = lambda level: (case["h"] >> level, case["w"] >> level)
    state = _prepare_wired(case, g, layers, cats, size_of, {"image": (3, 0)}, _FORWARD_OUTPUTS)
    if case["graph"]:
        _wired_pass(state)
        torch.cuda.synchronize()
        state["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(state["graph"]):
            state["result"] = _wired_pass(state)
    return state


def _prepare_odd(case, g):
    dt, k = DTYPES[case["dt"]], case["k"]
    ws = [_weights(g, case["mid"], case["ci"], 3, dt), _weights(g, case["co"], case["mid"], 1, dt)]
    layers = _prune_and_pack(ws, dt, k, B.rtoss_pattern_dict(k))
    return {"layers": layers, "stride": case["stride"], "x": _normal(g, (case["n"], case["h"], case["w"], case["ci"]), dt)}


def _prepare_prune(case, g):
    dt, k = DTYPES[case["dt"]], case["k"]
    masks = B.rtoss_pattern_dict(k)
    ws = [_weights(g, L["co"], L["ci"], L["ks"], dt) for L in _wiring(case["width"])[0]]
    layers = [pl.PackedLayer(w.shape[0], w.shape[1], w.shape[2], k, dt, masks) for w in ws]
    groups = [w.numel() // 9 for w in ws]
    at = np.concatenate([[0], np.cumsum(groups)]).tolist()
    idx = torch.empty(at[-1], dtype=torch.uint8, device="cuda")
    idxs = [idx[a:b] for a, b in zip(at, at[1:])]
    # the part of a packed blob that is public: the surviving values, then the pattern indices
    ends = [-(-G * k * wl.ELEM_BYTES[dt] // 256) * 256 + G for G in groups]
    pads = [(G * k * wl.ELEM_BYTES[dt], end - G) for G, end in zip(groups, ends)]
    for lay, (a, b) in zip(layers, pads):
        lay.blob[a:b] = 0
    return {"ws": ws, "dt": dt, "masks": masks, "layers": layers, "idx": idx, "idxs": idxs,
            "public": [lay.blob[:end] for lay, end in zip(layers, ends)]}


def _prepare_usage(case, g):
    dt = DTYPES[case["dt"]]
    w = torch.rand((case["kernels"], 9), generator=g, device="cuda") * 2 - 1
    return {"w": w.to(pl.TORCH_DTYPE[dt]), "dt": dt, "masks": B.rtoss_pattern_dict(case["k"])}


def prepare(case, seed):
    g, kind = _generator(seed), case["kind"]
    if kind in ("conv", "coherent", "step"):
        state = _prepare_stack(case, g)
    elif kind == "pyramid":
        state = _prepare_pyramid(case, g)
    elif kind == "block":
        layers, cats = _block_layers(case)
        state = _prepare_wired(case, g, layers, cats, lambda level: (case["h"], case["w"]), {"in": (case["c"], 0)}, ["out"])
    elif kind == "detector":
        state = _prepare_detector(case, g)
    elif kind == "odd":
        state = _prepare_odd(case, g)
    elif kind == "prune":
        state = _prepare_prune(case, g)
    else:
        state = _prepare_usage(case, g)
    state["kind"] = kind
    return state


# ---------------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------------
def _stack_pass(layers, x, stride):
    for i, lay in enumerate(layers):
        x = lay.conv(x, stride=stride, relu=i < len(layers) - 1)
    return x


def run(state):
    kind = state["kind"]
    if kind in ("conv", "coherent"):
        return _stack_pass(state["layers"], state["x"], state["stride"])
    if kind == "step":
        pl.select_patterns_batch(state["ws"], state["dt"], state["masks"], state["idxs"])
        pl.pack_layers(state["layers"], state["ws"], state["idxs"])
        return [_stack_pass(state["layers"], state["x"], state["stride"])] + state["idxs"]
    if kind == "pyramid":
        return [_stack_pass(state["layers"], x, 1) for x in state["xs"]]
    if kind in ("block", "detector"):
        if state["graph"] is not None:
            state["graph"].replay()
            return state["result"]
        return _wired_pass(state)
    if kind == "odd":
        mid = state["layers"][0].conv(state["x"], stride=state["stride"], relu=True)
        return state["layers"][1].conv(mid)
    if kind == "prune":
        pl.select_patterns_batch(state["ws"], state["dt"], state["masks"], state["idxs"])
        pl.pack_layers(state["layers"], state["ws"], state["idxs"])
        return [state["idx"]] + state["public"]
    idx = pl.select_patterns(state["w"], state["dt"], state["masks"])
    return [idx, pl.pattern_histogram(idx, len(state["masks"]))]


# ---------------------------------------------------------------------------------------------------------
# what a pass cannot do without, and how close two correct results are
# ---------------------------------------------------------------------------------------------------------
def _layer_work(eb, k, n, ci, co, ks, h, w, stride, residual=False):
    """Input and output once, k values and an index byte per group of 9; two operations per surviving weight and position."""
    ho, wo = (h - 1) // stride + 1, (w - 1) // stride + 1
    groups = co * ci * ks * ks // 9
    return (eb * n * (h * w * ci + ho * wo * co * (2 if residual else 1)) + groups * (k * eb + 1), 2 * n * ho * wo * k * groups)


def work(case):
    kind, k = case["kind"], case["k"]
    eb = wl.ELEM_BYTES[DTYPES[case["dt"]]]
    parts = []
    if kind in ("conv", "coherent", "step"):
        parts = [_layer_work(eb, k, case["n"], case["ci"], case["co"], case["ks"], case["h"], case["w"], case["stride"])] * case["depth"]
        if kind == "step":
            parts.append((case["depth"] * case["co"] * case["ci"] * (9 * eb + k * eb + 2), 0))
    elif kind == "pyramid":
        parts = [_layer_work(eb, k, case["n"], case["c"], case["c"], 3, h, w, 1) for h, w in _levels(case)] * case["depth"]
    elif kind in ("block", "detector"):
        layers = _block_layers(case)[0] if kind == "block" else _wiring(32)[0]
        parts = [_layer_work(eb, k, case["n"], L["ci"], L["co"], L["ks"], case["h"] >> L["level"], case["w"] >> L["level"],
                             L["stride"], L["shortcut"] is not None) for L in layers]
    elif kind == "odd":
        ho, wo = _stack_shapes(case)
        parts = [_layer_work(eb, k, case["n"], case["ci"], case["mid"], 3, case["h"], case["w"], case["stride"]),
                 _layer_work(eb, k, case["n"], case["mid"], case["co"], 1, ho, wo, 1)]
    elif kind == "prune":
        for L in _wiring(case["width"])[0]:
            elems = L["co"] * L["ci"] * L["ks"] ** 2
            parts.append((elems * eb + elems // 9 * (k * eb + 2), 0))
    else:
        # every pattern's retained energy of every kernel
        parts = [(case["kernels"] * (9 * eb + 1), case["kernels"] * (9 + len(B.rtoss_pattern_dict(k)) * k))]
    return {"bytes": sum(b for b, _ in parts), "flops": sum(f for _, f in parts)}


def tolerance(case):
    """Selections, packed values and counts are whole numbers and bytes.  Convolutions accumulate in fp32 in any order; a
    16-bit result is rounded once per layer, and a stack passes those roundings on."""
    if case["kind"] in ("prune", "usage"):
        return "exact"
    return {"f32": {"rel": 1e-5}, "f16": {"rel": 2e-3}, "bf16": {"rel": 1e-2}}[case["dt"]]
