"""Timed cases of the ChebBooster online stage on one MI355X.

Each case is one call (or the few calls of one step) that a sampler makes
through the package's public entry points: the skipped step's prediction for
one target or for all targets between two full steps, the full step's push,
the residual forms, and the stateless combination.  Sizes are those of the
workloads the repository is exercised on (DiT-XL/2, PixArt-Sigma, FLUX.1-dev
and the single-tensor one), at the batch sizes and history lengths of the
paper's tables, plus odd token counts and ragged tensors.

``listed()`` names the cases, ``draw(rng)`` gives more of the same ranges,
``prepare`` builds what a program holds before the call, ``run`` is one pass,
``work`` the bytes and operations it cannot do without, ``exact`` the same
result in 64-bit arithmetic and plain torch.
"""
import math
from fractions import Fraction

import numpy as np
import torch

import paper_2608_23429_amd as cheb

DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
STEPS = 50                       # sampling steps; abscissa of step s is 1 - s / STEPS


# -- the cases ---------------------------------------------------------------

def _case(name, kind, family, n, m, dtype="bf16", layout="slots", batch=1, tokens=1, text=0,
          hidden=1152, blocks=28):
    c = {"kind": kind, "family": family, "n": n, "m": m, "dtype": dtype, "layout": layout,
         "batch": batch, "tokens": tokens, "text": text, "hidden": hidden, "blocks": blocks}
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # One small tensor, four entries: the smallest call there is, where
        # the launch and the host path count.
        _case("tiny_predict", "predict", "flat", 4, 1, "f32", batch=2, tokens=256),
        # A caller's own tensors, no ring, and a size that is no multiple of
        # a 16-byte vector.
        _case("odd_combine", "combine", "flat", 3, 1, "f16", tokens=1179653, hidden=1),
        # DiT-XL/2 256x256, batch 8 with guidance, one skipped step.
        _case("dit256_predict", "predict", "dit", 5, 1, batch=16, tokens=256),
        # FLUX.1-dev 1024x1024, one skipped step: the largest prediction.
        _case("flux_predict", "predict", "flux", 6, 1, layout="interleaved", tokens=4096, text=512,
              hidden=3072, blocks=19),
        # PixArt-Sigma 1024x1024 in half precision: all skipped steps between
        # two full ones from one pass.
        _case("pixart1024_multi", "multi", "dit", 6, 3, "f16", batch=2, tokens=4096),
        # PixArt-Sigma 512x512, refresh 6 and two entries (the paper's
        # FLOPs headline setting), rows from the offline table.
        _case("pixart512_steps", "steps", "dit", 2, 5, batch=2, tokens=1024),
        # FLUX.1-dev: a full step's 76 module outputs stored in the ring.
        _case("flux_push", "push", "flux", 2, 1, tokens=4096, text=512, hidden=3072, blocks=19),
        # DiT-XL/2 256x256 for one image with guidance, interval 3, three
        # entries: the ring filled, then both skipped steps predicted.
        _case("dit256_online", "online", "dit", 3, 2, layout="interleaved", batch=2, tokens=256),
        # FLUX.1-dev: a skipped step applied to the residual stream.
        _case("flux_residual", "residual", "flux", 6, 1, layout="interleaved", tokens=4096,
              text=512, hidden=3072, blocks=19),
        # The same for DiT-XL/2 256x256, one image with guidance.
        _case("dit256_residual", "residual", "dit", 3, 1, batch=2, tokens=256),
        # FLUX.1-dev: a full step folded into one residual-sized entry.
        _case("flux_collapse", "collapse", "flux", 2, 1, tokens=4096, text=512, hidden=3072,
              blocks=19),
        # DiT-XL/2 512x512, batch 8 with guidance, collapsed history kept
        # from the residual stream: one full and one skipped step.
        _case("dit512_collapsed", "collapsed", "flat", 4, 1, "f32", batch=16, tokens=1024),
    ]


KINDS = ("predict", "predict", "multi", "steps", "push", "online", "residual", "residual",
         "collapse", "collapsed", "combine")
MAX_BYTES = 6e9                  # of a drawn case, about half the largest listed one
MAX_VALUES = 8e8                 # of all its outputs
# Elements of one entry: from a small tensor to the largest listed cache.
MIN_ENTRY, MAX_ENTRY = 5e5, 8e8


def draw(rng):
    """One more case: any call, history of 1 to 8, up to 5 targets, every
    storage type and layout, entries of 5e5 to 8e8 elements, odd token
    counts, and for calls that take them tensors whose size is no multiple
    of 16 bytes."""
    while True:
        kind = rng.choice(KINDS)
        n = rng.choice((1, 2, 2, 3, 3, 4, 5, 6, 6, 7, 8))
        m = rng.randint(2, 5) if kind in ("multi", "steps", "online") else 1
        dtype = rng.choice(("bf16", "bf16", "bf16", "f16", "f32"))
        layout = rng.choice(("slots", "interleaved"))
        family = rng.choice(("dit", "dit", "flux"))
        size = math.exp(rng.uniform(math.log(MIN_ENTRY), math.log(MAX_ENTRY)))
        hidden = rng.choice((384, 768, 1152, 1152, 3072))
        if kind in ("predict", "multi", "steps", "push", "online") and rng.random() < 0.2:
            hidden = rng.choice((385, 1155, 3077))
        if kind in ("combine", "collapsed"):
            tokens = int(size) | 1 if kind == "combine" else max(1, int(min(size, 6e7)) // 1152)
            c = _case(None, kind, "flat", n, m, "f32" if kind == "collapsed" else dtype,
                      tokens=tokens, hidden=1 if kind == "combine" else 1152)
        else:
            blocks = rng.randint(1, 28 if family == "dit" else 19)
            batch = rng.choice((1, 2, 2, 4, 16)) if family == "dit" else 1
            per = size / (hidden * batch * blocks * (2 if family == "dit" else 3))
            tokens = max(1, int(per))
            text = rng.choice((0, rng.randint(1, 511), 512)) if family == "flux" else 0
            text = min(text, tokens)
            c = _case(None, kind, family, n, m, dtype, layout if kind != "collapse" else "slots",
                      batch, tokens, text, hidden, blocks)
        outputs = sum(_segments(c)) * (m if kind not in ("residual", "collapse") else 0)
        if work(c)["bytes"] <= MAX_BYTES and outputs <= MAX_VALUES:
            return c


# -- shapes and schedule -------------------------------------------------------

def _segments(c):
    """Element counts of the cached tensors of one full step."""
    if c["family"] == "flat":
        return [c["batch"] * c["tokens"] * c["hidden"]]
    if c["family"] == "dit":
        return [c["batch"] * c["tokens"] * c["hidden"]] * (2 * c["blocks"])
    img, txt = c["tokens"] * c["hidden"], c["text"] * c["hidden"]
    joint = img + txt
    return [img, txt] * c["blocks"] + [joint] * (2 * c["blocks"])


def _residual_map(c):
    """(residual offset of each cached tensor, residual elements): text
    tokens first, image tokens after them, joint tensors over both."""
    segs = _segments(c)
    if c["family"] != "flux":
        return [0] * len(segs), segs[0]
    img, txt = segs[0], segs[1]
    return [txt, 0] * c["blocks"] + [0] * (2 * c["blocks"]), img + txt


def _schedule(c):
    """(refresh interval, steps of the held entries, skipped steps)."""
    r = 4 if c["m"] == 1 else c["m"] + 1
    nodes = [1 + r * j for j in range(c["n"])]
    return r, nodes, [nodes[-1] + 1 + j for j in range(c["m"])]


def _x(step):
    return 1.0 - step / STEPS


def _offsets(c):
    """Offsets of the tensors in one flat entry (16-byte vectors), and its size."""
    vec = 4 if c["dtype"] == "f32" else 8
    off, pos = [], 0
    for n in _segments(c):
        off.append(pos)
        pos += -(-n // vec) * vec
    return off, pos


# -- inputs --------------------------------------------------------------------

def _features(c, seed, steps):
    """Per cached tensor, its stored values at the given steps: a random
    quadratic of the step per element plus noise, as in the repository's
    generator, rounded once to the storage type."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    for n in _segments(c):
        c0, c1, c2 = (torch.randn(n, generator=g, device="cuda") for _ in range(3))
        out = []
        for s in steps:
            v = torch.randn(n, generator=g, device="cuda").mul_(0.02)
            t = _x(s)
            v.add_(c0).add_(c1, alpha=t).add_(c2, alpha=t * t)
            out.append(v.to(DTYPES[c["dtype"]]))
        yield out


def _stream_values(c, seed):
    """A residual stream before the block stack, fp32."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) + 1_000_003)
    return torch.randn(_residual_map(c)[1], generator=g, device="cuda").mul_(3.0)


def prepare(case, seed):
    c = case
    r, nodes, targets = _schedule(c)
    kind, n, m = c["kind"], c["n"], c["m"]
    dt = DTYPES[c["dtype"]]
    s = {"kind": kind, "n": n, "x": [_x(v) for v in targets], "t": 0.0}
    if kind == "combine":
        s["srcs"] = next(_features(c, seed, nodes))
        s["w"] = _row(nodes, targets[0])
        s["out"] = torch.empty_like(s["srcs"][0])
        return s
    if kind == "collapsed":
        # The residual stream before and after the block stack of the full
        # steps; all but the newest are in the history already.
        hist = cheb.ResidualHistory(n, [0], _segments(c)[0])
        before = _stream_values(c, seed)
        after = [f.add_(before) for f in next(_features(c, seed, nodes))]
        for step, x_after in zip(nodes[:-1], after):
            hist.push_difference(_x(step), x_after, before)
        s.update(hist=hist, before=before, x_out=torch.empty_like(before), after=after, k=n - 1,
                 nodes=[_x(v) for v in nodes])
        return s
    if kind in ("push", "collapse"):
        s["segs"] = [f[0] for f in _features(c, seed, nodes[:1])]
        if kind == "push":
            s["cache"] = cheb.ChebCache(n, dt, _segments(c), layout=c["layout"])
            if c["layout"] == "interleaved":
                s["cache"].arena.zero_()
        else:
            off, size = _residual_map(c)
            s["hist"] = cheb.ResidualHistory(n, off, size)
        return s
    cache = cheb.ChebCache(n, dt, _segments(c), layout=c["layout"])
    s["cache"] = cache
    if kind == "online":
        s["full"] = [list(f) for f in zip(*_features(c, seed, nodes))]
        s["nodes"] = [_x(v) for v in nodes]
    else:
        # Written straight into a flat buffer per entry, then pushed.
        off, size = _offsets(c)
        flats = [torch.zeros(size, dtype=dt, device="cuda") for _ in nodes]
        for o, cnt, vals in zip(off, _segments(c), _features(c, seed, nodes)):
            for f, v in zip(flats, vals):
                f[o:o + cnt] = v
        for step, f in zip(nodes, flats):
            cache.push(_x(step), cache.segment_views(f))
    if kind == "residual":
        s["off"], size = _residual_map(c)
        s["x_in"] = _stream_values(c, seed)
        s["x_out"] = torch.empty_like(s["x_in"])
        return s
    s["outs"] = [cache.new_output() for _ in range(m)]
    if kind == "steps":
        s["table"] = cheb.ChebTable(STEPS, 1, 1, r, n, [_x(v) for v in range(STEPS)],
                                    cheb.CHEB_SHORT_LOWER)
        s["first"] = targets[0]
    return s


def run(state):
    s = state
    kind = s["kind"]
    if kind == "predict":
        out, w = s["cache"].extrapolate_at(s["x"][0], s["outs"][0])
        return {"out": out, "w": w}
    if kind == "multi":
        outs, w = s["cache"].extrapolate_at_multi(s["x"], s["outs"])
        return {"out": outs, "w": w}
    if kind == "steps":
        return {"out": s["cache"].extrapolate_steps(s["table"], s["first"], len(s["outs"]),
                                                    s["outs"])}
    if kind == "combine":
        return {"out": cheb.combine(s["srcs"], s["w"], s["out"])}
    if kind == "push":
        cache = s["cache"]
        if cache.layout == "interleaved":
            cache.reset()                      # a new sampling run's first full step
            cache.push(0.0, s["segs"])
            return {"arena": cache.arena.view(cache.dtype)}
        s["t"] -= 1.0                          # the oldest entry makes room
        cache.push(s["t"], s["segs"])
        return {"entry": cache.entry(len(cache.history()) - 1)}
    if kind == "online":
        cache = s["cache"]
        cache.reset()
        for x, segs in zip(s["nodes"], s["full"]):
            cache.push(x, segs)
        outs, w = cache.extrapolate_at_multi(s["x"], s["outs"])
        return {"out": outs, "w": w}
    if kind == "residual":
        cache = s["cache"]
        w = cheb.cheb_precompute_weights(cache.history(), s["x"][:1])[0]
        return {"x": cache.residual_apply(w, s["off"], s["x_out"], s["x_in"]), "w": w}
    if kind == "collapse":
        hist = s["hist"]
        s["t"] -= 1.0
        hist.push(s["t"], s["segs"])
        return {"entry": hist.cache.entry(len(hist.history()) - 1)}
    # collapsed: the newest full step's entry, then the skipped step.  Once
    # the ring is full, each pass replaces the oldest entry by its like.
    hist, k = s["hist"], s["k"]
    s["k"] = (k + 1) % s["n"]
    hist.push_difference(s["nodes"][k], s["after"][k], s["before"])
    return {"x": hist.predict(s["x"][0], s["x_out"], s["before"])[0]}


# -- what a pass cannot do without ---------------------------------------------

def work(case):
    c = case
    kind, n, m = c["kind"], c["n"], c["m"]
    esz = 4 if c["dtype"] == "f32" else 2
    numel = sum(_segments(c))
    predict = {"bytes": (n + m) * numel * esz, "flops": 2 * n * m * numel}
    if kind == "push":
        return {"bytes": 2 * numel * esz, "flops": 0}
    if kind == "online":
        return {"bytes": predict["bytes"] + 2 * n * numel * esz, "flops": predict["flops"]}
    if kind == "residual":
        return {"bytes": n * numel * esz + 8 * _residual_map(c)[1], "flops": 2 * n * numel}
    if kind == "collapse":
        return {"bytes": numel * esz + 4 * _residual_map(c)[1], "flops": numel}
    if kind == "collapsed":
        return {"bytes": (3 + n + 2) * numel * 4, "flops": (2 * n + 3) * numel}
    return predict


def tolerance(case):
    """Errors against 64-bit sums, times about four: one rounding of each
    result to its storage type, and for the collapsed history one more of
    each entry, times the weights."""
    if case["kind"] == "push":
        return "exact"                         # a copy
    if case["kind"] in ("residual", "collapse"):
        return {"rel": 1.2e-7}
    if case["kind"] == "collapsed":
        return {"rel": 1e-6}
    return {"rel": {"bf16": 7e-3, "f16": 9e-4, "f32": 1.2e-7}[case["dtype"]]}


# -- the same in 64 bits -------------------------------------------------------

def _row(nodes, target):
    """Lagrange coefficients of the abscissae at the target, exact and then
    rounded to fp64."""
    x = [Fraction(_x(v)) for v in nodes]
    t = Fraction(_x(target))
    out = []
    for j, xj in enumerate(x):
        w = Fraction(1)
        for k, xk in enumerate(x):
            if k != j:
                w *= (t - xk) / (xj - xk)
        out.append(float(w))
    return np.array(out, dtype=np.float64)


def _sum(w, values):
    acc = torch.zeros(values[0].numel(), dtype=torch.float64, device="cuda")
    for a, v in zip(w, values):
        acc.add_(v.double(), alpha=float(a))
    return acc


def exact(case, seed):
    c = case
    _, nodes, targets = _schedule(c)
    kind = c["kind"]
    if kind == "combine":
        return {"out": _sum(_row(nodes, targets[0]), next(_features(c, seed, nodes)))}
    if kind == "collapsed":
        before = _stream_values(c, seed)
        after = [f.add_(before) for f in next(_features(c, seed, nodes))]
        x = before.double()
        for a, f in zip(_row(nodes, targets[0]), after):
            x.add_(f.double().sub_(before), alpha=float(a))
        return {"x": x}
    if kind == "push":
        if c["layout"] == "interleaved":
            return None                        # a copy; its places are the ring's own
        off, size = _offsets(c)
        entry = torch.zeros(size, dtype=torch.float64, device="cuda")
        for o, cnt, f in zip(off, _segments(c), _features(c, seed, nodes[:1])):
            entry[o:o + cnt] = f[0]
        return {"entry": entry}
    if kind in ("residual", "collapse"):
        off, size = _residual_map(c)
        w = _row(nodes, targets[0]) if kind == "residual" else np.ones(1)
        x = torch.zeros(size, dtype=torch.float64, device="cuda")
        if kind == "residual":
            x += _stream_values(c, seed)
        steps = nodes if kind == "residual" else nodes[:1]
        for o, cnt, f in zip(off, _segments(c), _features(c, seed, steps)):
            x[o:o + cnt] += _sum(w, f)
        return {"x": x, "w": w} if kind == "residual" else {"entry": x}
    rows = [_row(nodes, t) for t in targets]
    off, size = _offsets(c)
    outs = [torch.zeros(size, dtype=torch.float64, device="cuda") for _ in targets]
    for o, cnt, f in zip(off, _segments(c), _features(c, seed, nodes)):
        for out, w in zip(outs, rows):
            out[o:o + cnt] = _sum(w, f)
    if kind == "steps":
        return {"out": outs}
    return {"out": outs[0], "w": rows[0]} if kind == "predict" else {"out": outs,
                                                                     "w": np.stack(rows)}
