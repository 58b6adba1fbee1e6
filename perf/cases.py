"""The work that users of this library have it do, as measurable cases.

A case is a dict of plain values. `listed()` names the standing ones, `draw()`
gives another of the same ranges, `prepare()` makes what a program holds
before the call (device buffers, a plan), `run()` is one pass through the
package's entry points, `work()` the bytes and operations that the pass cannot
do without, and `exact()` the result in 64 bits.

Three kinds of work: one convolution (`Plan`, or `conv2d` with its plan
cache), many uneven convolutions in one launch (`Batch`), and the hotspot
thermal stencil (`Hotspot`). All data is FP32, the library's one type.
"""
import math
import random

import torch

import paper_2407_11488_amd as C

# Filters of the plain path: the odd squares the library ships winners for,
# others without one, and rectangles.
SQUARE = (3, 5, 7, 9, 11, 13, 15, 17, 21, 25, 31)
# Filters of batches and of served requests.
BATCH_FILTERS = (3, 5, 9, 17)


def _conv(name, h, w, fh, fw, **kw):
    return dict(name=name, kind="conv", h=h, w=w, fh=fh, fw=fw, entry="plan", halo=False, **kw)


def listed():
    small = _conv("conv_128_f5_call", 128, 128, 5, 5)
    small["entry"] = "conv2d"
    padded = _conv("conv_1024_f17_zero_ring", 1024, 1024, 17, 17)
    padded["halo"] = True
    return [
        # The headline: a large image under a large filter, tuned.
        _conv("conv_4096_f17", 4096, 4096, 17, 17),
        # The ends of the filter sweep and its middle: bound by memory at 3x3,
        # between the two at 7x7, by arithmetic at 31x31 (the largest case).
        _conv("conv_4096_f3", 4096, 4096, 3, 3),
        _conv("conv_4096_f7", 4096, 4096, 7, 7),
        _conv("conv_4096_f31", 4096, 4096, 31, 31),
        # The ordinary image, padded by the caller to keep its size.
        padded,
        # A ragged image: a size nobody tuned, odd rows, a tuned filter size.
        _conv("conv_2047x3001_f9", 2047, 3001, 9, 9),
        # A filter size nobody tuned (the library's own choice serves it).
        _conv("conv_1500x1111_f11", 1500, 1111, 11, 11),
        # The smallest call, as a script makes it: launch and host latency.
        small,
        # 64 uneven images in one launch, arguments bound once.
        dict(name="batch_64", kind="batch", n=64, lo=256, hi=2048, shapes=3, by_size=False, bound=True),
        # What a server has at hand at a moment: a few smaller images, each
        # with its size's configuration, in buffers it holds.
        dict(name="batch_16_by_size", kind="batch", n=16, lo=128, hi=768, shapes=5, by_size=True, bound=True),
        # The chip simulation, and a smaller, ragged one of fewer steps.
        dict(name="hotspot_4096_s60", kind="hotspot", rows=4096, cols=4096, steps=60),
        dict(name="hotspot_1000x1501_s20", kind="hotspot", rows=1000, cols=1501, steps=20),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    u = rng.random()
    if u < 0.6:
        fh = fw = rng.choice(SQUARE)
        if rng.random() < 0.2:
            fh, fw = rng.randint(1, 17), rng.randint(1, 17)
        return dict(kind="conv", h=_log_int(rng, 128, 4096), w=_log_int(rng, 128, 4096), fh=fh, fw=fw,
                    entry=rng.choice(("plan", "plan", "conv2d")), halo=rng.random() < 0.25)
    if u < 0.8:
        return dict(kind="batch", n=_log_int(rng, 4, 64), lo=128, hi=rng.choice((512, 768, 1024, 2048)),
                    shapes=rng.randint(10, 1 << 20), by_size=rng.random() < 0.5, bound=rng.random() < 0.5)
    return dict(kind="hotspot", rows=_log_int(rng, 256, 4096), cols=_log_int(rng, 256, 4096),
                steps=_log_int(rng, 5, 60))


def _batch_shapes(case):
    rng = random.Random(case["shapes"])
    out = []
    for _ in range(case["n"]):
        side, f = _log_int(rng, case["lo"], case["hi"]), rng.choice(BATCH_FILTERS)
        out.append((side, side, f, f))
    return out


def _shapes(case):
    if case["kind"] == "batch":
        return _batch_shapes(case)
    return [(case["h"], case["w"], case["fh"], case["fw"])]


def _conv_data(case, seed):
    """Inputs and filters, uniform in [-1, 1), on the device."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    ins, filts = [], []
    for (h, w, fh, fw) in _shapes(case):
        x = torch.rand((h + fh - 1, w + fw - 1), generator=gen, device="cuda", dtype=torch.float32) * 2 - 1
        if case.get("halo"):
            ty, tx = (fh - 1) // 2, (fw - 1) // 2
            ring = torch.zeros_like(x)
            ring[ty:ty + h, tx:tx + w] = x[ty:ty + h, tx:tx + w]
            x = ring
        ins.append(x)
        filts.append(torch.rand((fh, fw), generator=gen, device="cuda", dtype=torch.float32) * 2 - 1)
    return ins, filts


def _chip(rows, cols):
    """Coefficients (cc, gx, gy, gz, t_amb) and a cell's peak power for a
    16 mm silicon chip, 0.5 mm thick, in rows x cols cells, at a quarter of
    the explicit step's stability limit; rounded to FP32 values."""
    side, t, k = 0.016, 0.0005, 100.0
    w, h = side / cols, side / rows
    gx, gy, gz = k * t * h / w, k * t * w / h, k * w * h / t
    cc = 0.25 / (2 * gx + 2 * gy + gz)
    co = [torch.tensor(v, dtype=torch.float32).item() for v in (cc, gx, gy, gz, 318.15)]
    return tuple(co), 3.0e6 * w * h


def _chip_data(case, seed):
    """Temperatures up to 30 K above ambient, powers with few hot cells."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    shape = (case["rows"], case["cols"])
    coeffs, p_max = _chip(*shape)
    temp = coeffs[4] + 30.0 * torch.rand(shape, generator=gen, device="cuda", dtype=torch.float32)
    power = p_max * torch.rand(shape, generator=gen, device="cuda", dtype=torch.float32) ** 2
    return temp, power, coeffs


def prepare(case, seed):
    if case["kind"] == "hotspot":
        temp, power, coeffs = _chip_data(case, seed)
        return dict(kind="hotspot", plan=C.Hotspot(case["rows"], case["cols"]), temp=temp, power=power,
                    steps=case["steps"], coeffs=coeffs, out=torch.empty_like(temp))
    ins, filts = _conv_data(case, seed)
    shapes = _shapes(case)
    outs = [torch.empty((h, w), device="cuda", dtype=torch.float32) for (h, w, _, _) in shapes]
    if case["kind"] == "batch":
        batch = C.Batch(shapes, C.CONV2D_BATCH_BY_SIZE if case["by_size"] else 0)
        state = dict(kind="batch", batch=batch, ins=ins, filts=filts, outs=outs, bound=None)
        if case["bound"]:
            state["bound"] = batch.bind(ins, filts, outs)
        return state
    if case["entry"] == "conv2d":
        return dict(kind="conv2d", inp=ins[0], filt=filts[0])
    return dict(kind="plan", plan=C.Plan(*shapes[0]), inp=ins[0], filt=filts[0], out=outs[0])


def run(state):
    kind = state["kind"]
    if kind == "plan":
        return state["plan"](state["inp"], state["filt"], out=state["out"])
    if kind == "conv2d":
        return C.conv2d(state["inp"], state["filt"])
    if kind == "batch":
        if state["bound"] is not None:
            return list(state["bound"]())
        return list(state["batch"](state["ins"], state["filts"], state["outs"]))
    return state["plan"](state["temp"], state["power"], state["steps"], state["coeffs"], out=state["out"])


def work(case):
    if case["kind"] == "hotspot":
        cells = case["rows"] * case["cols"]
        # two neighbour sums and three fused multiply-adds a cell and step
        return {"bytes": 12 * cells, "flops": 8 * cells * case["steps"]}
    nbytes = flops = 0
    for (h, w, fh, fw) in _shapes(case):
        nbytes += 4 * ((h + fh - 1) * (w + fw - 1) + fh * fw + h * w)
        flops += 2 * h * w * fh * fw
    return {"bytes": nbytes, "flops": flops}


def _exact_conv(x, f):
    x, taps = x.double(), f.double().tolist()
    fh, fw = f.shape
    h, w = x.shape[0] - fh + 1, x.shape[1] - fw + 1
    out = torch.zeros((h, w), device=x.device, dtype=torch.float64)
    for i in range(fh):
        for j in range(fw):
            out.add_(x[i:i + h, j:j + w], alpha=taps[i][j])
    return out


def _exact_hotspot(temp, power, steps, coeffs):
    cc, gx, gy, gz, t_amb = coeffs
    t, p = temp.double(), power.double()
    for _ in range(steps):
        up, down = torch.cat((t[:1], t[:-1])), torch.cat((t[1:], t[-1:]))
        left, right = torch.cat((t[:, :1], t[:, :-1]), 1), torch.cat((t[:, 1:], t[:, -1:]), 1)
        t = t + cc * (p + (up + down - 2 * t) * gy + (left + right - 2 * t) * gx + (t_amb - t) * gz)
    return t


def exact(case, seed):
    if case["kind"] == "hotspot":
        temp, power, coeffs = _chip_data(case, seed)
        return _exact_hotspot(temp, power, case["steps"], coeffs)
    ins, filts = _conv_data(case, seed)
    outs = [_exact_conv(x, f) for x, f in zip(ins, filts)]
    return outs if case["kind"] == "batch" else outs[0]
