"""The transforms that programs ask of this library, as cases to be timed.

A case is a dict of plain values: the operation ("fft", "ifft", "roundtrip",
"convolve" or "batch"), the grid, the schedule, the leaf precision and how
the program calls the library ("fftn": the module's functions, which allocate
the result; "plan": a kept Plan and kept buffers).  prepare() makes what the
program has before the call, run() is one pass through the public entry
points, exact() the same result in 64 bits from plain matrix products.
"""
import math

import torch

from paper_1904_10119_amd import dft3d

DEVICE = "cuda"


def _case(name, op, shape, schedule="auto", precision="fp32", call="fftn", values="uniform"):
    return {"name": name, "op": op, "n0": shape[0], "n1": shape[1], "n2": shape[2],
            "schedule": schedule, "precision": precision, "call": call, "values": values}


def _batch(name, count, sides, seed):
    return {"name": name, "op": "batch", "count": count, "sides": sides, "shape_seed": seed}


def listed():
    return [
        # a small grid called again and again (a time step, a local solve):
        # launches and host work are what it costs
        _case("cube32", "fft", (32, 32, 32)),
        # forward and back on kept buffers, as a spectral solver does each step
        _case("roundtrip64", "roundtrip", (64, 64, 64), call="plan"),
        # the usual plane-wave grid, with a factor 3
        _case("grid96", "fft", (96, 96, 96)),
        # whatever sides the data came with: a prime, an odd and an even one
        _case("ragged61x75x90", "ifft", (61, 75, 90)),
        # many uneven problems in one call (k-points, patches)
        _batch("batch96", 96, "32,64,128", 104),
        # one middle-sized volume, with a spectrum of a few strong lines
        _case("cube256", "fft", (256, 256, 256), values="waves"),
        # the same on the matrix cores with FP32 accuracy
        _case("cube256_bf16x6", "fft", (256, 256, 256), schedule="pencil", precision="bf16x6",
              call="plan", values="waves"),
        # a filter whose spectrum is kept, applied in the shuffled order
        _case("convolve256", "convolve", (256, 256, 256)),
        # a scanned volume: three uneven sides with small prime factors
        _case("ragged375x486x400", "fft", (375, 486, 400)),
        # uneven sides that are primes
        _case("primes257x251x263", "fft", (257, 251, 263)),
        # the largest decimal cube, back from the spectrum
        _case("cube1000", "ifft", (1000, 1000, 1000), call="plan"),
        # the largest cube of a power of two
        _case("cube1024", "fft", (1024, 1024, 1024), call="plan"),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _smooth(n):
    for f in (2, 3, 5, 7, 11, 13):
        while n % f == 0:
            n //= f
    return n == 1


def _sides(rng, points, lo, hi, ok):
    """Three sides in [lo, hi] that pass ok(), of about `points` in all."""
    while True:
        a = _log_uniform(rng, lo, hi)
        b = _log_uniform(rng, lo, hi)
        c = points / (a * b)
        if not lo <= c <= hi:
            continue
        sides = []
        for v in rng.sample((a, b, c), 3):
            n = max(lo, min(hi, round(v)))
            while not ok(n):
                n -= 1
            sides.append(n)
        return tuple(sides)


def _pow2_sides(rng, points, lo, hi):
    e = round(math.log2(points))
    a, b = int(math.log2(lo)), int(math.log2(hi))
    while True:
        x, y = rng.randint(a, b), rng.randint(a, b)
        if a <= e - x - y <= b:
            return (1 << x, 1 << y, 1 << (e - x - y))


def draw(rng):
    kind = rng.choice(("pow2", "pow2", "smooth", "smooth", "any", "split", "batch", "convolve"))
    op = rng.choice(("fft", "fft", "ifft", "roundtrip"))
    call = rng.choice(("fftn", "plan"))
    if kind == "batch":
        case = _batch("", rng.randint(8, 96), rng.choice(("32,64,128", "16,32,64")),
                      rng.randint(0, 999999))
    elif kind == "convolve":
        case = _case("", "convolve", _pow2_sides(rng, _log_uniform(rng, 1 << 15, 1 << 27), 16, 1024))
    elif kind == "split":
        case = _case("", op, _pow2_sides(rng, _log_uniform(rng, 1 << 15, 1 << 28), 16, 2048),
                     schedule="pencil", precision=rng.choice(("bf16x6", "bf16x9", "fp16x3")),
                     call=call, values="waves")
    elif kind == "pow2":
        case = _case("", op, _pow2_sides(rng, _log_uniform(rng, 1 << 13, 1 << 28), 16, 2048),
                     schedule=rng.choice(("auto", "auto", "auto", "slab", "pencil")), call=call,
                     values=rng.choice(("uniform", "waves")))
    elif kind == "smooth":
        case = _case("", op, _sides(rng, _log_uniform(rng, 1 << 14, 1 << 28), 18, 1100, _smooth),
                     call=call)
    else:
        case = _case("", op, _sides(rng, _log_uniform(rng, 1 << 14, 1 << 25), 18, 700,
                                    lambda n: True), call=call)
    del case["name"]
    return case


# ---- inputs ----------------------------------------------------------------

def _shape(case):
    return (case["n0"], case["n1"], case["n2"])


def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed))
    return g


def _uniform(shape, g):
    """Real and imaginary parts iid uniform on [-1, 1)."""
    x = torch.empty(*shape, 2, dtype=torch.float32, device=DEVICE)
    x.uniform_(-1.0, 1.0, generator=g)
    return torch.view_as_complex(x)


def _waves(shape, g):
    """Normal noise and eight plane waves of unit amplitude."""
    x = torch.empty(*shape, 2, dtype=torch.float32, device=DEVICE)
    x.normal_(0.0, 1.0, generator=g)
    x = torch.view_as_complex(x)
    picks = torch.rand(8, 4, generator=g, device=DEVICE).cpu().tolist()
    for u in picks:
        line = [torch.polar(torch.ones(n, dtype=torch.float64, device=DEVICE),
                            torch.arange(n, dtype=torch.float64, device=DEVICE)
                            * (2 * math.pi * int(v * n) / n)).to(torch.complex64)
                for n, v in zip(shape, u)]
        first = line[0] * complex(math.cos(2 * math.pi * u[3]), math.sin(2 * math.pi * u[3]))
        x += (first[:, None, None] * line[1][None, :, None]) * line[2][None, None, :]
    return x


def _values(case, seed):
    g = _generator(seed)
    return (_waves if case["values"] == "waves" else _uniform)(_shape(case), g)


def _batch_shapes(case):
    g = torch.Generator()
    g.manual_seed(case["shape_seed"])
    sides = [int(s) for s in case["sides"].split(",")]
    pick = torch.randint(len(sides), (case["count"], 3), generator=g).tolist()
    return [tuple(sides[i] for i in p) for p in pick]


def _batch_views(flat, shapes):
    views, at = [], 0
    for s in shapes:
        n = s[0] * s[1] * s[2]
        views.append(flat[at:at + n].view(s))
        at += n
    return views


def _batch_values(case, seed):
    shapes = _batch_shapes(case)
    total = sum(a * b * c for a, b, c in shapes)
    return shapes, _uniform((total,), _generator(seed))


def _filter(case, seed):
    """The filter's values: noise scaled so that filtered data keep their size."""
    n = case["n0"] * case["n1"] * case["n2"]
    return _uniform(_shape(case), _generator(seed + 7919)) / (n * math.sqrt(n))


def prepare(case, seed):
    if case["op"] == "batch":
        shapes, flat = _batch_values(case, seed)
        out = torch.empty_like(flat)
        return {"op": "batch", "xs": _batch_views(flat, shapes), "out": out,
                "outs": _batch_views(out, shapes)}
    state = {"op": case["op"], "x": _values(case, seed), "call": case["call"],
             "schedule": case["schedule"], "precision": case["precision"]}
    if case["op"] == "convolve":
        state["spectrum"] = dft3d.fftn(_filter(case, seed), schedule="volumetric",
                                       layout="shuffled")
    elif case["call"] == "plan":
        state["plan"] = dft3d.Plan(_shape(case), case["schedule"], precision=case["precision"])
        state["plan"].bind_workspace(state["x"].device)
        state["y"] = torch.empty_like(state["x"])
        if case["op"] == "roundtrip":
            state["z"] = torch.empty_like(state["x"])
    return state


def run(state):
    op = state["op"]
    if op == "batch":
        dft3d.fftn_batched(state["xs"], outs=state["outs"])
        return state["out"]
    if op == "convolve":
        y = dft3d.fftn(state["x"], schedule="volumetric", layout="shuffled")
        y *= state["spectrum"]
        return dft3d.ifftn(y, schedule="volumetric", layout="shuffled")
    if state["call"] == "plan":
        plan, x, y = state["plan"], state["x"], state["y"]
        plan.execute(x, y, inverse=op == "ifft")
        if op == "roundtrip":
            plan.execute(y, state["z"], inverse=True)
            return y, state["z"]
        return y
    how = {"schedule": state["schedule"], "precision": state["precision"]}
    if op == "ifft":
        return dft3d.ifftn(state["x"], **how)
    y = dft3d.fftn(state["x"], **how)
    if op == "roundtrip":
        return y, dft3d.ifftn(y, **how)
    return y


# ---- what a pass cannot do without -----------------------------------------

def work(case):
    shapes = _batch_shapes(case) if case["op"] == "batch" else [_shape(case)]
    points = [a * b * c for a, b, c in shapes]
    flops = sum(5.0 * n * math.log2(n) for n in points)
    total = 16.0 * sum(points)
    if case["op"] == "roundtrip":  # the input, the spectrum written, the result
        return {"bytes": total * 1.5, "flops": flops * 2}
    if case["op"] == "convolve":  # the input, the kept spectrum, the result
        return {"bytes": total * 1.5, "flops": flops * 2 + 6.0 * points[0]}
    return {"bytes": total, "flops": flops}


# ---- the same in 64 bits ---------------------------------------------------

def _dft_matrix(n, sign):
    j = torch.arange(n, dtype=torch.int64, device=DEVICE)
    angle = (j[:, None] * j[None, :] % n).to(torch.float64) * (sign * 2 * math.pi / n)
    return torch.polar(torch.ones_like(angle), angle)


def _dft(x, sign):
    """The unscaled 3D DFT of x (any complex type) in complex128: one matrix
    product along the last axis, which then becomes the first, three times."""
    for _ in range(3):
        n0, n1, n2 = x.shape
        rows = x.reshape(n0 * n1, n2)
        matrix = _dft_matrix(n2, sign)
        turned = torch.empty(n2, n0 * n1, dtype=torch.complex128, device=DEVICE)
        step = max(1, (1 << 27) // n2)
        for i in range(0, n0 * n1, step):
            turned[:, i:i + step] = (rows[i:i + step].to(torch.complex128) @ matrix).t()
        x = turned.view(n2, n0, n1)
        del rows, turned
    return x


def exact(case, seed):
    if case["op"] == "batch":
        shapes, flat = _batch_values(case, seed)
        return torch.cat([_dft(v, -1).reshape(-1) for v in _batch_views(flat, shapes)])
    x = _values(case, seed)
    if case["op"] == "convolve":
        return _dft(_dft(x, -1) * _dft(_filter(case, seed), -1), 1)
    if case["op"] == "ifft":
        return _dft(x, 1)
    y = _dft(x, -1)
    if case["op"] == "roundtrip":  # back exactly: the input times the points
        return y, x.to(torch.complex128) * (x.numel())
    return y
