"""The work that users of this library have it do, as measurable cases.

Each case is one call (or one call and its residual) through the Python
binding: a Jacobi or leapfrog run of some sweeps, a batch of grids, or one
pass of a generated program.  listed() holds the fixed ones, draw() more of
the same ranges; prepare() makes what a program holds before the call (inputs
on the GPU, the plan), run() is the call, work() what it cannot do without and
exact() the same outputs from plain torch in 64 bits.
"""
import math

import numpy as np
import torch

from paper_2306_13002_amd import saturator, synth
from paper_2306_13002_amd.stencil import BatchPlan, Plan

DEV = "cuda"
WAVE_COEF = (-2.847222, 1.6, -0.2, 0.025397, -0.001786)
OMEGA = 0.8


def listed():
    return [
        # the latency case: ten 2-D sweeps of a small plate and the convergence
        # check after them, the plan's defaults
        {"name": "heat2d5_256", "op": "heat2d5", "nx": 256, "ny": 256, "T": 10},
        # the same solver on a plate of ordinary size, ragged edges
        {"name": "heat2d5_2000", "op": "heat2d5", "nx": 1999, "ny": 1501, "T": 10},
        # a small 3-D solve: a few sweeps and the convergence check, the plan's defaults
        {"name": "heat3d7_small", "op": "heat3d7", "nx": 61, "ny": 48, "nz": 53, "T": 10, "variant": "auto"},
        # one mid-sized 3-D solve of many sweeps in the multi-sweep form
        {"name": "heat3d7_160_t3", "op": "heat3d7", "nx": 160, "ny": 160, "nz": 160, "T": 50,
         "variant": "saturated_t3"},
        # a grid that streams from HBM, one sweep per pass (the defaults)
        {"name": "heat3d7_400", "op": "heat3d7", "nx": 400, "ny": 400, "nz": 400, "T": 6, "variant": "auto"},
        # serving: 64 grids of uneven edges (32 to 160) advanced together
        {"name": "batch_64", "op": "batch", "count": 64, "lo": 32, "hi": 160, "T": 50, "variant": "saturated_t3"},
        # the pressure relaxation on its usual grid, two sweeps per pass
        {"name": "poisson19_129", "op": "poisson19", "nx": 127, "ny": 127, "nz": 255, "T": 20,
         "variant": "saturated_t2"},
        # the large one: ten leapfrog steps of a 512^3 wave field
        {"name": "wave25_512", "op": "wave25", "nx": 512, "ny": 512, "nz": 512, "T": 10},
        # a user's own stencil, bounded by arithmetic: FP64 box of radius 3, symmetric coefficients
        {"name": "generic_box3_f64", "op": "generic", "nx": 256, "ny": 256, "nz": 256, "T": 4, "radius": 3,
         "shape": "box", "sharing": "symmetric", "dtype": "f64"},
        # ... F32 storage, a long star with mirrored coefficients, ragged edges
        {"name": "generic_star4_f32", "op": "generic", "nx": 321, "ny": 190, "nz": 257, "T": 4, "radius": 4,
         "shape": "star", "sharing": "reflection", "dtype": "f32"},
        # ... F32 storage, a box whose 125 coefficients all differ
        {"name": "generic_box2_f32", "op": "generic", "nx": 201, "ny": 233, "nz": 160, "T": 4, "radius": 2,
         "shape": "box", "sharing": "distinct", "dtype": "f32"},
        # the rewritten many-statement loop body: 50 arrays in, 75 out
        {"name": "program_162", "op": "program", "nx": 162, "ny": 162, "nz": 162, "tx": 256, "ty": 2},
    ]


def _edge(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["heat2d5", "heat3d7", "heat3d7", "batch", "poisson19", "wave25", "generic", "generic", "program"])
    if op == "heat2d5":
        return {"op": op, "nx": _edge(rng, 64, 3000), "ny": _edge(rng, 64, 3000), "T": rng.randint(2, 16)}
    if op == "heat3d7":
        return {"op": op, "nx": _edge(rng, 24, 400), "ny": _edge(rng, 24, 400), "nz": _edge(rng, 24, 400),
                "T": rng.randint(2, 16), "variant": rng.choice(["auto", "saturated_t2", "saturated_t3"])}
    if op == "batch":
        lo = rng.randint(24, 64)
        return {"op": op, "count": rng.randint(6, 48), "lo": lo, "hi": rng.randint(lo + 8, 160),
                "T": rng.randint(6, 40), "variant": rng.choice(["auto", "saturated_t2", "saturated_t3"])}
    if op == "poisson19":
        return {"op": op, "nx": _edge(rng, 31, 255), "ny": _edge(rng, 31, 255), "nz": _edge(rng, 31, 255),
                "T": rng.randint(2, 20), "variant": rng.choice(["auto", "saturated_t2"])}
    if op == "wave25":
        return {"op": op, "nx": _edge(rng, 48, 448), "ny": _edge(rng, 48, 448), "nz": _edge(rng, 48, 448),
                "T": rng.randint(2, 8)}
    if op == "program":
        return {"op": op, "nx": _edge(rng, 32, 160), "ny": _edge(rng, 32, 160), "nz": _edge(rng, 32, 160),
                "tx": rng.choice([64, 128, 256]), "ty": 2}
    box = rng.random() < 0.5
    return {"op": "generic", "nx": _edge(rng, 64, 288), "ny": _edge(rng, 64, 288), "nz": _edge(rng, 64, 288),
            "T": rng.randint(1, 4), "radius": rng.randint(1, 3 if box else 4), "shape": "box" if box else "star",
            "sharing": rng.choice(["distinct", "reflection", "symmetric", "partition"]),
            "dtype": rng.choice(["f32", "f64"])}


# ------------------------------------------------------------------ inputs
def _n(c):
    return (c["nx"], c["ny"]) if c["op"] == "heat2d5" else (c["nx"], c["ny"], c["nz"])


def _rand(gen, shape, dtype=torch.float64):
    return torch.rand(shape, dtype=dtype, generator=gen, device=DEV)


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _inner(u, r):
    return u[tuple(slice(r, s - r) for s in u.shape)]


def _heat_grid(gen, n):
    """U[0,1) inside a fixed 0 ring."""
    u = torch.zeros([e + 2 for e in reversed(n)], dtype=torch.float64, device=DEV)
    _inner(u, 1).copy_(_rand(gen, [e for e in reversed(n)]))
    return u


def _batch_sizes(c):
    """The sizes a batch has, fixed by the case (a server's mix of grids)."""
    rng = np.random.RandomState(1000 + c["count"])
    return [tuple(int(v) for v in rng.randint(c["lo"], c["hi"] + 1, 3)) for _ in range(c["count"])]


def _slab(sizes):
    """Offsets of the padded grids in one allocation (each 512-byte aligned)
    and its length in doubles."""
    at, off = 0, []
    for n in sizes:
        off.append(at)
        at += -(-math.prod(e + 2 for e in n) // 64) * 64
    return off, at


def _views(slab, sizes, off):
    return [slab[o:o + math.prod(e + 2 for e in n)].view([e + 2 for e in reversed(n)]) for n, o in zip(sizes, off)]


def _batch_grids(c, seed):
    sizes = _batch_sizes(c)
    off, total = _slab(sizes)
    slab = torch.zeros(total, dtype=torch.float64, device=DEV)
    gen = _gen(seed)
    for u, n in zip(_views(slab, sizes, off), sizes):
        _inner(u, 1).copy_(_rand(gen, [e for e in reversed(n)]))
    return sizes, off, slab


def _poisson_grids(c, seed):
    """A pressure field near its quadratic profile, variable coefficients
    whose rows sum to at most one (the relaxation converges), a few solid
    cells (bnd = 0) and a small source; order a0 a1 a2 a3 b0 b1 b2 c0 c1 c2
    bnd wrk1."""
    shape = [e + 2 for e in reversed(_n(c))]
    gen = _gen(seed)
    f32 = torch.float32
    k = torch.arange(shape[0], dtype=f32, device=DEV) / (shape[0] - 1)
    p = (k * k)[:, None, None] + 0.01 * _rand(gen, shape, f32)
    face = lambda: 0.9 + 0.09 * _rand(gen, shape, f32)  # noqa: E731
    edge = lambda: 0.01 * _rand(gen, shape, f32) - 0.005  # noqa: E731
    a = [face() for _ in range(3)] + [torch.full(shape, 1.0 / 6.0, dtype=f32, device=DEV)]
    b = [edge() for _ in range(3)]
    cc = [face() for _ in range(3)]
    bnd = (_rand(gen, shape, f32) < 0.95).to(f32)
    wrk1 = 0.02 * _rand(gen, shape, f32) - 0.01
    return p, a + b + cc + [bnd, wrk1]


def _wave_grids(c, seed):
    shape = [e + 8 for e in reversed(_n(c))]
    gen = _gen(seed)
    vsq = ((1.5 + 3.0 * _rand(gen, shape)) * (0.4 / 4.5)) ** 2
    u = 1.0 + 0.1 * _rand(gen, shape)
    return u, vsq


def _taps(c):
    r = c["radius"]
    if c["shape"] == "box":
        return [(x, y, z) for z in range(-r, r + 1) for y in range(-r, r + 1) for x in range(-r, r + 1)]
    taps = [(0, 0, 0)]
    for ax in range(3):
        for q in range(1, r + 1):
            for s in (q, -q):
                taps.append(tuple(s if a == ax else 0 for a in range(3)))
    return taps


def _coefs(c, taps):
    """(coefficient id per tap, coefficients): the stencil is the case's, not
    the seed's; positive weights that sum to one over the taps."""
    rng = np.random.RandomState(77)
    if c["sharing"] == "distinct":
        ids = list(range(len(taps)))
    elif c["sharing"] == "partition":
        draws = rng.randint(0, max(2, len(taps) // 3), len(taps))
        ids = list(np.unique(draws, return_inverse=True)[1])
    else:
        keys = {}
        ids = []
        for d in taps:
            key = max(d, tuple(-v for v in d)) if c["sharing"] == "reflection" else tuple(sorted(abs(v) for v in d))
            ids.append(keys.setdefault(key, len(keys)))
    ids = [int(i) for i in ids]
    vals = 0.1 + 0.9 * rng.random_sample(max(ids) + 1)
    return ids, [float(v) for v in vals / vals[ids].sum()]


def _generic_grid(c, seed):
    r = c["radius"]
    return _rand(_gen(seed), [e + 2 * r for e in reversed(_n(c))],
                 torch.float32 if c["dtype"] == "f32" else torch.float64)


def _program_inputs(c, seed):
    """50 grids: F = 1 + U[0,1) (0..24), N = U[0,1) (25..49)."""
    ins = _rand(_gen(seed), [50] + [e + 2 for e in reversed(_n(c))])
    ins[:25] += 1.0
    return ins


# ------------------------------------------------------------------ the call
def prepare(case, seed):
    c, op, n = case, case["op"], (None if case["op"] == "batch" else _n(case))
    if op in ("heat2d5", "heat3d7"):
        coef = (0.6, 0.1) if op == "heat2d5" else (0.4, 0.1)
        u = _heat_grid(_gen(seed), n)
        plan = Plan(op, n, variant=c.get("variant", "auto"), coef=coef)
        return {"op": op, "T": c["T"], "plan": plan, "fields": [u, torch.empty_like(u)], "coefs": None}
    if op == "batch":
        sizes, off, slab = _batch_grids(c, seed)
        scratch = torch.empty_like(slab)
        plan = BatchPlan(sizes, coef=(0.4, 0.1), variant=c["variant"])
        fields = list(zip(_views(slab, sizes, off), _views(scratch, sizes, off)))
        return {"op": op, "T": c["T"], "plan": plan, "fields": fields, "slab": slab, "scratch": scratch}
    if op == "poisson19":
        p, coefs = _poisson_grids(c, seed)
        plan = Plan(op, n, variant=c["variant"], omega=OMEGA)
        return {"op": op, "T": c["T"], "plan": plan, "fields": [p, torch.empty_like(p)], "coefs": coefs}
    if op == "wave25":
        u, vsq = _wave_grids(c, seed)
        plan = Plan(op, n, coef=WAVE_COEF)
        return {"op": op, "T": c["T"], "plan": plan, "fields": [u, u.clone()], "coefs": [vsq]}
    if op == "generic":
        taps = _taps(c)
        ids, coef = _coefs(c, taps)
        u = _generic_grid(c, seed)
        plan = Plan(op, n, dtype=c["dtype"], radius=c["radius"], taps=taps, cids=ids, coef=coef)
        return {"op": op, "T": c["T"], "plan": plan, "fields": [u, torch.empty_like(u)], "coefs": None}
    ins = _program_inputs(c, seed)
    out = torch.zeros([75] + list(ins.shape[1:]), dtype=torch.float64, device=DEV)
    plan = saturator.ProgramPlan(synth.lhs_program(), n, "accsat", tile=(c["tx"], c["ty"]))
    return {"op": op, "plan": plan, "in": list(ins.unbind(0)), "out": list(out.unbind(0)), "out_slab": out}


def run(s):
    op = s["op"]
    if op == "program":
        s["plan"].run(s["in"], s["out"], synth.LHS_PARAMS)
        return s["out_slab"]
    if op == "batch":
        s["plan"].run(s["fields"], iterations=s["T"])
        return {"u": s["slab"], "residuals": np.array(s["plan"].residuals())}
    if op == "wave25":  # time stepping: the next call goes on from the two newest levels
        s["fields"] = list(s["plan"].run(s["fields"], s["coefs"], iterations=s["T"]))
        return {"older": s["fields"][0], "newer": s["fields"][1]}
    u = s["plan"].run(s["fields"], s["coefs"], iterations=s["T"])
    if op == "generic":
        return u
    return {"u": u, "residual": s["plan"].residual()}  # iterative solvers look at it after every call


def work(case):
    """Inputs once and outputs once per call; operations of every sweep."""
    c, op = case, case["op"]
    if op == "batch":
        pts = sum(math.prod(n) for n in _batch_sizes(c))
        return {"bytes": 16 * pts, "flops": 9 * pts * c["T"]}
    pts = math.prod(_n(c))
    if op == "heat2d5":
        return {"bytes": 16 * pts, "flops": 9 * pts * c["T"]}
    if op == "heat3d7":
        return {"bytes": 16 * pts, "flops": 9 * pts * c["T"]}
    if op == "poisson19":
        return {"bytes": 56 * pts, "flops": 34 * pts * c["T"]}
    if op == "wave25":
        return {"bytes": 40 * pts, "flops": 35 * pts * c["T"]}
    if op == "generic":
        taps = _taps(c)
        return {"bytes": (8 if c["dtype"] == "f32" else 16) * pts,
                "flops": (len(taps) + max(_coefs(c, taps)[0]) + 1) * pts * c["T"]}
    return {"bytes": 8 * 125 * pts, "flops": 215 * pts}


# ------------------------------------------------------------------ 64 bits
def _shift(u, r, dx=0, dy=0, dz=0):
    """The interior of u seen from an offset."""
    off = (dy, dx) if u.dim() == 2 else (dz, dy, dx)
    return u[tuple(slice(r + o, s - r + o) for o, s in zip(off, u.shape))]


def _heat_exact(u, cc, cn, T):
    for _ in range(T):
        s = _shift(u, 1, -1) + _shift(u, 1, 1) + _shift(u, 1, 0, -1) + _shift(u, 1, 0, 1)
        if u.dim() == 3:
            s += _shift(u, 1, 0, 0, -1) + _shift(u, 1, 0, 0, 1)
        v = u.clone()
        _inner(v, 1).copy_(cc * _inner(u, 1) + cn * s)
        last, u = u, v
    return u, float(((u - last) ** 2).sum())


def _poisson_exact(p, coefs, T):
    p = p.double()
    f = [_inner(x, 1).double() for x in coefs]
    S = lambda dx, dy, dz: _shift(p, 1, dx, dy, dz)  # noqa: E731
    for _ in range(T):
        s0 = f[0] * S(1, 0, 0) + f[1] * S(0, 1, 0) + f[2] * S(0, 0, 1)
        s0 += f[4] * (S(1, 1, 0) - S(1, -1, 0) - S(-1, 1, 0) + S(-1, -1, 0))
        s0 += f[5] * (S(0, 1, 1) - S(0, -1, 1) - S(0, 1, -1) + S(0, -1, -1))
        s0 += f[6] * (S(1, 0, 1) - S(-1, 0, 1) - S(1, 0, -1) + S(-1, 0, -1))
        s0 += f[7] * S(-1, 0, 0) + f[8] * S(0, -1, 0) + f[9] * S(0, 0, -1) + f[11]
        ss = (s0 * f[3] - _inner(p, 1)) * f[10]
        q = p.clone()
        _inner(q, 1).add_(OMEGA * ss)
        p = q
    return p, float((ss * ss).sum())


def _wave_exact(u, vsq, T):
    old, new = u, u.clone()
    v = _inner(vsq, 4)
    old = old.clone()
    for _ in range(T):
        L = 3.0 * WAVE_COEF[0] * _inner(new, 4)
        for q in range(1, 5):
            L += WAVE_COEF[q] * (_shift(new, 4, q) + _shift(new, 4, -q) + _shift(new, 4, 0, q) +
                                 _shift(new, 4, 0, -q) + _shift(new, 4, 0, 0, q) + _shift(new, 4, 0, 0, -q))
        _inner(old, 4).copy_(2.0 * _inner(new, 4) - _inner(old, 4) + v * L)
        old, new = new, old
    return {"older": old, "newer": new}


def _generic_exact(u, c):
    taps, r = _taps(c), c["radius"]
    ids, coef = _coefs(c, taps)
    u = u.double()
    for _ in range(c["T"]):
        s = torch.zeros_like(_inner(u, r))
        for d, i in zip(taps, ids):
            s.add_(_shift(u, r, *d), alpha=coef[i])
        u = u.clone()
        _inner(u, r).copy_(s)
    return u


def _program_exact(ins, out):
    dt, tz1, tz2 = synth.LHS_PARAMS[:3]
    dz = synth.LHS_PARAMS[3:]
    t1, t2 = dt * tz1, dt * tz2
    for m in range(5):
        for n in range(5):
            F, N, e = ins[5 * m + n], ins[25 + 5 * m + n], 5 * m + n
            d = t1 * dz[m] if m == n else 0.0
            _inner(out[e], 1).copy_(-t2 * _shift(F, 1, 0, 0, -1) - t1 * _shift(N, 1, 0, 0, -1) - d)
            _inner(out[25 + e], 1).copy_(2.0 * t1 * _inner(N, 1) + (1.0 + 2.0 * d if m == n else 0.0))
            _inner(out[50 + e], 1).copy_(t2 * _shift(F, 1, 0, 0, 1) - t1 * _shift(N, 1, 0, 0, 1) - d)
    return out


def exact(case, seed):
    c, op = case, case["op"]
    if op in ("heat2d5", "heat3d7"):
        u, res = _heat_exact(_heat_grid(_gen(seed), _n(c)), 0.6 if op == "heat2d5" else 0.4, 0.1, c["T"])
        return {"u": u, "residual": res}
    if op == "batch":
        sizes, off, slab = _batch_grids(c, seed)
        res = []
        for u in _views(slab, sizes, off):
            v, r = _heat_exact(u, 0.4, 0.1, c["T"])
            u.copy_(v)
            res.append(r)
        return {"u": slab, "residuals": np.array(res)}
    if op == "poisson19":
        p, res = _poisson_exact(*_poisson_grids(c, seed), c["T"])
        return {"u": p, "residual": res}
    if op == "wave25":
        return _wave_exact(*_wave_grids(c, seed), c["T"])
    if op == "generic":
        return _generic_exact(_generic_grid(c, seed), c)
    ins = _program_inputs(c, seed)
    return _program_exact(ins, torch.zeros([75] + list(ins.shape[1:]), dtype=torch.float64, device=DEV))
