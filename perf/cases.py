"""Performance cases of the free-space Poisson solver: the work its users run on one MI355X.

A case is a dict of plain values:

  kind    what one pass does
            solve    phi for one right-hand side on a plan that is kept (``Plan.solve``)
            grad     phi and its gradient in one call (``Plan.solve_grad``)
            batch    many right-hand sides of mixed sizes, one replay of a captured graph (``Batch.launch``)
            refresh  the Green's transform computed again on a kept plan, then a solve
            refit    a new plan for a box fitted to this step's charges, then a solve
  n0,n1,n2  grid points per axis (batch: unused)
  greens    "hockney" or "vico_dct"
  prec      "f32" or "f64"
  tuned     the program called ``autotune`` (batch: also ``autotune_batch``) when it built the plan
  periodic  bit a: axis a is periodic
  e0,e1,e2  box edge lengths
  count     batch: right-hand sides

Sources are sums of eight Gaussian blobs, the test sources of the accuracy
study, with centres, widths and weights drawn from the seed.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2405_02603_amd import Batch, Plan, autotune_batch

SIZES = (8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512)
BATCH_SIZES = (32, 48, 64, 96, 128)  # edge lengths of a mixed batch
DTYPE = {"f32": torch.float32, "f64": torch.float64}


def _case(kind, n=(0, 0, 0), greens="vico_dct", prec="f32", tuned=False, periodic=0, edges=(2.0, 2.0, 2.0), count=0,
          name=None):
    c = {"kind": kind, "n0": n[0], "n1": n[1], "n2": n[2], "greens": greens, "prec": prec, "tuned": tuned,
         "periodic": periodic, "e0": edges[0], "e1": edges[1], "e2": edges[2], "count": count}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest grids, in double precision, on a plan as created: a latency-bound inner solve
        _case("solve", (16, 16, 16), "hockney", "f64", name="solve_16_f64"),
        # a served request: the serving loop uses plans as created, one small solve at a time
        _case("solve", (64, 64, 64), name="solve_64_f32"),
        # a ragged box with three different edges and one periodic axis (a beam pipe, a channel)
        _case("solve", (48, 192, 96), "hockney", "f64", periodic=2, edges=(1.0, 1.5, 1.25), name="solve_48x192x96_f64"),
        # the middle of the range, a plan kept by a time-stepping program
        _case("solve", (128, 128, 128), tuned=True, name="solve_128_f32"),
        # the headline grid, both precisions
        _case("solve", (256, 256, 256), tuned=True, name="solve_256_f32"),
        _case("solve", (256, 256, 256), prec="f64", tuned=True, name="solve_256_f64"),
        # the largest grid
        _case("solve", (512, 512, 512), tuned=True, name="solve_512_f32"),
        # potential and field together, as a particle push needs them
        _case("grad", (256, 256, 256), tuned=True, name="grad_256_f32"),
        # 64 uneven right-hand sides in one captured step
        _case("batch", tuned=True, count=64, name="batch_64_f32"),
        # a particle bunch's box follows the bunch: new plan, new Green's transform, one solve
        _case("refit", (128, 128, 128), name="refit_128_f32"),
        _case("refit", (64, 64, 64), "hockney", "f64", edges=(1.0, 1.25, 1.5), name="refit_64_f64"),
        # the Green's transform of the headline grid refreshed, then used
        _case("refresh", (256, 256, 256), name="refresh_256_f32"),
    ]


def _log_pick(rng, lo, hi):
    return rng.choice([s for s in SIZES if lo <= s <= hi])  # the sizes are spread over their logarithm


def _shape(rng, lo, hi, most):
    """A cube, or three edges within a factor of four of each other, of at most `most` points."""
    while True:
        b = _log_pick(rng, lo, hi)
        n = (b, b, b) if rng.random() < 0.5 else tuple(_log_pick(rng, max(lo, b // 2), min(hi, 2 * b)) for _ in range(3))
        if n[0] * n[1] * n[2] <= most:
            return n


def draw(rng):
    kind = rng.choices(("solve", "grad", "batch", "refresh", "refit"), (55, 12, 10, 10, 13))[0]
    greens = rng.choice(("hockney", "vico_dct"))
    prec = rng.choice(("f32", "f32", "f64"))
    edges = tuple(1.0 + 0.125 * rng.randrange(5) for _ in range(3))
    tuned = rng.random() < 0.5
    cells = 2 ** 26 if prec == "f32" else 2 ** 25
    if kind == "solve":
        periodic = rng.randrange(1, 8) if rng.random() < 0.2 else 0
        return _case(kind, _shape(rng, 8, 512, cells), greens, prec, tuned, periodic, edges)
    if kind == "grad":
        return _case(kind, _shape(rng, 16, 256, cells // 4), greens, prec, tuned, 0, edges)
    if kind == "batch":
        return _case(kind, greens=greens, prec=prec, tuned=tuned, edges=edges, count=rng.randrange(8, 65))
    if kind == "refresh":
        return _case(kind, _shape(rng, 32, 256, cells // 4), greens, prec, tuned, 0, edges)
    return _case(kind, _shape(rng, 16, 128, 2 ** 21), greens, prec, False, 0, edges)


# ---------------------------------------------------------------- inputs
def _sizes(case):
    """Grid edges of a batch's right-hand sides (the mix is part of the case, not of its inputs)."""
    r = random.Random(4 + case["count"])
    return [r.choice(BATCH_SIZES) for _ in range(case["count"])]


def _box(case, seed):
    """The case's box; a refit moves and stretches it with the bunch."""
    e = [case["e0"], case["e1"], case["e2"]]
    lo = [-0.5 * x for x in e]
    if case["kind"] == "refit":
        r = random.Random(7 * seed + 1)
        e = [x * r.uniform(0.95, 1.05) for x in e]
        lo = [-0.5 * x + r.uniform(-0.1, 0.1) for x in e]
    return lo, [a + b for a, b in zip(lo, e)]


def _source(n, lo, hi, seed, dtype):
    """Eight Gaussian blobs of unit mass times a weight, sampled at the cell centres."""
    r = random.Random(seed)
    rho = torch.zeros(n, dtype=torch.float64, device="cuda")
    for _ in range(8):
        w = r.uniform(0.5, 1.5)
        rel = r.uniform(0.02, 0.08)
        s = rel * min(b - a for a, b in zip(lo, hi))
        g = []
        for a in range(3):
            h = (hi[a] - lo[a]) / n[a]
            x = lo[a] + (torch.arange(n[a], dtype=torch.float64, device="cuda") + 0.5) * h
            c = lo[a] + (hi[a] - lo[a]) * r.uniform(0.25, 0.75)
            g.append(torch.exp(-(x - c) ** 2 / (2.0 * s * s)))
        amp = w / ((2.0 * math.pi) ** 1.5 * s ** 3)
        rho += amp * g[0][:, None, None] * g[1][None, :, None] * g[2][None, None, :]
    return rho.to(dtype)


def _problems(case, seed):
    """(n, lo, hi, rho) of every right-hand side of the case."""
    lo, hi = _box(case, seed)
    dtype = DTYPE[case["prec"]]
    if case["kind"] == "batch":
        return [((n, n, n), lo, hi, _source((n, n, n), lo, hi, 1000 * seed + i, dtype))
                for i, n in enumerate(_sizes(case))]
    n = (case["n0"], case["n1"], case["n2"])
    return [(n, lo, hi, _source(n, lo, hi, 1000 * seed, dtype))]


def _plan(case, n, lo, hi, **kw):
    return Plan(n=n, lo=lo, hi=hi, greens=case["greens"], prec=case["prec"], grad=case["kind"] == "grad",
                periodic=tuple(bool(case["periodic"] >> a & 1) for a in range(3)), **kw)


def prepare(case, seed):
    problems = _problems(case, seed)
    n, lo, hi, rho = problems[0]
    if case["kind"] == "refit":
        return {"case": case, "n": n, "lo": lo, "hi": hi, "rho": rho, "phi": torch.empty_like(rho)}
    if case["kind"] == "batch":
        plans, rhos, tuned = [], [], set()
        for n, lo, hi, rho in problems:
            p = _plan(case, n, lo, hi)
            if case["tuned"] and n not in tuned:  # later plans of this grid start with its schedule
                tuned.add(n)
                p.autotune(rho)
            plans.append(p)
            rhos.append(rho)
        if case["tuned"]:
            autotune_batch(plans, rhos)
        return {"case": case, "batch": Batch(plans, rhos)}
    plan = _plan(case, n, lo, hi)
    s = {"case": case, "plan": plan, "rho": rho, "phi": torch.empty_like(rho)}
    if case["tuned"]:
        plan.autotune(rho, s["phi"])
    if case["kind"] == "grad":
        s["grad"] = torch.empty((3,) + n, dtype=rho.dtype, device=rho.device)
    return s


def run(state):
    case = state["case"]
    if case["kind"] == "solve":
        return state["plan"].solve(state["rho"], state["phi"])
    if case["kind"] == "grad":
        grad, phi = state["plan"].solve_grad(state["rho"], state["grad"], state["phi"])
        return {"grad": grad, "phi": phi}
    if case["kind"] == "batch":
        return state["batch"].launch()
    if case["kind"] == "refresh":
        state["plan"].precompute()
        return state["plan"].solve(state["rho"], state["phi"])
    plan = _plan(case, state["n"], state["lo"], state["hi"])
    return plan.solve(state["rho"], state["phi"])


# ---------------------------------------------------------------- least work
def _solve_work(n, rb, outs=1):
    """rho and the real octant of each output's transform read, each output written once; the transforms
    of the doubled grid with the zero half of their inputs and the dropped half of their outputs skipped."""
    n0, n1, n2 = n
    points, octant = n0 * n1 * n2, (n0 + 1) * (n1 + 1) * (n2 + 1)

    def fft(m):  # a length 2m transform of m inputs (or to m outputs): two of length m
        return 2 * 5.0 * m * math.log2(m) + 6.0 * m

    rows, cols1, cols0 = n0 * n1 * fft(n2) / 2, n0 * (n2 + 1) * fft(n1), 2 * n1 * (n2 + 1) * fft(n0)
    flops = rows + cols1 + cols0 + outs * (rows + cols1 + cols0 + 4 * n0 * n1 * (n2 + 1) * 2)
    return (points + outs * (octant + points)) * rb, flops


def _green_work(case, n, rb):
    """The octant written once; the samples of the kernel and the cosine transforms by a fast algorithm."""
    m = [(x + 1) for x in n]
    octant = m[0] * m[1] * m[2]
    flops = octant * (12.0 + 2.5 * sum(math.log2(2 * x) for x in n))
    if case["greens"] == "vico_dct":
        w = [2 * x + 1 for x in n]
        flops += 30.0 * w[0] * w[1] * w[2]
        flops += 2.5 * (w[0] * math.log2(4 * n[0]) * w[1] * w[2] + m[0] * w[1] * math.log2(4 * n[1]) * w[2]
                        + m[0] * m[1] * w[2] * math.log2(4 * n[2]))
    return octant * rb, flops


def work(case):
    rb = 4 if case["prec"] == "f32" else 8
    if case["kind"] == "batch":
        parts = [_solve_work((n, n, n), rb) for n in _sizes(case)]
    else:
        n = (case["n0"], case["n1"], case["n2"])
        parts = [_solve_work(n, rb, 4 if case["kind"] == "grad" else 1)]
        if case["kind"] in ("refresh", "refit"):
            parts.append(_green_work(case, n, rb))
    return {"bytes": int(sum(p[0] for p in parts)), "flops": int(sum(p[1] for p in parts))}


# ---------------------------------------------------------------- the same in 64 bits
def _along(c, x, a):
    return torch.movedim(torch.tensordot(c, x, dims=([1], [a])), 0, a).contiguous()


def _axis(n):
    return torch.arange(n, dtype=torch.float64, device="cuda")


def _kernels(case, n, lo, hi):
    """The kernel on the offsets m in [0, n], and for a gradient its three derivatives."""
    h = [(b - a) / m for a, b, m in zip(lo, hi, n)]
    parts = [None] + ([0, 1, 2] if case["kind"] == "grad" else [])
    if case["greens"] == "hockney":
        x = [_axis(n[a] + 1) * h[a] for a in range(3)]
        x = [x[0][:, None, None], x[1][None, :, None], x[2][None, None, :]]
        r = torch.sqrt(x[0] ** 2 + x[1] ** 2 + x[2] ** 2)
        out = []
        for d in parts:
            k = 1.0 / (4.0 * math.pi * r) if d is None else -x[d] / (4.0 * math.pi * r ** 3)
            k[0, 0, 0] = 1.0 / (4.0 * math.pi) if d is None else 0.0
            out.append(k)
        return out
    k = [_axis(2 * n[a] + 1) * (math.pi / (2 * n[a] * h[a])) for a in range(3)]
    kk = torch.sqrt(k[0][:, None, None] ** 2 + k[1][None, :, None] ** 2 + k[2][None, None, :] ** 2)
    length = 1.1 * math.sqrt(sum((b - a) ** 2 for a, b in zip(lo, hi)))
    g = 2.0 * (torch.sin(0.5 * length * kk) / kk) ** 2
    g[0, 0, 0] = 0.5 * length * length
    del kk
    out = []
    for d in parts:
        t = g
        for a in range(3):
            w = torch.full((2 * n[a] + 1,), 2.0, dtype=torch.float64, device="cuda")
            w[0] = w[-1] = 1.0
            turn = torch.outer(_axis(n[a] + 1), _axis(2 * n[a] + 1)) % (4 * n[a]) * (math.pi / (2 * n[a]))
            c = w * torch.cos(turn) if a != d else -w * k[a] * torch.sin(turn)
            t = _along(c, t, a)
        out.append(t / (64.0 * n[0] * n[1] * n[2] * h[0] * h[1] * h[2]))
    return out


def _convolve(case, n, lo, hi, rho):
    """V sum_j K[|i - j|] rho_j for the potential's kernel and each derivative's, on the doubled grid."""
    v = math.prod((b - a) / m for a, b, m in zip(lo, hi, n))

    def forward(t):
        t = torch.fft.rfft(t, n=2 * n[2], dim=2)
        t = torch.fft.fft(t, n=2 * n[1], dim=1)
        return torch.fft.fft(t, n=2 * n[0], dim=0)

    kernels = _kernels(case, n, lo, hi)
    spectrum, out = forward(rho.double()), []
    for d, k in enumerate(kernels):
        for a in range(3):
            if case["periodic"] >> a & 1:  # the nearest image's value
                m = torch.arange(n[a] + 1, device="cuda")
                k = k.index_select(a, torch.minimum(m, n[a] - m))
            mirror = k.narrow(a, 1, n[a] - 1).flip(a)
            if d == a + 1:
                k = k.clone()
                k.narrow(a, n[a], 1).zero_()
                mirror = -mirror
            k = torch.cat([k, mirror], dim=a)
        s = forward(k)
        del k
        s *= spectrum
        s = torch.fft.ifft(s, dim=0)[: n[0]]
        s = torch.fft.ifft(s, dim=1)[:, : n[1]]
        out.append(torch.fft.irfft(s, n=2 * n[2], dim=2)[:, :, : n[2]] * v)
        del s
    return out


def exact(case, seed):
    values = [_convolve(case, *p) for p in _problems(case, seed)]
    if case["kind"] == "batch":
        return [x[0] for x in values]
    if case["kind"] == "grad":
        return {"grad": torch.stack(values[0][1:]), "phi": values[0][0]}
    return values[0][0]
