"""Timed workloads of the framework, through its public Python entry points.

Sizes, orders, leaf sizes and distributions are those of the benchmark, the
serving trace and the tests: N from 10^3 to 2^22, p = 3 (treecodes) and 6 to 12
(FMM), leaves of at most 32 or 64 particles, the uniform cube and the Plummer
sphere, equal, unequal and mixed-sign masses.  A pass goes from FP64 inputs in
device memory to outputs in device memory, allocations included, as a program
that calls the library with its default arguments has it.

Kinds of work:
  solve     one evaluation of new particles (tree, upward, evaluation)
  resident  new masses on a kept tree, evaluated at separate points
  leapfrog  steps of the N-body simulation with a kept tree
  direct    the direct sum
"""
import math

import torch

from paper_1010_1482_amd import hfmm

DEV = "cuda:0"
EXACT_PAIRS = 1.2e11  # direct sums in 64 bits up to this many pairs


def listed():
    return [
        # a serving request of the smallest size of the trace: launches and
        # read backs are what it costs
        dict(name="serve_1k", kind="solve", dist="plummer", n=1000, mass="equal",
             method="fmm", p=6, leaf=64, prec="fp32"),
        # the trace's middle size, at an odd count
        dict(name="serve_32k", kind="solve", dist="uniform", n=31623, mass="equal",
             method="fmm", p=8, leaf=64, prec="fp32"),
        # a larger request on clustered particles of unequal mass
        dict(name="serve_200k", kind="solve", dist="plummer", n=200003, mass="unequal",
             method="fmm", p=10, leaf=64, prec="fp32"),
        # the headline workload
        dict(name="fmm_1M", kind="solve", dist="uniform", n=1 << 20, mass="equal",
             method="fmm", p=10, leaf=64, prec="fp32"),
        # the large clustered workload: an adaptive tree with every list
        dict(name="fmm_plummer_4M", kind="solve", dist="plummer", n=1 << 22, mass="equal",
             method="fmm", p=8, leaf=32, prec="fp32"),
        # the large high-order workload in a split precision form
        dict(name="fmm_bf16x3_4M", kind="solve", dist="uniform", n=1 << 22, mass="equal",
             method="fmm", p=12, leaf=64, prec="bf16x3"),
        # everything in double precision, charges of both signs
        dict(name="fmm_fp64_262k", kind="solve", dist="uniform", n=262147, mass="mixed",
             method="fmm", p=8, leaf=64, prec="fp64"),
        # the Barnes-Hut treecode at its large size
        dict(name="treecode_4M", kind="solve", dist="plummer", n=1 << 22, mass="equal",
             method="treecode", p=3, leaf=32, prec="fp32"),
        # the treecode over the FMM lists
        dict(name="fmmlist_1M", kind="solve", dist="plummer", n=1 << 20, mass="equal",
             method="treecode_fmmlist", p=3, leaf=32, prec="fp32"),
        # fixed sources whose masses change (an iterative solver), the field
        # wanted at other points
        dict(name="resident_262k", kind="resident", dist="plummer", n=1 << 18, nt=100003,
             mass="unequal", method="fmm", p=8, leaf=64, prec="fp32"),
        # five steps of an N-body simulation
        dict(name="leapfrog_131k", kind="leapfrog", dist="plummer", n=1 << 17, mass="equal",
             method="fmm", p=8, leaf=64, prec="fp32", steps=5),
        # all pairs, below the size at which a tree pays
        dict(name="direct_30k", kind="direct", dist="uniform", n=30011, mass="equal",
             method="direct", p=1, leaf=64, prec="fp32"),
    ]


def _size(rng, lo, hi):
    """Log-uniform; every other one odd, some a power of two."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    how = rng.random()
    if how < 0.5:
        return n | 1
    if how < 0.65:
        return min(hi, 1 << int(round(math.log2(n))))
    return n


def draw(rng):
    kind = rng.choice(["fmm", "fmm", "fmm", "lowp", "fp64", "treecode", "fmmlist", "resident",
                       "leapfrog", "direct"])
    c = dict(kind="solve", dist=rng.choice(["uniform", "plummer"]), n=0,
             mass=rng.choice(["equal", "unequal", "mixed"]), method="fmm",
             p=rng.choice([6, 8, 10]), leaf=rng.choice([32, 64]), prec="fp32")
    if kind == "fmm":
        c["n"] = _size(rng, 1000, 2 << 20)
    elif kind == "lowp":
        c["prec"] = rng.choice(["bf16x3", "fp16x3", "fp16", "bf16"])
        c["p"] = rng.choice([8, 10, 12])
        c["n"] = _size(rng, 30000, 2 << 20)
    elif kind == "fp64":
        c.update(prec="fp64", n=_size(rng, 1000, 1 << 19))
    elif kind == "treecode":
        c.update(method="treecode", p=3, leaf=rng.choice([16, 32]), n=_size(rng, 1000, 2 << 20))
    elif kind == "fmmlist":
        c.update(method="treecode_fmmlist", p=3, leaf=32, n=_size(rng, 1000, 2 << 20))
    elif kind == "resident":
        c.update(kind="resident", n=_size(rng, 1000, 1 << 20), nt=_size(rng, 500, 1 << 19))
    elif kind == "leapfrog":
        c.update(kind="leapfrog", dist="plummer", mass="equal", n=_size(rng, 1000, 1 << 18),
                 steps=rng.choice([2, 3, 5]))
    else:
        c.update(kind="direct", method="direct", p=1, leaf=64, n=_size(rng, 500, 100000),
                 prec=rng.choice(["fp32", "fp32", "fp64"]))
        if c["prec"] == "fp64":
            c["n"] = min(c["n"], 50000)
    return c


# ---------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(1 + int(seed))
    return g


def _rand(g, *shape):
    return torch.rand(*shape, dtype=torch.float64, device=DEV, generator=g)


def _directions(g, n):
    cz = 2.0 * _rand(g, n) - 1.0
    ph = (2.0 * math.pi) * _rand(g, n)
    sz = torch.sqrt(torch.clamp(1.0 - cz * cz, min=0.0))
    return sz * torch.cos(ph), sz * torch.sin(ph), cz


def _positions(g, dist, n):
    if dist == "uniform":
        return [_rand(g, n) for _ in range(3)]
    # Plummer sphere of scale radius 1 cut at r = 20: the mass within r is
    # (1 + r^-2)^(-3/2) of the whole
    u = (1.0 - _rand(g, n)) * (1.0 + 1.0 / 400.0) ** -1.5
    r = 1.0 / torch.sqrt(u ** (-2.0 / 3.0) - 1.0)
    return [(r * d).contiguous() for d in _directions(g, n)]


def _masses(g, kind, n):
    if kind == "equal":
        return torch.full((n,), 1.0 / n, dtype=torch.float64, device=DEV)
    mag = 10.0 ** (2.0 * _rand(g, n) - 1.0)
    mag /= mag.sum()
    if kind == "mixed":
        return torch.where(_rand(g, n) < 0.5, -mag, mag)
    return mag


def _inputs(case, seed):
    """Positions, masses, and the targets (resident) or velocities (leapfrog)."""
    g = _gen(seed)
    n = case["n"]
    pos = _positions(g, case["dist"], n)
    m = _masses(g, case["mass"], n)
    more = None
    if case["kind"] == "resident":
        more = _positions(g, case["dist"], case["nt"])
    elif case["kind"] == "leapfrog":
        # isotropic velocities of about the Plummer sphere's own dispersion
        v = 0.7 * (1.0 + sum(a * a for a in pos)) ** -0.25 * _rand(g, n)
        more = [(v * d).contiguous() for d in _directions(g, n)]
    return pos, m, more


DT, EPS2, SLACK = 1e-4, 1e-6, 1.0 / 16.0  # the time loop's step, softening and slack


def prepare(case, seed):
    pos, m, more = _inputs(case, seed)
    s = dict(case=case, pos=pos, m=m, more=more)
    if case["kind"] == "resident":
        s["tree"] = hfmm.Tree(*pos, leaf_max=case["leaf"], max_targets=case["nt"])
    return s


def run(s):
    c = s["case"]
    if c["kind"] == "solve":
        return hfmm.solve(*s["pos"], s["m"], p=c["p"], method=c["method"], precision=c["prec"],
                          leaf_max=c["leaf"])
    if c["kind"] == "resident":
        s["tree"].upward(s["m"], c["p"], c["method"], c["prec"])
        return s["tree"].evaluate(targets=s["more"])
    if c["kind"] == "leapfrog":
        # the call moves the particles in place: the program keeps its start
        pos = [a.clone() for a in s["pos"]]
        vel = [a.clone() for a in s["more"]]
        field = hfmm.leapfrog(*pos, *vel, s["m"], DT, c["steps"], p=c["p"], method=c["method"],
                              precision=c["prec"], leaf_max=c["leaf"], eps2=EPS2, slack=SLACK)
        return field, pos, vel
    return hfmm.direct(*s["pos"], s["m"], precision=c["prec"])


# ---------------------------------------------------------------- reference

def _direct64(pos, m, tgt, eps2=0.0):
    """phi, ax, ay, az of the direct sum in 64 bits; pairs at zero separation skipped."""
    n, nt = m.numel(), tgt[0].numel()
    src = torch.stack([m, m * pos[0], m * pos[1], m * pos[2]], 1)
    out = torch.empty(4, nt, dtype=torch.float64, device=DEV)
    rows = max(1, min(nt, (1 << 24) // max(n, 1)))
    for a in range(0, nt, rows):
        b = min(nt, a + rows)
        d = tgt[0][a:b, None] - pos[0][None, :]
        r2 = d * d
        for k in (1, 2):
            torch.sub(tgt[k][a:b, None], pos[k][None, :], out=d)
            r2.addcmul_(d, d)
        r2.masked_fill_(r2 == 0.0, math.inf).add_(eps2)
        w = r2.rsqrt_()
        out[0, a:b] = w @ m
        torch.mul(w, w, out=d)
        f = (d.mul_(w)) @ src
        for k in range(3):
            out[k + 1, a:b] = f[:, k + 1] - tgt[k][a:b] * f[:, 0]
    return out


def exact(case, seed):
    n, nt = case["n"], case.get("nt", case["n"])
    if float(n) * nt * (case.get("steps", 0) + 1) > EXACT_PAIRS:
        return None
    pos, m, more = _inputs(case, seed)
    if case["kind"] == "resident":
        return tuple(_direct64(pos, m, more))
    if case["kind"] == "leapfrog":
        vel = more
        f = _direct64(pos, m, pos, EPS2)
        for _ in range(case["steps"]):
            vel = [v + (0.5 * DT) * a for v, a in zip(vel, f[1:])]
            pos = [x + DT * v for x, v in zip(pos, vel)]
            f = _direct64(pos, m, pos, EPS2)
            vel = [v + (0.5 * DT) * a for v, a in zip(vel, f[1:])]
        return tuple(f), pos, vel
    return tuple(_direct64(pos, m, pos))


# ---------------------------------------------------------------- work

def _leaf_count(n, leaf):
    """Particles in a leaf of the uniform cube's tree."""
    c = float(n)
    while c > leaf:
        c /= 8.0
    return c


def work(case):
    """Inputs read once and outputs written once; the pairs summed directly
    (21 flops each: the paper's 19 and the potential) and the translations
    (2 p^4 per M2L pair, 80 per M2P at p = 3) of a tree whose leaves hold as
    many particles as the uniform cube's."""
    n, p = float(case["n"]), case["p"]
    nt = float(case.get("nt", n))
    e = 8 if case["prec"] == "fp64" else 4
    evals = case.get("steps", 0) + 1
    byts = (32.0 * n + 4 * e * nt + (24.0 * nt if case["kind"] == "resident" else 0.0)) * 1.0
    if case["kind"] == "leapfrog":
        byts += 96.0 * n * case["steps"]
    if case["kind"] == "direct":
        return dict(bytes=byts, flops=21.0 * n * nt)
    c = _leaf_count(n, case["leaf"])
    leaves = n / c
    near = 21.0 * nt * min(n, 27.0 * c)
    if case["method"] == "fmm":
        far = 189.0 * leaves * 8.0 / 7.0 * 2.0 * p ** 4 if leaves > 64 else 0.0
    else:
        levels = max(0.0, math.log(leaves, 8.0) - 1.0) if leaves > 1 else 0.0
        far = 80.0 * nt * 189.0 * levels
    return dict(bytes=byts, flops=evals * (near + far))
