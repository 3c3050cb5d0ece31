"""Timed workloads of the framework, each one call (or the few calls of one step) of its public
front ends, with inputs drawn from a seed and reference values in plain torch.

listed() are the workloads themselves, draw() gives further ones of the same ranges; prepare()
makes what a program keeps between calls (hierarchies, fields, chain states), run() is one pass,
work() the bytes and operations a pass cannot do without, and exact() the same outputs computed
in float64 by dense, FFT and periodic-shift formulas that share no code with the library.

All fields are synthetic: chains start from the zero field, right-hand sides are N(0, 1), points
are uniform in the channel.  h = 1 and kT = 1 throughout.
"""
import math

import numpy as np
import torch

from paper_1003_2680_amd.api import Hierarchy
from paper_1003_2680_amd.batch import BatchRunner, Instance
from paper_1003_2680_amd.composite import CompositeSampler
from paper_1003_2680_amd.grid2d import Hierarchy2D
from paper_1003_2680_amd.selm import SELM

COARSEST_MAX = 512
SWEEPS = 4          # V(2, 2)
F64 = torch.float64


# ------------------------------------------------------------------------------------ workloads

def listed():
    return [
        # The smallest chain in use (200 cycles of it are the plain method's check): every
        # launch is tiny, so latency and the number of launches decide.
        dict(name="chain_16", kind="chain", nx=16, ny=16, nz=16, ncomp=1, n=50, stride=1,
             levels=3, precision="fp64"),
        # A grid whose extents are no powers of two and differ per axis, two components.
        dict(name="chain_ragged", kind="chain", nx=72, ny=40, nz=48, ncomp=2, n=10, stride=1,
             precision="fp64"),
        # One three-component velocity field on the headline grid, a sample every two cycles:
        # the latency-bound form a single simulation runs.
        dict(name="chain_128", kind="chain", nx=128, ny=128, nz=128, ncomp=3, n=4, stride=2,
             levels=6, precision="fp64"),
        # The grid that exceeds every cache: one chain, one cycle per sample.
        dict(name="chain_512", kind="chain", nx=512, ny=512, nz=256, ncomp=1, n=1, stride=1,
             precision="fp64"),
        # The throughput form of the headline workload: eight chains of the three-component field
        # in every launch, two stream groups, eight observables of each emitted sample.
        dict(name="chains_128", kind="chains", nx=128, ny=128, nz=128, chains=8, cpc=3, n=2,
             stride=2, levels=6, precision="fp64"),
        # Deterministic response: the three-component field solved to 1e-12.
        dict(name="solve_128", kind="solve", nx=128, ny=128, nz=128, ncomp=3, rtol=1e-12,
             levels=6, precision="fp64"),
        # A served request: one component, flat channel, FP32-refined, to 1e-10.
        dict(name="solve_served", kind="solve", nx=256, ny=256, nz=64, ncomp=1, rtol=1e-10,
             precision="fp32_refined"),
        # 64 instances of uneven size in one call, FP32-refined, float32 samples.
        dict(name="uneven_64", kind="uneven", instances=64, edges="32,48,64,96", n=2,
             precision="fp32_refined"),
        # The adaptive workload: 12 M composite unknowns, FAC cycles of three composite sweeps
        # around a V(1, 0) base cycle.
        dict(name="composite_cycles", kind="composite", nx=256, ny=256, nz=128, cycles=2, nu=3,
             mu1=1, mu2=0, precision="fp64"),
        # A solve on a smaller adaptive mesh of the same shape.
        dict(name="composite_solve", kind="composite_solve", nx=64, ny=64, nz=32, nu=3, mu1=1,
             mu2=0, rtol=1e-10, precision="fp64"),
        # One Euler-Maruyama step of 64 structure points in the headline channel: mobility
        # solves, a driving field, projections.
        dict(name="selm_step", kind="selm", nx=128, ny=128, nz=128, points=64, rtol=1e-10),
        # The two-dimensional sampler as the decorrelation study runs it: eight chains.
        dict(name="plane_128", kind="plane", nx=128, nz=128, chains=8, n=20),
    ]


def level_dims(dims, levels=0):
    """Extents of the levels, finest first ((nx, ny, nz) or (nx, nz)): halve while even,
    smoothable and short of `levels` (0: while more than COARSEST_MAX unknowns)."""
    out = [tuple(dims)]
    while True:
        d = out[-1]
        per, nz = d[:-1], d[-1]
        first = len(out) == 1
        ok = all(v % 2 == 0 for v in d) and all(v % (2 if first else 4) == 0 for v in per)
        if not ok or (len(out) == levels if levels else math.prod(d) <= COARSEST_MAX):
            return out
        out.append(tuple(v // 2 for v in d))


def _spread(rng, lo, hi, step):
    """A multiple of `step` in [lo, hi], uniform over its logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def _grid(rng, lo, hi, most, nz_lo=None):
    """Extents whose coarsest level stays small, with at most `most` cells."""
    while True:
        d = (_spread(rng, lo, hi, 8), _spread(rng, lo, hi, 8),
             _spread(rng, nz_lo or lo, min(hi, 128), 4))
        if math.prod(d) <= most and math.prod(level_dims(d)[-1]) <= 800:
            return d


def draw(rng):
    kind = rng.choice(["chain", "chain", "chains", "solve", "solve", "uneven", "composite",
                       "composite_solve", "selm", "plane"])
    prec = rng.choice(["fp64", "fp64", "fp32_refined"])
    if kind == "chain":
        nx, ny, nz = _grid(rng, 16, 256, 1 << 22)
        return dict(kind=kind, nx=nx, ny=ny, nz=nz, ncomp=rng.choice([1, 2, 3]),
                    n=rng.randint(1, 6), stride=rng.choice([1, 2]), precision=prec)
    if kind == "chains":
        nx, ny, nz = _grid(rng, 16, 128, 1 << 20)
        return dict(kind=kind, nx=nx, ny=ny, nz=nz, chains=rng.randint(2, 10),
                    cpc=rng.choice([1, 3]), n=rng.randint(1, 4), stride=2, precision=prec)
    if kind == "solve":
        nx, ny, nz = _grid(rng, 16, 256, 1 << 22)
        return dict(kind=kind, nx=nx, ny=ny, nz=nz, ncomp=rng.choice([1, 3]),
                    rtol=rng.choice([1e-10, 1e-12]), precision=prec)
    if kind == "uneven":
        edges = sorted(rng.sample([16, 32, 40, 48, 56, 64, 80, 96], rng.randint(2, 5)))
        return dict(kind=kind, instances=rng.randint(6, 48), edges=",".join(map(str, edges)),
                    n=rng.randint(1, 3), precision=prec)
    if kind in ("composite", "composite_solve"):
        nx, ny = 16 * rng.randint(2, 8), 16 * rng.randint(2, 8)
        nz = 8 * rng.randint(2, 8)
        while math.prod(level_dims((nx, ny, nz))[-1]) > 800:
            nx, ny = 16 * rng.randint(2, 8), 16 * rng.randint(2, 8)
            nz = 8 * rng.randint(2, 8)
        c = dict(kind=kind, nx=nx, ny=ny, nz=nz, nu=rng.choice([2, 3]), mu1=1,
                 mu2=rng.choice([0, 1]), precision=prec)
        return dict(c, cycles=rng.randint(1, 4)) if kind == "composite" else dict(c, rtol=1e-10)
    if kind == "selm":
        nx, ny, nz = _grid(rng, 16, 96, 1 << 19)
        return dict(kind=kind, nx=nx, ny=ny, nz=nz, points=rng.randint(1, 128),
                    rtol=rng.choice([1e-8, 1e-10]))
    while True:
        nx, nz = _spread(rng, 16, 256, 4), _spread(rng, 16, 256, 4)
        if math.prod(level_dims((nx, nz))[-1]) <= 800:
            return dict(kind="plane", nx=nx, nz=nz, chains=rng.randint(1, 12),
                        n=rng.randint(2, 20))


# ---------------------------------------------------------------------------- prepare and run

def _gen(seed, k=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * k + int(seed))
    return g


def _normal(shape, seed, k=0):
    return torch.randn(shape, generator=_gen(seed, k), dtype=F64, device="cuda")


def _box(c):
    """The central half in x and y, the lowest quarter in z next to the wall."""
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    return (nx // 4, nx // 4 + nx // 2, ny // 4, ny // 4 + ny // 2, 0, nz // 4)


def _modes(c):
    """Long-wave observables: (a, b, m) real eigenvectors of the channel's operator."""
    return [(0, 0, 1), (1, 0, 1), (2, 0, 1), (0, 1, 1), (0, 2, 1), (0, 0, 2), (1, 1, 1),
            (2, 2, 1)]


def _edges(c, seed):
    sizes = [int(v) for v in c["edges"].split(",")]
    pick = np.random.default_rng(2026).integers(0, len(sizes), c["instances"])
    return [Instance((sizes[k],) * 3, 1000 * seed + i) for i, k in enumerate(pick)]


def _points(c, seed):
    """Points at least two cells from the walls, and their forces."""
    ext = torch.tensor([c["nx"], c["ny"], c["nz"] - 4.0], dtype=F64, device="cuda")
    X = torch.rand((c["points"], 3), generator=_gen(seed, 1), dtype=F64, device="cuda") * ext
    X[:, 2] += 2.0
    return X, _normal((c["points"], 3), seed, 2)


def prepare(case, seed):
    c, kind = case, case["kind"]
    s = {"case": c, "seed": int(seed)}
    if kind == "chain":
        # a continued chain: the state and the next cycle stay with the caller
        s["H"] = Hierarchy(c["nx"], c["ny"], c["nz"], ncomp=c["ncomp"], stride=c["stride"],
                           levels=c.get("levels", 0), precision=c["precision"])
        s["x"], s["cycle"] = s["H"].new_state(), 0
    elif kind == "chains":
        s["H"] = Hierarchy(c["nx"], c["ny"], c["nz"], ncomp=c["chains"] * c["cpc"],
                           stride=c["stride"], levels=c.get("levels", 0),
                           precision=c["precision"])
        s["H"].set_stream_groups(2)
        s["x"], s["cycle"] = s["H"].new_state(), 0
    elif kind == "solve":
        s["H"] = Hierarchy(c["nx"], c["ny"], c["nz"], ncomp=c["ncomp"],
                           levels=c.get("levels", 0), precision=c["precision"])
        s["f"] = _normal(s["H"].shape, seed)
    elif kind == "uneven":
        s["R"] = BatchRunner(_edges(c, seed), precision=c["precision"], stream_groups=2)
        s["R"].start()
    elif kind in ("composite", "composite_solve"):
        s["S"] = CompositeSampler(c["nx"], c["ny"], c["nz"], _box(c), nu=c["nu"], mu1=c["mu1"],
                                  mu2=c["mu2"], precision=c["precision"])
        if kind == "composite":
            s["x"], s["cycle"] = s["S"].zeros(), 0
        else:
            s["f"] = _rhs_composite(c, seed)
    elif kind == "selm":
        s["E"] = SELM(c["nx"], c["ny"], c["nz"], max_points=c["points"])
        s["X"], s["F"] = _points(c, seed)
        s["xi"], s["step"] = s["E"].new_state(), 0
    else:
        s["H"] = Hierarchy2D(c["nx"], c["nz"], ncomp=c["chains"])
        s["x"], s["cycle"] = s["H"].new_state(), 0
    return s


def run(s):
    c, kind, seed = s["case"], s["case"]["kind"], s["seed"]
    if kind == "chain":
        out, _ = s["H"].sample(c["n"], seed, first_cycle=s["cycle"], state=s["x"])
        s["cycle"] += c["n"] * c["stride"]
        return {"samples": out, "state": s["x"]}
    if kind == "chains":
        nc = c["chains"]
        out = torch.empty((c["n"],) + s["H"].shape, dtype=F64, device="cuda")
        _, obs, _ = s["H"].sample_batch(c["n"], seeds=[seed + 10 * k for k in range(nc)],
                                        first_cycles=[s["cycle"]] * nc, state=s["x"], out=out,
                                        modes=_modes(c), with_obs=True)
        s["cycle"] += c["n"] * c["stride"]
        return {"samples": out, "obs": obs}
    if kind == "solve":
        return s["H"].solve(s["f"], rtol=c["rtol"])[0]
    if kind == "uneven":
        return list(s["R"].sample(c["n"]).values())
    if kind == "composite":
        s["S"].sample(s["x"][0], s["x"][1], c["cycles"], seed, first_cycle=s["cycle"])
        s["cycle"] += c["cycles"]
        return {"coarse": s["x"][0], "fine": s["x"][1]}
    if kind == "composite_solve":
        uc, uf, _ = s["S"].solve(s["f"][0], s["f"][1], rtol=c["rtol"])
        return {"coarse": uc, "fine": uf}
    if kind == "selm":
        s["E"].step(s["X"], s["F"], 1e-3, seed, s["step"], s["xi"], rtol=c["rtol"])
        s["step"] += 1
        return {"X": s["X"], "state": s["xi"]}
    out, _ = s["H"].sample(c["n"], seed, first_cycle=s["cycle"], state=s["x"])
    s["cycle"] += c["n"]
    return {"samples": out, "state": s["x"]}


# --------------------------------------------------------------------------------------- work

def _cycle_work(dims, width, sweeps=SWEEPS):
    """One V-cycle of one component: every sweep reads and writes its level's field once (and
    reads the right-hand side below level 0); the transfers read the field once more and touch
    the coarse level.  Operations: the separable stencils, the 8 x 8 (4 x 4) block solves, the
    random numbers (about 60 per value)."""
    b = f = 0.0
    for l, d in enumerate(level_dims(dims)):
        n = math.prod(d)
        b += n * width * (sweeps * (2 if l == 0 else 3) + 4)
        f += n * sweeps * ((10 if l == 0 else 200) + 60) + 40 * n
    return b, f


def work(case):
    c, kind = case, case["kind"]
    if kind in ("composite", "composite_solve"):
        n = c["nx"] * c["ny"] * c["nz"]
        box = _box(c)
        fine = 8 * math.prod(box[2 * a + 1] - box[2 * a] for a in range(3))
        cycles = c.get("cycles", 8)
        w = 8 if c["precision"] == "fp64" else 4
        b, f = _cycle_work((c["nx"], c["ny"], c["nz"]), w, c["mu1"] + c["mu2"])
        b += (n + fine) * w * (2 * c["nu"] + 3)
        f += (n + fine) * (c["nu"] * 75 + 20)
        return {"bytes": cycles * b, "flops": cycles * f}
    if kind == "plane":
        b, f = _cycle_work((c["nx"], c["nz"]), 8)
        k = c["chains"] * c["n"]
        return {"bytes": k * (b + 8.0 * c["nx"] * c["nz"]), "flops": k * f}
    if kind == "uneven":
        w = 8 if c["precision"] == "fp64" else 4
        b = f = 0.0
        for inst in _edges(c, 0):
            bi, fi = _cycle_work(inst.dims, w)
            n = math.prod(inst.dims)
            b += c["n"] * (bi + 4.0 * n + (0 if w == 8 else 24.0 * n))
            f += c["n"] * fi
        return {"bytes": b, "flops": f}
    dims = (c["nx"], c["ny"], c["nz"])
    n = math.prod(dims)
    if kind == "selm":
        # two scalar solves, one of three components (about 9 cycles each at 1e-10), two cycles
        # of the driving chain and its projection's solve
        b, f = _cycle_work(dims, 8)
        return {"bytes": (9 * (3 + 3) + 6) * b + 8.0 * n * 30, "flops": (9 * 6 + 6) * f}
    b, f = _cycle_work(dims, 8 if c["precision"] == "fp64" else 4)
    if c["precision"] != "fp64":
        b += 24.0 * n  # the float64 state read and written, and the float64 residual's inputs
    if kind == "solve":
        cycles = round(math.log(c["rtol"]) / math.log(0.08))
        return {"bytes": c["ncomp"] * (cycles * (b + 8.0 * n) + 16.0 * n),
                "flops": c["ncomp"] * cycles * f}
    comps = c["ncomp"] if kind == "chain" else c["chains"] * c["cpc"]
    k = comps * c["n"] * c["stride"]
    return {"bytes": k * b + 8.0 * n * comps * (c["n"] + 2), "flops": k * f}


# -------------------------------------------------------------------------------------- exact

def _philox(call, word1, cycle, seed):
    """Philox4x32-10 words of counter (call, word1, cycle lo, cycle hi); int64 tensors."""
    m32 = 0xFFFFFFFF
    w0, w1 = torch.broadcast_tensors(call, word1)
    w2 = torch.full_like(w0, cycle & m32)
    w3 = torch.full_like(w0, (cycle >> 32) & m32)
    k0, k1 = seed & m32, (seed >> 32) & m32
    for _ in range(10):
        p0, p1 = w0 * 0xD2511F53, w2 * 0xCD9E8D57
        w0, w1, w2, w3 = (((p1 >> 32) & m32) ^ w1 ^ k0, p1 & m32,
                          ((p0 >> 32) & m32) ^ w3 ^ k1, p0 & m32)
        k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
    return w0, w1, w2, w3


def _uniform(a, b):
    return (((a << 21) | (b >> 11)).to(F64) + 0.5) * 2.0 ** -53


def _normals(site, sid, comp, cycle, seed):
    """N(0, 1) of each site (call site >> 1, cosine for the even site, sine for the odd)."""
    w0, w1, w2, w3 = _philox(site >> 1, comp * 65536 + sid, cycle, seed)
    r = torch.sqrt(-2.0 * torch.log(_uniform(w0, w1)))
    t = 2.0 * math.pi * _uniform(w2, w3)
    return r * torch.where(site % 2 == 0, torch.cos(t), torch.sin(t))


def _prolongation(nc, wall):
    P = torch.zeros((2 * nc, nc), dtype=F64)
    for j in range(nc):
        for fine, other in ((2 * j, j - 1), (2 * j + 1, j + 1)):
            P[fine, j] += 0.75
            if not wall:
                P[fine, other % nc] += 0.25
            elif 0 <= other < nc:
                P[fine, other] += 0.25
            else:
                P[fine, j] -= 0.25
    return P


def _laplacian(n, wall):
    A = 2.0 * torch.eye(n, dtype=F64)
    for i in range(n):
        for j in (i - 1, i + 1):
            if wall and not 0 <= j < n:
                A[i, i] += 1.0
            else:
                A[i, j % n] -= 1.0
    return A


class _Chain:
    """The stochastic V(2, 2) chain of one seed: dims (nx, ny, nz) or (nx, nz), fields
    [components, nz, (ny,) nx]."""

    def __init__(self, dims, device, levels=0):
        self.dims, self.dev, self.lv = level_dims(dims, levels), device, []
        nax = len(dims)
        A = [_laplacian(n, a == nax - 1) for a, n in enumerate(dims)]
        M = [torch.eye(n, dtype=F64) for n in dims]
        for l, d in enumerate(self.dims):
            if l:
                P = [_prolongation(n, a == nax - 1) for a, n in enumerate(d)]
                A = [p.T @ a @ p for p, a in zip(P, A)]
                M = [p.T @ m @ p for p, m in zip(P, M)]
                self.lv[-1]["P"] = [p.to(device) for p in P]
            lev = {"d": d, "A": [a.to(device) for a in A], "M": [m.to(device) for m in M]}
            if l and l + 1 < len(self.dims):
                lev["block"] = self._blocks(A, M, d)
            if l + 1 == len(self.dims):
                full = 0
                for k in range(nax):
                    t = torch.ones((1, 1), dtype=F64)
                    for a in range(nax - 1, -1, -1):
                        t = torch.kron(t, A[a] if a == k else M[a])
                    full = full + t
                lev["L"] = torch.linalg.cholesky(full).to(device)
            self.lv.append(lev)

    def _blocks(self, A, M, d):
        nax, out = len(d), []
        for bz in range(d[-1] // 2):
            full = 0
            for k in range(nax):
                t = torch.ones((1, 1), dtype=F64)
                for a in range(nax - 1, -1, -1):
                    o = 2 * bz if a == nax - 1 else 0
                    t = torch.kron(t, (A[a] if a == k else M[a])[o:o + 2, o:o + 2])
                full = full + t
            out.append(full)
        B = torch.stack(out)
        Lt = torch.linalg.inv(torch.linalg.cholesky(B)).transpose(1, 2)
        return torch.linalg.inv(B).to(self.dev), Lt.contiguous().to(self.dev)

    @staticmethod
    def _along(m, x, axis):
        """Dense matrix m applied along `axis` (0 = x, last dimension)."""
        x = x.movedim(-1 - axis, -1)
        return (x.reshape(-1, x.shape[-1]) @ m.T).reshape(x.shape[:-1] + (m.shape[0],)).movedim(
            -1, -1 - axis)

    def _ring(self, m, x, axis):
        """Periodic band: the sum of shifted copies."""
        row, out = m[0].tolist(), 0
        for j, v in enumerate(row):
            if v != 0.0:
                out = out + v * torch.roll(x, -j, dims=-1 - axis)
        return out

    def apply(self, l, x):
        lev, nax = self.lv[l], len(self.dims[0])
        out = 0
        for k in range(nax):
            t = x
            for a in range(nax):
                m = lev["A"][a] if a == k else lev["M"][a]
                if l == 0 and a != k:
                    continue
                t = self._along(m, t, a) if a == nax - 1 else self._ring(m, t, a)
            out = out + t
        return out

    def _colours(self, l, x, b, slot, post, seed, cycle):
        lev, d = self.lv[l], self.dims[l]
        nax, nc = len(d), x.shape[0]
        comp = torch.arange(nc, device=self.dev).reshape((nc,) + (1,) * nax)
        if l == 0:
            lex = torch.arange(math.prod(d), device=self.dev).reshape(d[::-1])
            par = sum(torch.arange(n, device=self.dev).reshape((n,) + (1,) * a)
                      for a, n in enumerate(d)) % 2
            dia = torch.full((d[-1],), 2.0 * nax, dtype=F64, device=self.dev)
            dia[0] += 1.0
            dia[-1] += 1.0
            dia = dia.reshape((-1,) + (1,) * (nax - 1))
            for colour in ((1, 0) if post else (0, 1)):
                z = _normals(lex >> 1, l | slot << 4 | colour << 12, comp, cycle, seed)
                new = x + (b - self.apply(l, x)) / dia + z / torch.sqrt(dia)
                x = torch.where(par == colour, new, x)
            return x
        Ai, Lt = lev["block"]
        nb = [n // 2 for n in d]
        kk = torch.arange(2 ** nax, device=self.dev)
        for colour in (range(2 ** nax - 1, -1, -1) if post else range(2 ** nax)):
            bits = [(colour >> a) & 1 for a in range(nax)]
            bi = [torch.arange(bits[a], nb[a], 2, device=self.dev) for a in range(nax)]
            shape, sel = [nc], [slice(None)]
            for a in range(nax - 1, -1, -1):
                shape += [nb[a], 2]
                sel += [slice(bits[a], None, 2), slice(None)]
            perm = [0] + [1 + 2 * a for a in range(nax)] + [2 + 2 * a for a in range(nax)]
            r = (b - self.apply(l, x)).reshape(shape)[tuple(sel)].permute(perm)
            outer = r.shape
            bid = sum((v * math.prod(nb[:a])).reshape((-1,) + (1,) * a)
                      for a, v in enumerate(bi)).unsqueeze(-1)
            z = _normals(2 ** nax * bid + kk, l | slot << 4 | colour << 12,
                         comp.unsqueeze(-1), cycle, seed)
            nz = outer[1]
            upd = (torch.matmul(r.reshape(nc, nz, -1, 2 ** nax),
                                Ai[bits[-1]::2].transpose(1, 2).contiguous())
                   + torch.matmul(z.reshape(nc, nz, -1, 2 ** nax),
                                  Lt[bits[-1]::2].transpose(1, 2).contiguous()))
            x = x.clone()
            x.view(shape)[tuple(sel)].permute(perm).add_(upd.reshape(outer))
        return x

    def cycle(self, x, b, seed, cycle, l=0):
        if l + 1 == len(self.dims):
            L, nc = self.lv[l]["L"], x.shape[0]
            site = torch.arange(L.shape[0], device=self.dev)
            z = _normals(site, l | 1 << 24, torch.arange(nc, device=self.dev)[:, None], cycle,
                         seed)
            rhs = torch.linalg.solve_triangular(L, b.reshape(nc, -1).T, upper=False) + z.T
            return torch.linalg.solve_triangular(L.T, rhs, upper=True).T.reshape(x.shape)
        for s in range(2):
            x = self._colours(l, x, b, s, False, seed, cycle)
        r, P = b - self.apply(l, x), self.lv[l]["P"]
        for a, p in enumerate(P):
            r = self._along(p.T, r, a)
        e = self.cycle(torch.zeros_like(r), r, seed, cycle, l + 1)
        for a, p in enumerate(P):
            e = self._along(p, e, a)
        x = x + e
        for s in range(2, 4):
            x = self._colours(l, x, b, s, True, seed, cycle)
        return x

    def run(self, x, cycles, stride, seed, first=0):
        """Every stride-th field of `cycles` cycles from x (b = 0), and the last."""
        out, b = [], torch.zeros_like(x)
        for k in range(cycles):
            x = self.cycle(x, b, seed, first + k)
            if (k + 1) % stride == 0:
                out.append(x)
        return torch.stack(out), x


def _wall_modes(nz, device):
    m = torch.arange(1, nz + 1, dtype=F64, device=device)
    z = torch.arange(nz, dtype=F64, device=device) + 0.5
    V = torch.sin(math.pi * m[:, None] * z / nz)
    return V / torch.linalg.norm(V, dim=1, keepdim=True), 4.0 * torch.sin(
        math.pi * m / (2 * nz)) ** 2


def _solve(f):
    """A^-1 f for f [..., nz, ny, nx] by Fourier in x and y and sines in z."""
    nz, ny, nx = f.shape[-3:]
    V, lz = _wall_modes(nz, f.device)
    lx = 4.0 * torch.sin(math.pi * torch.arange(nx, dtype=F64, device=f.device) / nx) ** 2
    ly = 4.0 * torch.sin(math.pi * torch.arange(ny, dtype=F64, device=f.device) / ny) ** 2
    g = torch.fft.rfft2(_Chain._along(V, f, 2))
    g = g / (lz[:, None, None] + ly[:, None] + lx[:nx // 2 + 1])
    return _Chain._along(V.T.contiguous(), torch.fft.irfft2(g, s=(ny, nx)), 2)


def _observables(c, x):
    """Projections of x [..., nz, ny, nx] on the modes, and the energy 1/2 x^T A x."""
    def ring(n, a):
        i = torch.arange(n, dtype=F64, device=x.device)
        if a == 0:
            return torch.full((n,), n ** -0.5, dtype=F64, device=x.device)
        t = 2.0 * math.pi * ((a + 1) // 2) * i / n
        return math.sqrt(2.0 / n) * (torch.cos(t) if a % 2 else torch.sin(t))
    V, _ = _wall_modes(c["nz"], x.device)
    obs = []
    for a, b, m in _modes(c):
        w = V[m - 1][:, None, None] * ring(c["ny"], b)[:, None] * ring(c["nx"], a)
        obs.append((x * w).sum(dim=(-3, -2, -1)))
    d = [((torch.roll(x, -1, k) - x) ** 2).sum(dim=(-3, -2, -1)) for k in (-1, -2)]
    dz = ((x[..., 1:, :, :] - x[..., :-1, :, :]) ** 2).sum(dim=(-3, -2, -1))
    wall = 2.0 * (x[..., 0, :, :] ** 2 + x[..., -1, :, :] ** 2).sum(dim=(-2, -1))
    return torch.stack(obs + [0.5 * (d[0] + d[1] + dz + wall)], dim=-1)


def _rhs_composite(c, seed):
    """N(0, 1) on the base cells and on the fine cells of the box."""
    x0, x1, y0, y1, z0, z1 = _box(c)
    return (_normal((c["nz"], c["ny"], c["nx"]), seed, 1),
            _normal((2 * (z1 - z0), 2 * (y1 - y0), 2 * (x1 - x0)), seed, 2))


def _composite_apply(c, uc, uf):
    """A u on the composite mesh from its face fluxes (covered base cells hold and give 0)."""
    x0, x1, y0, y1, z0, z1 = _box(c)
    open_ = torch.ones_like(uc)
    open_[z0:z1, y0:y1, x0:x1] = 0.0
    ac, af = torch.zeros_like(uc), torch.zeros_like(uf)
    for dim in (1, 2):  # coarse faces in y and x
        for sh in (1, -1):
            ac += open_ * torch.roll(open_, sh, dim) * (uc - torch.roll(uc, sh, dim))
    g = open_[1:] * open_[:-1] * (uc[1:] - uc[:-1])
    ac[1:] += g
    ac[:-1] -= g
    ac[0] += 2.0 * open_[0] * uc[0]
    ac[-1] += 2.0 * uc[-1]
    for dim in range(3):  # fine faces: area 1/4 over distance 1/2
        n = uf.shape[dim]
        g = 0.5 * (uf.narrow(dim, 1, n - 1) - uf.narrow(dim, 0, n - 1))
        af.narrow(dim, 1, n - 1).add_(g)
        af.narrow(dim, 0, n - 1).sub_(g)
    af[0] += uf[0]  # the lower wall: twice the value over half a fine cell
    lo, hi = (z0, y0, x0), (z1, y1, x1)
    for dim in range(3):  # faces between the box and the base grid: distance 3/4
        for side in (0, 1):
            if dim == 0 and side == 0:
                continue
            fine = uf.select(dim, uf.shape[dim] - 1 if side else 0)
            mean = fine.reshape(fine.shape[0] // 2, 2, fine.shape[1] // 2, 2).mean(dim=(1, 3))
            at = (hi[dim] if side else lo[dim] - 1) % uc.shape[dim]
            rest = [k for k in range(3) if k != dim]

            def face(t):
                t = t.select(dim, at)
                for q, k in enumerate(rest):
                    t = t.narrow(q, lo[k], hi[k] - lo[k])
                return t
            g = (4.0 / 3.0) * (face(uc) - mean)
            face(ac).add_(g)
            af.select(dim, uf.shape[dim] - 1 if side else 0).sub_(
                0.25 * g.repeat_interleave(2, 0).repeat_interleave(2, 1))
    return ac, af


def _composite_solve(c, fc, ff):
    """Conjugate gradients on the composite operator to 1e-14."""
    x0, x1, y0, y1, z0, z1 = _box(c)
    fc = fc.clone()
    fc[z0:z1, y0:y1, x0:x1] = 0.0
    dot = lambda a, b: float((a[0] * b[0]).sum() + (a[1] * b[1]).sum())  # noqa: E731
    u, r = (torch.zeros_like(fc), torch.zeros_like(ff)), (fc, ff)
    p, rr = r, dot(r, r)
    stop = 1e-28 * rr
    for _ in range(5000):
        if rr <= stop:
            break
        q = _composite_apply(c, *p)
        a = rr / dot(p, q)
        u = tuple(v + a * w for v, w in zip(u, p))
        r = tuple(v - a * w for v, w in zip(r, q))
        new = dot(r, r)
        p, rr = tuple(v + (new / rr) * w for v, w in zip(r, p)), new
    return u


def _peskin(r):
    r = r.abs()
    near = (3.0 - 2.0 * r + torch.sqrt((1.0 + 4.0 * r - 4.0 * r * r).clamp(min=0.0))) / 8.0
    far = (5.0 - 2.0 * r - torch.sqrt((-7.0 + 12.0 * r - 4.0 * r * r).clamp(min=0.0))) / 8.0
    return torch.where(r < 1.0, near, torch.where(r < 2.0, far, torch.zeros_like(r)))


class _Coupling:
    """Interpolation, spreading, projection and mobility of the structure points."""

    def __init__(self, c, X):
        dims, self.dev = (c["nx"], c["ny"], c["nz"]), X.device
        k = torch.arange(4, device=self.dev)
        idx, wgt = [], []
        for a, n in enumerate(dims):
            i = torch.floor(X[:, a] - 0.5).long()[:, None] - 1 + k
            w = _peskin(i.to(F64) + 0.5 - X[:, a:a + 1])
            if a == 2:  # beyond a wall: minus the mirror cell
                low, high = i < 0, i >= n
                w = torch.where(low | high, -w, w)
                i = torch.where(low, -1 - i, torch.where(high, 2 * n - 1 - i, i))
            idx.append(i % n)
            wgt.append(w)
        self.cell = ((idx[2][:, :, None, None] * dims[1] + idx[1][:, None, :, None]) * dims[0]
                     + idx[0][:, None, None, :]).reshape(len(X), 64)
        self.w = (wgt[2][:, :, None, None] * wgt[1][:, None, :, None]
                  * wgt[0][:, None, None, :]).reshape(len(X), 64)
        self.shape = (3, dims[2], dims[1], dims[0])
        V, lz = _wall_modes(dims[2], self.dev)
        self.root = V.T @ (torch.sqrt(lz)[:, None] * V)

    def interpolate(self, u):
        v = u.reshape(3, -1)[:, self.cell]
        return (v * self.w).sum(dim=-1).T.contiguous()

    def spread(self, F):
        out = torch.zeros((3, math.prod(self.shape[1:])), dtype=F64, device=self.dev)
        for a in range(3):
            out[a].index_add_(0, self.cell.reshape(-1), (self.w * F[:, a:a + 1]).reshape(-1))
        return out.reshape(self.shape)

    def project(self, u):
        div = (torch.roll(u[0], -1, -1) - u[0] + torch.roll(u[1], -1, -2) - u[1]
               + _Chain._along(self.root, u[2], 2))
        p = _solve(div)
        return torch.stack([u[0] - (torch.roll(p, 1, -1) - p), u[1] - (torch.roll(p, 1, -2) - p),
                            u[2] - _Chain._along(self.root, p, 2)])


def exact(case, seed):
    c, kind = case, case["kind"]
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    if kind == "composite":
        return None  # the Galerkin base operators near the box have no short closed form
    if kind == "chain":
        ch = _Chain((c["nx"], c["ny"], c["nz"]), dev, c.get("levels", 0))
        x = torch.zeros((c["ncomp"], c["nz"], c["ny"], c["nx"]), dtype=F64, device=dev)
        out, x = ch.run(x, c["n"] * c["stride"], c["stride"], seed)
        return {"samples": out, "state": x}
    if kind == "chains":
        ch = _Chain((c["nx"], c["ny"], c["nz"]), dev, c.get("levels", 0))
        x = torch.zeros((c["cpc"], c["nz"], c["ny"], c["nx"]), dtype=F64, device=dev)
        out = torch.cat([ch.run(x, c["n"] * c["stride"], c["stride"], seed + 10 * k)[0]
                         for k in range(c["chains"])], dim=1)
        return {"samples": out, "obs": _observables(c, out)}
    if kind == "solve":
        return _solve(_normal((c["ncomp"], c["nz"], c["ny"], c["nx"]), seed))
    if kind == "uneven":
        insts, chains, by = _edges(c, seed), {}, {}
        for i, inst in enumerate(insts):  # in the order of the runner's groups
            by.setdefault(inst.dims, []).append(i)
        out = []
        for dims, members in by.items():
            ch = chains.setdefault(dims, _Chain(dims, dev))
            for i in members:
                x = torch.zeros((1,) + dims[::-1], dtype=F64, device=dev)
                out.append(ch.run(x, c["n"], 1, insts[i].seed)[0][:, 0])
        return out
    if kind == "composite_solve":
        uc, uf = _composite_solve(c, *_rhs_composite(c, seed))
        return {"coarse": uc, "fine": uf}
    if kind == "selm":
        X, F = _points(c, seed)
        G = _Coupling(c, X)
        ch = _Chain((c["nx"], c["ny"], c["nz"]), dev)
        V = G.interpolate(G.project(_solve(G.project(G.spread(F)))))
        _, xi = ch.run(torch.zeros(G.shape, dtype=F64, device=dev), 2, 1, seed)
        g = math.sqrt(2.0) * G.interpolate(G.project(xi))
        return {"X": X + 1e-3 * V + math.sqrt(1e-3) * g, "state": xi}
    ch = _Chain((c["nx"], c["nz"]), dev)
    x = torch.zeros((c["chains"], c["nz"], c["nx"]), dtype=F64, device=dev)
    out, x = ch.run(x, c["n"], 1, seed)
    return {"samples": out, "state": x}
