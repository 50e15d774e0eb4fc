"""Performance cases: what a program that uses this library has it do.

A case is one pass through a public entry point, with the inputs and the handle that a
program holds before the call:

- kind "solve": mg.Solver.solve, a whole Poisson solve from a zero iterate to rtol
  (2D or 3D; FP64 or mixed precision; every smoother, coarse operator and order);
- kind "rbc": rbc.solve, a whole solve by red-black coarsening (2D, five-point operator);
- kind "serve": a burst of independent 2D requests of mixed sizes through serve.Server.

Sides are 2^k + 1 (what standard coarsening needs), so rows are odd and unaligned at
every size.  Right-hand sides are seeded sine series with random coefficients or smoothed
noise, made on the device; exact() is the discrete solution by sine transforms.
"""
import math

import torch

from paper_2008_03885_amd import mg, rbc, serve

NG, GALERKIN, NG2, G2 = (mg.MG_COARSE_NG, mg.MG_COARSE_GALERKIN, mg.MG_COARSE_NG2,
                         mg.MG_COARSE_G2)
JACOBI, RBJ = mg.MG_SMOOTH_JACOBI, mg.MG_SMOOTH_RBJ
FP64, MIXED = mg.MG_PREC_FP64, mg.MG_PREC_MIXED


def _solve(name, **kw):
    c = dict(kind="solve", dim=2, n=129, order=4, coarse=NG, smoother=JACOBI, nu1=2, nu2=1,
             gamma=1, precision=FP64, inner=4, rhs="series", rtol=1e-10)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest solve of the served sizes: a program that solves many small
        # problems one after another (latency, launches, the one-workgroup tail).
        _solve("solve2d-65-fp64-v21", n=65),
        # One mixed-precision solve of a middle served size, alone on the device.
        _solve("solve2d-513-mixed-v21", n=513, precision=MIXED),
        # The method's own strong combination (Galerkin coarse operators, red-black
        # smoothing) at an ordinary size.
        _solve("solve2d-1025-fp64-galerkin-rb-v21", n=1025, coarse=GALERKIN, smoother=RBJ),
        # The 2D benchmark configuration: 4097^2, fourth order, omega-Jacobi V(2,1).
        _solve("solve2d-4097-fp64-v21", n=4097),
        # A W-cycle: the robust choice of the paper's cycles, bound by its coarse levels.
        _solve("solve2d-2049-fp64-w21", n=2049, gamma=2),
        # A small 3D problem, as in a time step of a small simulation.
        _solve("solve3d-65-fp64-v21", dim=3, n=65),
        # An ordinary 3D problem with the benchmark's Galerkin W(2,2) cycle in FP64.
        _solve("solve3d-257-fp64-galerkin-w22", dim=3, n=257, coarse=GALERKIN, gamma=2, nu2=2),
        # The 3D benchmark configuration of rough data: 513^3, mixed precision V(2,1).
        _solve("solve3d-513-mixed-v21", dim=3, n=513, precision=MIXED, inner=8, rhs="noise"),
        # The largest benchmark configuration: 1025^3, Galerkin W(2,2), mixed precision.
        _solve("solve3d-1025-mixed-galerkin-w22", dim=3, n=1025, coarse=GALERKIN, gamma=2, nu2=2,
               precision=MIXED, inner=1),
        # Red-black coarsening on a small and on the benchmark's grid.
        dict(name="rbc-257-g1-v11", kind="rbc", n=257, coarse=rbc.MG_RBC_G1, gamma=1, nu1=1, nu2=1,
             omega=0.0, rtol=1e-10),
        dict(name="rbc-4097-g1-v11", kind="rbc", n=4097, coarse=rbc.MG_RBC_G1, gamma=1, nu1=1, nu2=1,
             omega=0.0, rtol=1e-10),
        # A burst of requests of all served sizes in the serving benchmark's settings.
        dict(name="serve-48-mixed-v21", kind="serve", count=48, kmin=6, kmax=11, smoother=JACOBI,
             inner=4, rtol=1e-10),
    ]


def draw(rng):
    kind = rng.choices(["solve2d", "solve3d", "rbc", "serve"], [5, 3, 2, 1])[0]
    rtol = float("%.1e" % 10.0 ** -rng.uniform(6.0, 10.0))  # engineering to tight tolerances
    if kind == "solve2d":
        gamma = 2 if rng.random() < 0.25 else 1
        k = rng.randint(6, 11 if gamma == 2 else 12)
        smoother = rng.choice([JACOBI, JACOBI, RBJ])
        return _solve(None, n=2 ** k + 1, gamma=gamma, smoother=smoother,
                      order=rng.choices([4, 2, 6], [6, 1, 1])[0],
                      coarse=rng.choices([NG, GALERKIN, NG2, G2], [4, 3, 1, 1])[0],
                      nu1=rng.choice([1, 2, 2]), nu2=rng.choice([1, 1, 2]),
                      precision=rng.choice([FP64, FP64, MIXED]),
                      inner=2 if smoother == RBJ else 4, rtol=rtol)
    if kind == "solve3d":
        gamma = 2 if rng.random() < 0.4 else 1
        k = rng.randint(5, 8 if gamma == 2 else 9)
        smoother = rng.choice([JACOBI, JACOBI, RBJ])
        precision = rng.choice([FP64, MIXED])
        return _solve(None, dim=3, n=2 ** k + 1, gamma=gamma, smoother=smoother,
                      order=rng.choices([4, 2, 6], [6, 1, 1])[0],
                      coarse=rng.choices([NG, GALERKIN, NG2, G2], [4, 3, 1, 1])[0],
                      nu1=2, nu2=rng.choice([1, 2]), precision=precision,
                      inner=rng.choice([1, 2, 4]), rhs=rng.choice(["series", "noise"]),
                      rtol=rtol)
    if kind == "rbc":
        return dict(kind="rbc", n=2 ** rng.randint(6, 12) + 1,
                    coarse=rng.choice([rbc.MG_RBC_G1, rbc.MG_RBC_G1, rbc.MG_RBC_GN, rbc.MG_RBC_NG]),
                    gamma=1, nu1=rng.choice([1, 1, 2]), nu2=1,
                    omega=rng.choice([0.0, 0.0, 1.1, 1.2]), rtol=rtol)
    kmin = rng.randint(6, 8)
    smoother = rng.choice([JACOBI, JACOBI, RBJ])
    return dict(kind="serve", count=rng.randint(6, 60), kmin=kmin, kmax=rng.randint(kmin + 1, 11),
                smoother=smoother, inner=2 if smoother == RBJ else 4, rtol=rtol)


# ------------------------------------------------------------------------- inputs ----

def _device():
    return torch.device("cuda") if torch.cuda.is_available() else torch.device("cpu")


def _sin_rows(K, n, dev):
    """sin(pi k i / (n-1)) for k = 1..K (rows), i = 0..n-1, the argument reduced in whole numbers."""
    k = torch.arange(1, K + 1, device=dev).unsqueeze(1)
    i = torch.arange(n, device=dev).unsqueeze(0)
    p = (k * i) % (2 * (n - 1))
    s = torch.sin(p.to(torch.float64) * (math.pi / (n - 1)))
    s[p % (n - 1) == 0] = 0.0
    return s


def _along(t, m, axis):
    """t with axis `axis` contracted with the rows' index of m (K x n)."""
    return torch.tensordot(t, m, dims=([axis], [0])).movedim(-1, axis)


def _series(coeffs, n):
    """sum_k c_k prod_a sin(k_a pi x_a) on the n-point grid."""
    t = coeffs
    for a in range(coeffs.dim()):
        t = _along(t, _sin_rows(coeffs.shape[a], n, coeffs.device), a)
    return t.contiguous()


def _coeffs(dim, n, seed, dev):
    """Random coefficients of a smooth right-hand side: 2D g/|k| up to 64 modes an axis,
    3D N(0,1) up to 8."""
    K = min(64, (n - 1) // 4) if dim == 2 else min(8, n - 2)
    g = torch.Generator().manual_seed(int(seed))
    c = torch.randn((K,) * dim, generator=g, dtype=torch.float64)
    if dim == 2:
        k = torch.arange(1, K + 1, dtype=torch.float64)
        c = c / torch.sqrt(k[:, None] ** 2 + k[None, :] ** 2)
    return c.to(dev)


def _noise(dim, n, seed, dev):
    """Uniform noise with a zero boundary, three neighbour averages."""
    g = torch.Generator(device=dev).manual_seed(int(seed))
    inner = (slice(1, n - 1),) * dim
    f = torch.zeros((n,) * dim, dtype=torch.float64, device=dev)
    f[inner] = torch.rand((n - 2,) * dim, generator=g, dtype=torch.float64, device=dev) * 2.0 - 1.0
    for _ in range(3):
        s = None
        for a in range(dim):
            for o in (0, 2):
                sl = [slice(1, n - 1)] * dim
                sl[a] = slice(o, o + n - 2)
                s = f[tuple(sl)].clone() if s is None else s.add_(f[tuple(sl)])
        f[inner] = s.div_(2.0 * dim)
    return f


def _rhs(case, seed, dev):
    if case.get("rhs") == "noise":
        return _noise(case["dim"], case["n"], seed, dev)
    return _series(_coeffs(case.get("dim", 2), case["n"], seed, dev), case["n"])


def _serve_sides(case):
    """The burst's sides: every side of the range in turn, in a shuffled order."""
    ks = [case["kmin"] + i % (case["kmax"] - case["kmin"] + 1) for i in range(case["count"])]
    g = torch.Generator().manual_seed(17)
    return [2 ** ks[j] + 1 for j in torch.randperm(len(ks), generator=g).tolist()]


# ------------------------------------------------------------------ prepare and run ----

def _rbc_levels(n):
    """The fewest levels whose last one the coarsest solve takes."""
    def unknowns(l):
        inner = ((n - 1) // 2 ** (l // 2) - 1) ** 2
        return inner if l % 2 == 0 else (inner + 1) // 2
    levels = 2
    while unknowns(levels - 1) > rbc.MG_RBC_MAX_COARSEST:
        levels += 1
    return levels


class _RbcSolve:
    """A red-black coarsening handle on torch's current stream."""

    def __init__(self, case):
        self.max_cycles = 60
        cfg = rbc.make_config(n=case["n"], levels=_rbc_levels(case["n"]), coarse=case["coarse"],
                              gamma=case["gamma"], nu1=case["nu1"], nu2=case["nu2"],
                              omega=case["omega"], rtol=case["rtol"], max_cycles=self.max_cycles)
        self.h = rbc.setup(cfg, torch.cuda.current_stream().cuda_stream)

    def solve(self, f, u):
        rbc.solve(self.h, f.data_ptr(), u.data_ptr(), self.max_cycles)

    def __del__(self):
        if getattr(self, "h", None):
            rbc.destroy(self.h)
            self.h = None


def prepare(case, seed):
    dev = torch.device("cuda")
    if case["kind"] == "serve":
        server = serve.Server(4 << 30, 16, 1, 3, n=65, dim=2, coarse=NG, gamma=1, nu1=2, nu2=1,
                              precision=MIXED, rtol=case["rtol"], max_cycles=30,
                              inner_cycles=case["inner"], smoother=case["smoother"])
        fs = [_series(_coeffs(2, n, seed * 1000 + i, dev), n)
              for i, n in enumerate(_serve_sides(case))]
        torch.cuda.synchronize()  # the server reads f on streams of its own
        return {"kind": "serve", "handle": server, "f": fs, "u": [torch.empty_like(f) for f in fs]}
    f = _rhs(case, seed, dev)
    if case["kind"] == "rbc":
        handle = _RbcSolve(case)
    else:
        handle = mg.Solver(dim=case["dim"], n=case["n"], order=case["order"], coarse=case["coarse"],
                           smoother=case["smoother"], nu1=case["nu1"], nu2=case["nu2"],
                           gamma=case["gamma"], precision=case["precision"],
                           inner_cycles=case["inner"], rtol=case["rtol"], max_cycles=100)
    return {"kind": case["kind"], "handle": handle, "f": f, "u": torch.zeros_like(f)}


def run(state):
    h, f, u = state["handle"], state["f"], state["u"]
    if state["kind"] == "serve":
        for tag, (fi, ui) in enumerate(zip(f, u)):
            if h.submit(tag, fi, ui) != mg.MG_OK:
                raise RuntimeError(mg.last_error())
        h.wait_all(len(f))
        return u
    u.zero_()
    h.solve(f, u)
    return u


# ------------------------------------------------------------------- work and exact ----

def _cycles(case):
    """About how many cycles a solve to 1e-10 takes (Fourier analysis and experience)."""
    if case["kind"] == "rbc":
        return 8
    if case["smoother"] == RBJ:
        return 7 if case.get("dim", 2) == 2 else 8
    if case.get("rhs") == "noise":
        return 24
    return 10 if case.get("coarse", NG) in (GALERKIN, G2) else 18


def _solve_work(dim, n, gamma, cycles, outer, es, flops):
    """One fused pass before and one after the coarse correction on every level visit, each
    reading the iterate and the right-hand side and writing the iterate (plus the coarse
    transfer); a refinement step also reads f and u and writes u in FP64."""
    pts = float(n) ** dim
    ratio = gamma / 2.0 ** dim
    visits = 1.0 / (1.0 - ratio)
    per = 2.0 * (3.0 + 0.5 ** dim) * es * visits
    return {"bytes": pts * (cycles * per + outer * 24.0), "flops": pts * cycles * flops * visits}


def work(case):
    if case["kind"] == "serve":
        parts = [_solve_work(2, n, 1, 18, 5, 4, 90.0) for n in _serve_sides(case)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    if case["kind"] == "rbc":  # every level holds half the points of the one above
        w = _solve_work(1, case["n"], 1, _cycles(case), 0, 8, 50.0)
        return {k: v * case["n"] for k, v in w.items()}
    es = 4 if case["precision"] == MIXED else 8
    cyc = _cycles(case)
    outer = -(-cyc // case["inner"]) if case["precision"] == MIXED else 0
    return _solve_work(case["dim"], case["n"], case["gamma"], cyc, outer, es,
                       10.0 * case["dim"] * (case["nu1"] + case["nu2"] + 1))


def _eig(n, order, K, dev):
    """The 1D symbol at theta = k pi h, k = 1..K."""
    h = 1.0 / (n - 1)
    s = torch.sin(torch.arange(1, K + 1, device=dev, dtype=torch.float64) * (math.pi * h / 2.0)) ** 2
    v = s
    if order >= 4:
        v = v + s * s / 3.0
    if order >= 6:
        v = v + 8.0 * s ** 3 / 45.0
    return v * (4.0 / h ** 2)


def _sum_axes(e, dim):
    t = e
    for _ in range(dim - 1):
        t = t.unsqueeze(-1) + e
    return t


def _exact_series(coeffs, n, order):
    lam = _sum_axes(_eig(n, order, coeffs.shape[0], coeffs.device), coeffs.dim())
    return _series(coeffs / lam, n)


def _exact_transform(f, order):
    """The discrete solution for any right-hand side: sine transforms as matrix products."""
    dim, n = f.dim(), f.shape[0]
    S = _sin_rows(n - 2, n, f.device)[:, 1:-1].contiguous()
    t = f[(slice(1, n - 1),) * dim]
    for a in range(dim):
        t = _along(t, S, a)
    t = t / _sum_axes(_eig(n, order, n - 2, f.device), dim) * (2.0 / (n - 1)) ** dim
    for a in range(dim):
        t = _along(t, S, a)
    u = torch.zeros_like(f)
    u[(slice(1, n - 1),) * dim] = t
    return u


def exact(case, seed):
    dev = _device()
    if case["kind"] == "serve":
        return [_exact_series(_coeffs(2, n, seed * 1000 + i, dev), n, 4)
                for i, n in enumerate(_serve_sides(case))]
    if case.get("rhs") == "noise":
        return _exact_transform(_rhs(case, seed, dev), case["order"])
    c = _coeffs(case.get("dim", 2), case["n"], seed, dev)
    return _exact_series(c, case["n"], case.get("order", 2))
