"""Red-black coarsening levels as one pass per half visit (GPU): cycles and solves against
the separate partial-step, restriction and interpolation kernels (MG_RBC_PASSES=0) and the
oracle.  Bar: 1e-12 of the largest value, that of the other red-black coarsening tests."""
import numpy as np
import pytest

from gpu_util import dev, host, torch
from test_gpu_rbc import Pair, _close, _grid
from paper_2008_03885_amd import mg, rbc

pytestmark = pytest.mark.gpu

CASES = [
    # n, levels, coarse, gamma, nu1, nu2, omega: MG_RBC_TAIL=0, so that passes run down to 17^2
    (17, 4, "G1", 1, 1, 1, 1.0), (33, 6, "NG", 1, 1, 1, 1.0), (65, 7, "G1", 2, 1, 1, 1.0),
    (129, 8, "GN", 1, 2, 1, 1.2), (129, 9, "G1", 2, 2, 2, 0.9), (257, 11, "G1", 1, 1, 3, 1.1),
    (1025, 14, "NG", 1, 3, 1, 1.0), (2049, 15, "G1", 1, 1, 1, 1.0),
]


@pytest.mark.parametrize("n,levels,coarse,gamma,nu1,nu2,omega", CASES)
def test_passes_equal_separate_kernels(n, levels, coarse, gamma, nu1, nu2, omega, monkeypatch):
    monkeypatch.setenv("MG_RBC_TAIL", "0")
    f, u0 = _grid(n, 40 + n) * (n - 1) ** 2, _grid(n, 41 + n)
    u0[0, :], u0[:, -1] = 0.5, np.linspace(0.0, 1.0, n)  # Dirichlet values are kept
    f[0, :] = f[:, 0] = np.nan  # boundary entries of f are ignored
    out = []
    for env in ("0", "1"):
        monkeypatch.setenv("MG_RBC_PASSES", env)
        P = Pair(n, levels, coarse, gamma, nu1, nu2, omega)
        try:
            fd, ud = dev(f), dev(u0)
            rbc.cycles(P.h, fd.data_ptr(), ud.data_ptr(), 2)
            out.append(host(ud))
        finally:
            P.close()
    _close(out[1], out[0], "passes against separate kernels")
    assert np.array_equal(out[1][0], u0[0]) and np.array_equal(out[1][:, -1], u0[:, -1])


@pytest.mark.parametrize("n,levels,nu1,nu2,gamma,max_cycles", [(65, 7, 1, 1, 1, 40), (257, 9, 2, 1, 2, 40),
                                                               (513, 11, 2, 2, 1, 40), (129, 8, 1, 1, 1, 3)])
def test_solve_with_the_stopping_rule_on_the_device(n, levels, nu1, nu2, gamma, max_cycles, monkeypatch):
    """The same cycle count, history and solution as the solve that synchronizes after every
    cycle, also when it ends at max_cycles; a second solve on the handle starts afresh."""
    f = _grid(n, 50 + n) * (n - 1) ** 2
    out = []
    for env in ("0", "1"):
        monkeypatch.setenv("MG_RBC_PASSES", env)
        P = Pair(n, levels, "G1", gamma, nu1, nu2, 1.0, max_cycles=max_cycles)
        try:
            for _ in range(2):
                fd, ud = dev(f), dev(np.zeros((n, n)))
                st, k, hist = rbc.solve(P.h, fd.data_ptr(), ud.data_ptr(), max_cycles)
            out.append((st, k, np.array(hist), host(ud)))
        finally:
            P.close()
    (s0, k0, h0, u0), (s1, k1, h1, u1) = out
    assert (s0, k0) == (s1, k1) and s0 == (mg.MG_OK if max_cycles == 40 else mg.MG_ENOCONV)
    assert np.all(np.abs(h1 - h0) <= 1e-9 * h0 + 1e-13 * h0[0])
    _close(u1, u0, "solution")


def test_solve_from_zero_and_nonfinite_data():
    """A zero residual stops at once with u untouched; a residual that turns infinite is
    reported."""
    P = Pair(65, 7, "G1")
    try:
        z = torch().zeros(65, 65, dtype=torch().float64, device="cuda")
        u = z.clone()
        assert rbc.solve(P.h, z.data_ptr(), u.data_ptr(), 40)[:2] == (mg.MG_OK, 0)
        assert not u.any()
        f = z.clone()
        f[30, 31] = 1e308
        st, k, hist = rbc.solve(P.h, f.data_ptr(), u.data_ptr(), 40)
        # the squared norm overflows: not a decrease, so no cycle runs
        assert (st, k) == (mg.MG_OK, 0) and not np.isfinite(hist[0])
    finally:
        P.close()


TAIL_CASES = [
    # n, levels (the last one 17^2), coarse, gamma, nu1, nu2, omega
    (33, 3, "G1", 1, 1, 1, 1.0), (33, 3, "NG", 2, 2, 1, 1.2), (65, 5, "G1", 2, 1, 1, 1.0), (65, 5, "NG", 1, 0, 2, 1.0),
    (65, 5, "GN", 1, 2, 0, 0.9), (129, 7, "G1", 2, 2, 2, 1.1), (257, 9, "NG", 2, 1, 1, 1.0), (513, 11, "G1", 1, 1, 2, 1.0),
]


@pytest.mark.parametrize("side", ["33", "65"])
@pytest.mark.parametrize("n,levels,coarse,gamma,nu1,nu2,omega", TAIL_CASES)
def test_lds_tail_equals_per_level_kernels(n, levels, coarse, gamma, nu1, nu2, omega, side, monkeypatch):
    """The tail resident in LDS (hierarchies that end in the standard 17^2 level) against the
    separate kernels down to the dense coarsest solve; with n = 33 and 65 the whole cycle is
    the tail, Dirichlet values in u and junk in f's boundary included."""
    f, u0 = _grid(n, 60 + n) * (n - 1) ** 2, _grid(n, 61 + n)
    u0[0, :], u0[-1, :], u0[:, 0], u0[:, -1] = 0.5, np.linspace(0.5, 2.0, n), 0.25, np.linspace(1.0, 0.0, n)
    f[0, :] = f[:, 0] = f[-1, :] = f[:, -1] = np.nan
    out = []
    monkeypatch.setenv("MG_RBC_PASSES", "0")
    for env in ("0", side):
        monkeypatch.setenv("MG_RBC_TAIL", env)
        P = Pair(n, levels, coarse, gamma, nu1, nu2, omega)
        try:
            fd, ud = dev(f), dev(u0)
            rbc.cycles(P.h, fd.data_ptr(), ud.data_ptr(), 2)
            out.append(host(ud))
        finally:
            P.close()
    _close(out[1], out[0], "tail against separate kernels")
    for edge in (np.s_[0, :], np.s_[-1, :], np.s_[:, 0], np.s_[:, -1]):
        assert np.array_equal(out[1][edge], u0[edge])


def test_solve_whose_cycle_is_the_tail():
    """n = 65 with the 17^2 coarsest level: every cycle one launch, checks on the device."""
    P = Pair(65, 5, "G1", 1, 1, 1, 1.0, max_cycles=40)
    try:
        f = _grid(65, 77) * 64.0 ** 2
        fd, ud = dev(f), dev(np.zeros((65, 65)))
        st, k, hist = rbc.solve(P.h, fd.data_ptr(), ud.data_ptr(), 40)
        assert st == mg.MG_OK and len(hist) == k + 1 and hist[-1] <= 1e-10 * hist[0] < hist[-2]
        u = np.zeros((65, 65))
        for _ in range(k):
            u = P.o.cycle(f, u)
        _close(host(ud), u, "solution")
    finally:
        P.close()
