"""The one-workgroup 2D tail of the levels 65^2 .. 9^2 (GPU): whole cycles whose tail starts
at each of its sides, for every operator shape, smoother and cycle that it runs, against the
oracle (FP64, the bar of the whole-cycle tests) and against the per-level kernels (FP32)."""
import numpy as np
import pytest

from gpu_util import Handle, dev, host, rand_grid
from paper_2008_03885_amd import mg

pytestmark = pytest.mark.gpu

# n = 17, 33, 65: the level-0 iterate itself is in the tail; 129: the tail is visited
CASES = [
    # n, order, coarse, smoother, gamma, nu1, nu2, prolong
    (17, 4, 0, 0, 1, 2, 1, 3), (17, 6, 1, 1, 2, 1, 2, 1),
    (33, 4, 0, 0, 2, 2, 1, 3), (33, 4, 1, 0, 2, 1, 1, 3), (33, 2, 0, 1, 1, 0, 1, 1),
    (65, 4, 0, 0, 1, 2, 1, 3), (65, 4, 0, 1, 2, 3, 0, 3), (65, 4, 1, 0, 2, 2, 2, 3),
    (65, 6, 0, 0, 1, 2, 1, 3), (65, 2, 3, 1, 1, 1, 1, 1), (65, 4, 2, 0, 2, 0, 2, 3),
    (129, 4, 0, 0, 2, 2, 1, 3), (129, 4, 1, 1, 2, 2, 1, 3), (129, 6, 3, 0, 1, 5, 1, 3),
]


def _handle(case, **kw):
    n, order, coarse, smoother, gamma, nu1, nu2, prolong = case
    return Handle(2, n, order=order, coarse=coarse, smoother=smoother, gamma=gamma, nu1=nu1, nu2=nu2,
                  prolong=prolong, **kw)


@pytest.mark.parametrize("case", CASES)
def test_cycles_match_oracle(case):
    H = _handle(case)
    try:
        n = case[0]
        f, u0 = rand_grid(n, 2, 11), rand_grid(n, 2, 12)
        fd, ud = dev(f), dev(u0)
        mg.mg_run_cycles(H.h, fd.data_ptr(), ud.data_ptr(), 3)
        u_ref = u0.copy()
        H.oracle.solve(u_ref, f, rtol=0.0, max_cycles=3)
        u = host(ud)
        assert np.linalg.norm(u - u_ref) <= 1e-12 * np.linalg.norm(u_ref)
        assert not u[0].any() and not u[-1].any() and not u[:, 0].any() and not u[:, -1].any()
    finally:
        H.close()


@pytest.mark.parametrize("top", ["17", "33", "65"])
@pytest.mark.parametrize("coarse,smoother,gamma", [(0, 0, 1), (1, 0, 2), (0, 1, 2)])
def test_fp32_cycle_against_level_kernels(top, coarse, smoother, gamma, monkeypatch):
    """One refinement step of one FP32 cycle from each tail side against the same cycle by
    the per-level kernels: FP32 rounding of about 1e2 sums, 1e2 x 6e-8 of the largest value."""
    n = 129
    f = rand_grid(n, 2, 13)
    out = []
    for t in (top, "0"):
        monkeypatch.setenv("MG_TAIL_N", t)
        H = _handle((n, 4, coarse, smoother, gamma, 2, 1, 3), precision=1, inner_cycles=1)
        try:
            fd, ud = dev(f), dev(np.zeros_like(f))
            mg.mg_run_cycles(H.h, fd.data_ptr(), ud.data_ptr(), 1)
            out.append(host(ud))
        finally:
            H.close()
    assert np.abs(out[0] - out[1]).max() <= 6e-6 * np.abs(out[1]).max()
