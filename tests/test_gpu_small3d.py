"""The direct kernels of the small rediscretized 3D levels (up to 65^3) against the marching
kernels, which a forced tile shape keeps, on every step.  Both evaluate
the same sums; where the order of an interpolation or weighting differs, a value moves by a
few units in the last place of its largest term, of which 32 are allowed."""
import numpy as np
import pytest

from gpu_util import Handle, dev, host, rand_grid
from paper_2008_03885_amd import mg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp32", [0, 1])
@pytest.mark.parametrize("n,prolong", [(9, 3), (17, 1), (33, 3), (33, 1), (65, 3), (65, 1)])
def test_direct_equals_marching(n, prolong, fp32, monkeypatch):
    H = Handle(3, n, prolong=prolong, n_coarsest=5)
    try:
        n_l, s = H.level(0)
        assert n_l == n
        d = s[(s.shape[0] // 2,) * 3]
        nc = (n - 1) // 2 + 1
        u, f, v = rand_grid(n, 3, 61), rand_grid(n, 3, 62) * d, rand_grid(nc, 3, 63)
        ud, fd, vd = dev(u, fp32), dev(f, fp32), dev(v, fp32)

        def steps():
            out = {}

            def run(name, side, call):
                o = dev(np.full((side,) * 3, np.nan), fp32)
                call(o.data_ptr())
                out[name] = host(o)

            run("smooth", n, lambda o: mg.mg_kernel_smooth(H.h, 0, fp32, fd.data_ptr(), ud.data_ptr(), o))
            for c in (0, 1, 2):
                run("colour %d" % c, n, lambda o: mg.mg_kernel_smooth_colour(
                    H.h, 0, fp32, c, fd.data_ptr(), ud.data_ptr(), o))
            run("residual", n, lambda o: mg.mg_kernel_residual(H.h, 0, fp32, fd.data_ptr(), ud.data_ptr(), o))
            run("restrict", nc, lambda o: mg.mg_kernel_residual_restrict(
                H.h, 0, fp32, fd.data_ptr(), ud.data_ptr(), o))
            run("prolong", n, lambda o: mg.mg_kernel_prolong_correct(
                H.h, 0, fp32, vd.data_ptr(), ud.data_ptr(), o))
            return out

        got = steps()
        for var in ("MG_X3_W", "MG_P3_W", "MG_XRR_TALL"):
            monkeypatch.setenv(var, "0")
        ref = steps()
        eps = np.finfo(np.float32 if fp32 else np.float64).eps
        big = np.abs(u).max() + np.abs(f).max() / d + np.abs(v).max()
        for name in got:
            scale = big * (d if name in ("residual", "restrict") else 1.0)
            assert np.abs(got[name] - ref[name]).max() <= 32 * eps * scale, name
    finally:
        H.close()
