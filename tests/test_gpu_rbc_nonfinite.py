"""mg_rbc_solve on data that are not finite (GPU): MG_ENUMERIC before any cycle, u untouched,
and the handle solves the next problem."""
import numpy as np
import pytest

from gpu_util import dev, host
from test_gpu_rbc import Pair, _grid
from paper_2008_03885_amd import mg, rbc

pytestmark = pytest.mark.gpu


# the level-0 pass, the tail as the whole cycle, and the separate kernels form the norm
@pytest.mark.parametrize("n,levels,passes", [(129, 8, "1"), (65, 5, "1"), (129, 8, "0")])
@pytest.mark.parametrize("where,value", [("f", np.nan), ("f", np.inf), ("f", -np.inf), ("u", np.nan), ("u", np.inf)])
def test_nonfinite_data(n, levels, passes, where, value, monkeypatch):
    monkeypatch.setenv("MG_RBC_PASSES", passes)
    f, u0 = _grid(n, 90) * (n - 1) ** 2, _grid(n, 91)
    good = f.copy()
    (f if where == "f" else u0)[n // 2, n // 2 + 1] = value
    P = Pair(n, levels, "G1", max_cycles=40)
    try:
        fd, ud = dev(f), dev(u0)
        st, k, hist = rbc.solve(P.h, fd.data_ptr(), ud.data_ptr(), 40)
        assert (st, k) == (mg.MG_ENUMERIC, 0) and not np.isfinite(hist[0])
        assert "not finite" in mg.last_error()
        assert np.array_equal(host(ud), u0, equal_nan=True)
        gd, ud = dev(good), dev(np.zeros((n, n)))
        st, k, hist = rbc.solve(P.h, gd.data_ptr(), ud.data_ptr(), 40)
        assert st == mg.MG_OK and 0 < k < 40 and hist[-1] <= 1e-10 * hist[0]
    finally:
        P.close()
