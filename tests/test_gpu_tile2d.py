"""Block sizes of the 2D tile passes: a launch takes 1024 threads per block up to 600 blocks
and 256 beyond.  A level of 257 points has 153 tiles per system, so batches of up to three
systems take the wide blocks and four or more the narrow ones; a system's result and its
defect norms have to be the same bits on both sides of that line, for the cross and the
separable operator, and the solution right to its residual."""
import numpy as np
import pytest

from paper_2008_03885_amd import inputs, mg
from test_gpu_serve import _check_exact, _rhs, _serve, _solo

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("coarse,smoother", [(0, mg.MG_SMOOTH_JACOBI), (1, mg.MG_SMOOTH_JACOBI),
                                             (1, mg.MG_SMOOTH_RBJ)])
@pytest.mark.parametrize("precision", [mg.MG_PREC_FP64, mg.MG_PREC_MIXED])
@pytest.mark.parametrize("slots", [3, 4])
def test_batch_equals_standalone_on_both_sides_of_the_line(slots, precision, coarse, smoother):
    n = 257
    reqs = [(i, n, _rhs(n, inputs.SEED_BASE + 1700 + i)) for i in range(slots)]
    over = dict(precision=precision, coarse=coarse, smoother=smoother, max_cycles=60)
    out, stats = _serve(reqs, max_slots=slots, **over)
    assert stats["completed"] == slots
    for tag, _, f in reqs:
        ref, st, hist = _solo(n, f, **over)
        u, c = out[tag]
        assert c.status == mg.MG_OK and st == mg.MG_OK
        assert np.array_equal(u, ref)
        assert c.result.hist() == hist
        _check_exact(u, f, "tile %d" % tag)
