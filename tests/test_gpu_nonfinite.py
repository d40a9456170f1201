"""A residual evaluation that is not a number ends a solve with HOM_E_NAN: it is
never taken for a small one. The macro strains are finite, the fields they give
are not (an infinite trace in the law: inf - inf)."""
import numpy as np
import pytest

from paper_2109_14403_amd import hom
from paper_2109_14403_amd import workloads as W

pytestmark = pytest.mark.gpu

HUGE = {hom.FP64: 1e306, hom.FP32: 1e60}
GOOD = [1e-3, -2e-4, 3e-4, 1e-4, -5e-5, 2e-4]


def cell(shape, laws):
    img = (np.random.default_rng(3).random(shape) < 0.3).astype(np.uint8)
    return img, [W.pa66(), W.e_glass()] if laws == "pa66" else [W.small_sphere_matrix(), W.small_sphere_inclusion()]


# (16, 16, 16): a plane of one kx in LDS; (48, 48, 16): separate y and z passes
@pytest.mark.parametrize("laws", ["elastic", "pa66"])
@pytest.mark.parametrize("shape", [(16, 16, 16), (48, 48, 16)])
@pytest.mark.parametrize("precision", [hom.FP64, hom.FP32])
@pytest.mark.parametrize("scheme", [hom.SCHEME_NEWTON_CG, hom.SCHEME_BASIC])
def test_not_a_number_is_no_convergence(scheme, precision, shape, laws):
    img, lw = cell(shape, laws)
    opts = dict(scheme=scheme, precision=precision, tol=1e-6)
    with hom.Context(img, lw, **opts) as ctx:
        bad = ctx.solve_increment([HUGE[precision]] * 3 + [0.0] * 3, 300.0, [0.0] * 3, 1.0, check=False)
        assert bad["status"] == hom.HOM_E_NAN and bad["rc"] == hom.HOM_E_NAN
        # nothing was committed
        got = ctx.solve_increment(GOOD, 300.0, [0.0] * 3, 1.0)
    with hom.Context(img, lw, **opts) as ctx:
        ref = ctx.solve_increment(GOOD, 300.0, [0.0] * 3, 1.0)
    assert np.array_equal(got["stress"], ref["stress"])
