"""Stress control from a stress-free start: at the reference temperature and zero
strain the stress field is exactly zero, and the prescribed mean stress is all
the residual there is. Bounds: those of the mixed loads in FP64 and FP32 (1e-6
and 2e-6 of the largest component)."""
import numpy as np
import pytest

from oracle import solver
from paper_2109_14403_amd import hom
from paper_2109_14403_amd import workloads as W

pytestmark = pytest.mark.gpu

ALL = [True] * 6
LATERAL = [False, True, True, True, True, True]


@pytest.mark.parametrize("precision,bound", [(hom.FP64, 1e-6), (hom.FP32, 2e-6)])
@pytest.mark.parametrize("mask", [ALL, LATERAL])
@pytest.mark.parametrize("shape,laws", [((16, 16, 16), "elastic"), ((48, 48, 16), "elastic"), ((16, 16, 16), "pa66")])
def test_prescribed_stress_on_a_stress_free_cell(shape, laws, mask, precision, bound):
    img = (np.random.default_rng(5).random(shape) < 0.3).astype(np.uint8)
    lw = [W.pa66(293.0), W.e_glass(293.0)] if laws == "pa66" else [W.small_sphere_matrix(), W.small_sphere_inclusion()]
    stress = [0.0, 4.0, -2.0, 1.0, 0.5, -1.0] if mask is LATERAL else [6.0, 4.0, -2.0, 1.0, 0.5, -1.0]
    o = solver.Cell(img, lw).solve_load([0.0] * 6, stress, mask, 293.0, [0.0] * 3, 1.0, tol=1e-11)
    with hom.Context(img, lw, precision=precision, tol=1e-10 if precision == hom.FP64 else 1e-6) as ctx:
        g = ctx.solve_load([0.0] * 6, 293.0, [0.0] * 3, 1.0, stress=stress, stress_mask=mask)
    for k in ("stress", "strain"):
        err = np.abs(g[k] - o[k]).max() / np.abs(o[k]).max()
        print(f"{shape} {laws} precision {precision} {k}: {err:.2e}, newton {g['newton_iters']}", flush=True)
        assert err <= bound
