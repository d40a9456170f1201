"""The passes of a Newton-CG iteration at every transform length on every axis:
an increment of a two-phase cell (mechanics and conduction) against the oracle.
The lengths select the kernels' instantiations and, with the grid's other two
axes, the way the y and z transforms are split over work-groups."""
import numpy as np
import pytest

from oracle import solver
from paper_2109_14403_amd import hom
from paper_2109_14403_amd import workloads as W

pytestmark = pytest.mark.gpu

# FP64: a relative residual of 1e-10 bounds the error of the effective stress
# by its contrast-weighted size; FP32: the stated bound of the effective outputs
TOL = {hom.FP64: 1e-8, hom.FP32: 2e-6}
SHAPES = sorted({tuple(np.roll((n, 16, 16), k)) for n in (16, 24, 32, 48, 64, 96, 128, 256) for k in range(3)}
                | {(24, 48, 32), (32, 32, 32), (48, 48, 24), (64, 48, 16), (24, 128, 16)})


@pytest.mark.parametrize("precision", [hom.FP64, hom.FP32])
@pytest.mark.parametrize("shape", SHAPES)
def test_increment_matches_oracle(shape, precision):
    rng = np.random.default_rng(sum(shape) + precision)
    img = (rng.random(shape) < 0.3).astype(np.uint8)
    laws = [W.small_sphere_matrix(), W.small_sphere_inclusion()]
    strain = np.array([4e-3, -1e-3, 2e-3, 1e-3, -2e-3, 3e-3])
    grad = [1.0, -0.5, 0.25]
    o = solver.Cell(img, laws).solve_increment(strain, 323.0, grad, 2.0, tol=1e-11)
    with hom.Context(img, laws, precision=precision, tol=1e-10 if precision == hom.FP64 else 1e-6) as ctx:
        for _ in range(2):  # the second increment starts from the solution of the first
            g = ctx.solve_increment(strain, 323.0, grad, 2.0)
            for k in ("stress", "heat_flux"):
                err = np.abs(g[k] - o[k]).max() / np.abs(o[k]).max()
                print(f"{shape} precision {precision} {k}: {err:.2e}", flush=True)
                assert err <= TOL[precision]


# planes of these sizes are transformed in LDS only when a launch has enough of
# them: the batch takes the plane pass, a single cell the separate passes
@pytest.mark.parametrize("shape,count,precision", [((48, 48, 16), 15, hom.FP32), ((32, 32, 16), 15, hom.FP64),
                                                   ((24, 48, 32), 8, hom.FP64)])
def test_batch_of_large_planes_equals_single_cells(shape, count, precision):
    rng = np.random.default_rng(count)
    imgs = [(rng.random(shape) < 0.3).astype(np.uint8) for _ in range(count)]
    laws = [W.small_sphere_matrix(), W.small_sphere_inclusion()]
    strains = rng.normal(size=(count, 6)) * 2e-3
    grads = rng.normal(size=(count, 3))
    opts = dict(precision=precision, tol=1e-10 if precision == hom.FP64 else 1e-6)
    with hom.Batch(imgs, laws, **opts) as b:
        r = b.solve_increment(strains, [323.0] * count, grads, [2.0] * count)
    for i in (0, count // 2, count - 1):
        with hom.Context(imgs[i], laws, **opts) as ctx:
            g = ctx.solve_increment(strains[i], 323.0, grads[i], 2.0)
        for k in ("stress", "heat_flux"):
            err = np.abs(r[i][k] - g[k]).max() / np.abs(g[k]).max()
            print(f"{shape} problem {i} precision {precision} {k}: {err:.2e}", flush=True)
            assert err <= 2 * TOL[precision]


# The fixed-point scheme contracts by (k - 1) / (k + 1) for a stiffness contrast
# k = 23: the strain is off by at most tol (k + 1) / 2 where it stops, the stress
# by k times as much, relative to the effective one.
BASIC = 23 * 12
BASIC_TOL = {hom.FP64: 1e-10, hom.FP32: 1e-6}


@pytest.mark.parametrize("precision", [hom.FP64, hom.FP32])
@pytest.mark.parametrize("shape", [(16, 16, 16), (24, 16, 32), (16, 48, 64), (96, 16, 24), (128, 16, 16), (48, 48, 48),
                                   (16, 16, 256)])
def test_fixed_point_increment_matches_oracle(shape, precision):
    """The x pass of the fixed-point scheme (plane pass and separate passes,
    few and many lines): an increment with a temperature gradient, twice, alone
    and in a batch whose problems end after different numbers of iterations."""
    rng = np.random.default_rng(sum(shape) + 7 * precision)
    img = (rng.random(shape) < 0.3).astype(np.uint8)
    laws = [W.small_sphere_matrix(), W.small_sphere_inclusion()]
    strain = np.array([4e-3, -1e-3, 2e-3, 1e-3, -2e-3, 3e-3])
    grad = [1.0, -0.5, 0.25]
    tol = BASIC_TOL[precision]
    opts = dict(scheme=hom.SCHEME_BASIC, precision=precision, tol=tol)
    o = solver.Cell(img, laws).solve_increment(strain, 323.0, grad, 2.0, tol=1e-11)
    with hom.Context(img, laws, **opts) as ctx:
        for _ in range(2):
            g = ctx.solve_increment(strain, 323.0, grad, 2.0)
            for k in ("stress", "heat_flux"):
                err = np.abs(g[k] - o[k]).max() / np.abs(o[k]).max()
                print(f"{shape} precision {precision} {k}: {err:.2e}", flush=True)
                assert err <= BASIC * tol
    with hom.Batch([img, np.zeros_like(img), img], laws, **opts) as b:
        r = b.solve_increment([strain, strain, 3 * strain], [323.0] * 3, [grad] * 3, [2.0] * 3)
    assert r[1]["newton_iters"] < r[0]["newton_iters"]
    err = np.abs(r[0]["stress"] - o["stress"]).max() / np.abs(o["stress"]).max()
    assert err <= BASIC * tol
