"""The autotuner on grids whose y and z transforms are passes of their own (a
group whose planes are transformed in LDS is not tuned)."""
import numpy as np
import pytest

from paper_2109_14403_amd import hom
from paper_2109_14403_amd import workloads as W

pytestmark = pytest.mark.gpu

PASSES = ("y_mech", "z_mech", "y_thermal", "z_thermal")
DEFAULT = {"tile": 4, "plan": 0}
# two solves to the tolerance: FP64 by the contrast-weighted size of the
# residual, FP32 twice the bound of the effective outputs
TOL, BOUND = {hom.FP64: 1e-10, hom.FP32: 1e-6}, {hom.FP64: 1e-8, hom.FP32: 4e-6}


@pytest.mark.parametrize("scheme,discretization", [(hom.SCHEME_NEWTON_CG, hom.DISC_COLLOCATION),
                                                   (hom.SCHEME_NEWTON_CG, hom.DISC_ROTATED),
                                                   (hom.SCHEME_BASIC, hom.DISC_COLLOCATION)])
@pytest.mark.parametrize("precision", [hom.FP64, hom.FP32])
@pytest.mark.parametrize("laws", ["elastic", "pa66"])
def test_tuned_schedules_solve_alike(laws, scheme, precision, discretization):
    rng = np.random.default_rng(11)
    imgs = [(rng.random(s) < 0.3).astype(np.uint8) for s in ((64, 64, 16), (64, 64, 16), (48, 48, 24))]
    lw = [W.pa66(), W.e_glass()] if laws == "pa66" else [W.small_sphere_matrix(), W.small_sphere_inclusion()]
    opts = dict(scheme=scheme, precision=precision, tol=TOL[precision], discretization=discretization)
    # the fixed-point scheme stops by its steps: tol k (k + 1) / 2 at a contrast k = 23
    bound = 276 * TOL[precision] if scheme == hom.SCHEME_BASIC else BOUND[precision]
    strains = rng.normal(size=(3, 6)) * 2e-3
    args = (strains, [300.0] * 3, rng.normal(size=(3, 3)), [1.0] * 3)
    with hom.Batch(imgs, lw, autotune=1, **opts) as tuned, hom.Batch(imgs, lw, autotune=0, **opts) as plain:
        sched = tuned.schedules()
        print(f"autotuned schedules: {sched}", flush=True)
        assert sorted(tuple(s["grid"]) for s in sched) == [(16, 64, 64), (24, 48, 48)]
        assert all(s[k]["tile"] in (2, 4, 8) and s[k]["plan"] in (0, 1) for s in sched for k in PASSES)
        assert all(s[k] == DEFAULT for s in plain.schedules() for k in PASSES)
        for a, b in zip(tuned.solve_increment(*args), plain.solve_increment(*args)):
            for k in ("stress", "heat_flux"):
                err = np.abs(a[k] - b[k]).max() / np.abs(b[k]).max()
                print(f"{laws} scheme {scheme} precision {precision} {k}: {err:.2e}", flush=True)
                assert err <= bound


def test_groups_of_whole_planes_report_the_default():
    img = np.zeros((16, 16, 16), np.uint8)
    with hom.Context(img, [W.small_sphere_matrix()], autotune=1) as ctx:
        (s,) = ctx.schedules()
    assert all(s[k] == DEFAULT for k in PASSES)
