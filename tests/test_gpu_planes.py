"""The plane pass at every plane size it has (each ny x nz is a kernel of its own,
with its own rounds of lines and idle threads), element by element against
the oracle's operators. nx = 16 where a few planes take the pass, else 256, whose
129 planes do. Bounds of the pipeline's kernel tests."""
import numpy as np
import pytest

from paper_2109_14403_amd import hom
from test_gpu_kernels import TOL, oracle_apply

pytestmark = pytest.mark.gpu


def planes(precision):
    """(nx, ny, nz) of the plane sizes that fit, by the bytes of 6 (ny + 1) nz
    values and the twiddles."""
    size, few = (16, 64) if precision == hom.FP64 else (8, 104)
    for ny in (16, 24, 32, 48, 64, 96, 128):
        for nz in (16, 24, 32, 48, 64, 96, 128):
            lds = size * (6 * (ny + 1) * nz + ny + nz)
            if lds <= 120 * 1024:
                yield (16 if lds <= few * 1024 else 256), ny, nz


CASES = [(p, *s) for p in (hom.FP64, hom.FP32) for s in planes(p)]


@pytest.mark.parametrize("precision,nx,ny,nz", CASES)
def test_plane_of_every_size_matches_oracle(precision, nx, ny, nz):
    rng = np.random.default_rng(1000 * ny + nz)
    lengths = (1.0, 0.9, 1.2)
    for op, p0, p1, C in ((hom.OP_PROJECTOR, 0.0, 0.0, 6), (hom.OP_GAMMA_CONDUCTION, 0.6, 0.0, 3)):
        f = rng.normal(size=(C, nz, ny, nx)) + 0.25
        gpu = hom.apply_operator(f, op, p0, p1, precision=precision, lengths=lengths)
        ref = oracle_apply(f, op, p0, p1, lengths)
        err = np.abs(gpu - ref).max() / np.abs(ref).max()
        print(f"plane {ny} x {nz}, nx {nx}, op {op} precision {precision}: {err:.2e}", flush=True)
        assert err <= TOL[precision]
