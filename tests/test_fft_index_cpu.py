"""The twiddle indices of the line transforms are formed without a remainder.

With `j % NS` the compiler narrowed the remainder to 8 bits (the thread's range
is known), and its load-store vectorizer joined two twiddles that lie 256 bytes
apart into one access: the y and z passes of 96 points in FP64 took the
imaginary part of one butterfly's twiddle for another's. The kernels here hold
every plan at both ends of what a tile gives (3 and 48 lines)."""
import os
import shutil
import subprocess

import pytest

from paper_2109_14403_amd import build

KERNELS = """
#include "fft_core.h"
namespace hom {
template <typename T, int N, int V, int L>
__global__ void __launch_bounds__(1024) k_line(c2<T>* x, const c2<T>* w) {
  using P = Plan<N, V>;
  extern __shared__ __align__(16) unsigned char smem[];
  c2<T>* tw = reinterpret_cast<c2<T>*>(smem);
  c2<T>* buf = tw + N;
  for (unsigned i = threadIdx.x; i < N; i += blockDim.x) tw[i] = w[i];
  const int tid = threadIdx.x, t = tid / L, l = tid - t * L;
  c2<T> r[P::M];
  for (int m = 0; m < P::M; ++m) r[m] = x[m * 1024 + tid];
  __syncthreads();
  P::run(r, t, tw, buf, L, l, true);
  for (int m = 0; m < P::M; ++m) x[m * 1024 + tid] = r[m];
}
#define ONE(T, N, V) template __global__ void k_line<T, N, V, 3>(c2<T>*, const c2<T>*); \\
                     template __global__ void k_line<T, N, V, 48>(c2<T>*, const c2<T>*);
#define ALL(T, N) ONE(T, N, 0) ONE(T, N, 1)
#define LENGTHS(T) ALL(T, 16) ALL(T, 24) ALL(T, 32) ALL(T, 48) ALL(T, 64) ALL(T, 96) ALL(T, 128) ALL(T, 256)
LENGTHS(float)
LENGTHS(double)
}  // namespace hom
"""


def test_twiddle_indices_take_no_remainder(tmp_path):
    if not shutil.which(build._hipcc()) and not os.path.exists(build._hipcc()):
        pytest.skip("no device compiler here")
    src, out = tmp_path / "lines.hip", tmp_path / "lines.ll"
    src.write_text(KERNELS)
    subprocess.run([build._hipcc()] + build.FLAGS + ["-I", build.CSRC, "--cuda-device-only", "-emit-llvm", "-S",
                                                     str(src), "-o", str(out)], check=True, capture_output=True)
    lines = out.read_text().splitlines()
    assert sum("define" in s and "k_line" in s for s in lines) == 64
    bad = [s.strip() for s in lines if " urem " in s or " srem " in s]
    assert not bad, f"{len(bad)} remainders, e.g. {bad[0]}"
