// The FFT / Green-operator pipeline of one solver iteration.
//
//   xmid   (Newton-CG) inverse transforms along x of the last application of
//          the operator, the CG updates of r, p and x per voxel, the
//          algorithmic tangent applied to the new direction, and its forward
//          transforms along x: the half spectrum kx = 0..nx/2 is replaced in
//          place (two real components packed into one complex line). A
//          residual evaluation only transforms the stress / flux field.
//   ypass  complex transforms along y on tiles of TX contiguous kx columns.
//   zgreen forward transform along z, Green operator per frequency on all
//          components, inverse transform along z.
//   ypass  inverse along y.
// or, where a plane of one kx fits into LDS,
//   yzplane  the y and z transforms both ways with the Green operator between.
//
// The CG scalars are known before a pass needs them: alpha = r.r / p.C p from
// the partial sums of the x pass (p is compatible and the projector
// orthogonal, so p.A p = p.C p); the norm of A p by Parseval's theorem from
// the spectrum the Green operator leaves; then
//   |r - alpha A p|^2 = alpha^2 |A p|^2 - r.r,
// because r.A p = p.A p for conjugate directions. So beta and the stopping
// test are there when the x pass starts, and one pass over the fields does
// what an inverse and a forward pass with a reduction between them did. r.r
// itself is summed from the updated residual in every x pass: the estimate
// decides beta and the end of the solve, and never accumulates. The end of a
// Newton step is decided by the true residual of its evaluation (|r| by
// Parseval's theorem, |sigma| from the x pass).
//
// The fixed-point scheme has no such recurrence. Without internal variables (and
// for conduction) it takes
//   xbasic  inverse transforms along x, the update of the strain, the law and
//           the forward transforms, with the sums that end the iteration before:
//           the z or plane pass behind it moves the solver's state;
// with them, around the same y and z passes,
//   xfwd    forward transforms along x of the stress field,
//   xinv    complex-to-real inverse along x, scaled by 1/(nx ny nz), the update
//           of the strain and FP64 partial sums for the reduction that ends the
//           iteration.
//
// CG keeps three fields (x, r, p): the step x += alpha p of iteration k is
// deferred to the x pass of iteration k + 1 (or to the next constitutive
// evaluation), which reads the old p anyway.
//
// Every kernel serves all problems of a group in one launch: blockIdx.x runs
// over (problem, tile), and a block whose problem is not iterating exits at
// once.
#pragma once
#include "common.h"
#include "pipe_launch.h"

namespace hom {

// Sum of per-thread doubles over the block, deterministic (fixed tree).
template <int K>
__device__ __forceinline__ void block_sum(double (&v)[K], double* red /* >= K * 16 doubles */) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int nw = (blockDim.x + 63) >> 6;
#pragma unroll
  for (int k = 0; k < K; ++k) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v[k] += __shfl_down(v[k], off, 64);
  }
  __syncthreads();
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) red[k * 16 + wave] = v[k];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      double s = 0.0;
      for (int w = 0; w < nw; ++w) s += red[k * 16 + w];
      v[k] = s;
    }
  }
}

// ---------------------------------------------------------------------------
// Green operators on a Mandel (C = 6) or vector (C = 3) complex array.
// ---------------------------------------------------------------------------
// Signed frequency of index k on an n-point axis over a length with
// reciprocal il; the Nyquist entry of an even axis is nulled.
template <typename T>
__device__ __forceinline__ T frequency_component(int k, int n, T il) {
  int sk = k < (n + 1) / 2 ? k : k - n;
  if ((n & 1) == 0 && k == n / 2) sk = 0;
  return T(sk) * il;
}

// 1 / sqrt(m2) for m2 > 0: the hardware reciprocal square root (1 ulp) in
// FP32, the correctly rounded quotient in FP64
__device__ __forceinline__ float inv_norm(float m2) { return __builtin_amdgcn_rsqf(m2); }
__device__ __forceinline__ double inv_norm(double m2) { return 1.0 / sqrt(m2); }

template <typename T>
__device__ __forceinline__ void green_mech(c2<T>* v, T n0, T n1, T n2, T cs, T hcn) {
  // out = cs (n (x) u + u (x) n) - cn (n . u) n (x) n with u = tau n, applied
  // to real and imaginary parts (projector: cs = 1, cn = 1), as
  //   w = cs u - (cn / 2) (n . u) n,  out_ii = 2 n_i w_i,
  //   out_jk = sqrt2 (n_j w_k + n_k w_j)  (Mandel);  hcn = cn / 2.
  // Mandel off-diagonal entries carry sqrt2: tau_jk = v / sqrt2.
  const T r2 = T(0.70710678118654752);
  const T s2 = T(1.4142135623730951);
  const T m0 = n0 * r2, m1 = n1 * r2, m2 = n2 * r2;
  const c2<T> u0 = cscale(v[0], n0) + cscale(v[5], m1) + cscale(v[4], m2);
  const c2<T> u1 = cscale(v[5], m0) + cscale(v[1], n1) + cscale(v[3], m2);
  const c2<T> u2 = cscale(v[4], m0) + cscale(v[3], m1) + cscale(v[2], n2);
  const c2<T> hq = cscale(cscale(u0, n0) + cscale(u1, n1) + cscale(u2, n2), hcn);
  const c2<T> w0 = cscale(u0, cs) - cscale(hq, n0);
  const c2<T> w1 = cscale(u1, cs) - cscale(hq, n1);
  const c2<T> w2 = cscale(u2, cs) - cscale(hq, n2);
  v[0] = cscale(w0, n0 + n0);
  v[1] = cscale(w1, n1 + n1);
  v[2] = cscale(w2, n2 + n2);
  const T q0 = n0 * s2, q1 = n1 * s2, q2 = n2 * s2;
  v[3] = cscale(w2, q1) + cscale(w1, q2);
  v[4] = cscale(w2, q0) + cscale(w0, q2);
  v[5] = cscale(w1, q0) + cscale(w0, q1);
}

// Rotated finite-difference scheme: with e_j = exp(i 2 pi k_j / n_j) and
// h_j = L_j / n_j, k_j = (e_j - 1) / h_j * prod_{l != j} (1 + e_l) / 2 (the
// difference of a corner displacement along j averaged over the 4 cell edges
// parallel to j); n = k / |k|, zero where |k| < 1e-12 sqrt(sum_j (2 / h_j)^2).
// ex, ey, ez are exp(-i 2 pi k_j / n_j) (forward twiddles).
template <typename T>
__device__ __forceinline__ void rotated_direction(c2<T> ex, c2<T> ey, c2<T> ez, int nx, int ny, int nz,
                                                  const double* len, c2<T>* n, bool& zero) {
  const c2<T> e[3] = {conjg(ex), conjg(ey), conjg(ez)};
  const T ih[3] = {T(nx / len[0]), T(ny / len[1]), T(nz / len[2])};
  c2<T> d[3], av[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    d[j] = cscale(e[j] - mk(T(1), T(0)), ih[j]);
    av[j] = cscale(e[j] + mk(T(1), T(0)), T(0.5));
  }
  n[0] = cmul(d[0], cmul(av[1], av[2]));
  n[1] = cmul(d[1], cmul(av[0], av[2]));
  n[2] = cmul(d[2], cmul(av[0], av[1]));
  T m2 = T(0);
#pragma unroll
  for (int j = 0; j < 3; ++j) m2 += n[j].x * n[j].x + n[j].y * n[j].y;
  const T kmax2 = T(4) * (ih[0] * ih[0] + ih[1] * ih[1] + ih[2] * ih[2]);
  zero = !(m2 > T(1e-24) * kmax2);
  const T inv = zero ? T(0) : T(1) / sqrt(m2);
#pragma unroll
  for (int j = 0; j < 3; ++j) n[j] = cscale(n[j], inv);
}

// Hermitian orthogonal projector onto sym(n (x) a) for a complex unit n:
// u = tau conj(n), q = conj(n) . u, out = sym(n (x) (2 u - q n)).
template <typename T>
__device__ __forceinline__ void green_mech_herm(c2<T>* v, const c2<T>* n) {
  const T r2 = T(0.70710678118654752);
  const c2<T> t[3][3] = {{v[0], cscale(v[5], r2), cscale(v[4], r2)},
                         {cscale(v[5], r2), v[1], cscale(v[3], r2)},
                         {cscale(v[4], r2), cscale(v[3], r2), v[2]}};
  const c2<T> nb[3] = {conjg(n[0]), conjg(n[1]), conjg(n[2])};
  c2<T> u[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) u[i] = cmul(t[i][0], nb[0]) + cmul(t[i][1], nb[1]) + cmul(t[i][2], nb[2]);
  const c2<T> q = cmul(nb[0], u[0]) + cmul(nb[1], u[1]) + cmul(nb[2], u[2]);
  c2<T> w[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) w[i] = cscale(u[i], T(2)) - cmul(n[i], q);
  v[0] = cmul(n[0], w[0]);
  v[1] = cmul(n[1], w[1]);
  v[2] = cmul(n[2], w[2]);
  v[3] = cscale(cmul(n[1], w[2]) + cmul(n[2], w[1]), r2);  // sqrt2 * (n1 w2 + n2 w1) / 2
  v[4] = cscale(cmul(n[0], w[2]) + cmul(n[2], w[0]), r2);
  v[5] = cscale(cmul(n[0], w[1]) + cmul(n[1], w[0]), r2);
}

// n (conj(n) . g) for a complex unit n.
template <typename T>
__device__ __forceinline__ void green_grad_herm(c2<T>* v, const c2<T>* n) {
  const c2<T> s = cmul(conjg(n[0]), v[0]) + cmul(conjg(n[1]), v[1]) + cmul(conjg(n[2]), v[2]);
  v[0] = cmul(n[0], s);
  v[1] = cmul(n[1], s);
  v[2] = cmul(n[2], s);
}

template <typename T>
__device__ __forceinline__ void green_grad(c2<T>* v, T n0, T n1, T n2, T s) {
  c2<T> q = cscale(cscale(v[0], n0) + cscale(v[1], n1) + cscale(v[2], n2), s);
  v[0] = cscale(q, n0);
  v[1] = cscale(q, n1);
  v[2] = cscale(q, n2);
}

// ---------------------------------------------------------------------------
// 16-byte global accesses: four consecutive reals, a run of complex values
// ---------------------------------------------------------------------------
template <typename T>
struct Q4 {
  T v[4];
};
// Every field and spectrum element is touched once per pass, and a pass moves
// far more data than the caches hold: the contiguous streaming accesses of the
// x passes are non-temporal (on gfx950 a 1 GiB copy runs 5-15 % faster that
// way). The y / z passes keep cached accesses: their tiles fill 128-byte lines
// from neighbouring work-groups, which the L2 merges.
typedef float nt_f2 __attribute__((ext_vector_type(2)));
typedef float nt_f4 __attribute__((ext_vector_type(4)));
typedef double nt_d2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ Q4<float> ld4(const float* p) {
  const nt_f4 t = __builtin_nontemporal_load(reinterpret_cast<const nt_f4*>(p));
  return Q4<float>{{t.x, t.y, t.z, t.w}};
}
__device__ __forceinline__ Q4<double> ld4(const double* p) {
  const nt_d2 a = __builtin_nontemporal_load(reinterpret_cast<const nt_d2*>(p));
  const nt_d2 b = __builtin_nontemporal_load(reinterpret_cast<const nt_d2*>(p) + 1);
  return Q4<double>{{a.x, a.y, b.x, b.y}};
}
__device__ __forceinline__ void st4(float* p, const float (&v)[4]) {
  const nt_f4 t = {v[0], v[1], v[2], v[3]};
  __builtin_nontemporal_store(t, reinterpret_cast<nt_f4*>(p));
}
__device__ __forceinline__ void st4(double* p, const double (&v)[4]) {
  const nt_d2 a = {v[0], v[1]}, b = {v[2], v[3]};
  __builtin_nontemporal_store(a, reinterpret_cast<nt_d2*>(p));
  __builtin_nontemporal_store(b, reinterpret_cast<nt_d2*>(p) + 1);
}
// one complex value
__device__ __forceinline__ c2<float> ldc(const c2<float>* p) {
  const nt_f2 t = __builtin_nontemporal_load(reinterpret_cast<const nt_f2*>(p));
  return mk(t.x, t.y);
}
__device__ __forceinline__ c2<double> ldc(const c2<double>* p) {
  const nt_d2 t = __builtin_nontemporal_load(reinterpret_cast<const nt_d2*>(p));
  return mk(t.x, t.y);
}
__device__ __forceinline__ void stc(c2<float>* p, c2<float> v) {
  const nt_f2 t = {v.x, v.y};
  __builtin_nontemporal_store(t, reinterpret_cast<nt_f2*>(p));
}
__device__ __forceinline__ void stc(c2<double>* p, c2<double> v) {
  const nt_d2 t = {v.x, v.y};
  __builtin_nontemporal_store(t, reinterpret_cast<nt_d2*>(p));
}

// Element v of a uniform base, with the byte offset formed in 32-bit unsigned
// arithmetic so the access takes the scalar-base + 32-bit-offset form (needs
// v * sizeof(T) < 2^32 inside one component of one problem: true for every
// supported grid, n <= 256).
template <typename T>
__device__ __forceinline__ const T* at(const T* base, unsigned v) {
  return reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + v * (unsigned)sizeof(T));
}
template <typename T>
__device__ __forceinline__ T* at(T* base, unsigned v) {
  return reinterpret_cast<T*>(reinterpret_cast<char*>(base) + v * (unsigned)sizeof(T));
}

// Staging layout of the x passes between the per-voxel phases and the line
// transforms: one row of SP complex values per transform lane, x fastest. A
// thread's four consecutive voxels are 32 contiguous bytes, and the odd pitch
// puts neighbouring transform lanes on different LDS banks.
constexpr int xstage_pitch(int n) { return n + 1; }

// Dynamic LDS of the pipeline kernels in complex values: N twiddles, then the
// work buffer. The launchers size their launches from these, so kernel and
// launch cannot disagree.
template <int N, int NL, int C>
constexpr int xfwd_lds_elems() {
  return N + NL * ((C + 1) / 2) * xstage_pitch(N);  // staging rows (>= N * L, the exchange)
}
template <int N, int NL, int C>
constexpr int xinv_lds_elems() {
  // staged half spectra, or the staging rows (>= N * L, the exchange)
  return N + (NL * (N / 2 + 1) * C > NL * ((C + 1) / 2) * xstage_pitch(N) ? NL * (N / 2 + 1) * C
                                                                            : NL * ((C + 1) / 2) * xstage_pitch(N));
}
template <int N, int TX, int C>
constexpr int tile_lds_elems() {
  return N + N * TX * C;  // y and z passes: the transform exchange of TX * C lines
}

// ---------------------------------------------------------------------------
// x forward: pre-operation + packed real-to-complex transforms
// ---------------------------------------------------------------------------
// Threads of an x work-group: the G * L of the line transforms, or one per
// four-voxel work item of the per-voxel phase if that is more (the extra
// threads idle through the transforms), so that the per-voxel phase, whose
// loads dominate, takes one memory round trip; whole waves
template <int N, int NL, int C>
constexpr int x_threads() {
  constexpr int ft = (N / Plan<N>::M) * NL * ((C + 1) / 2);
  constexpr int items = NL * N / 4;
  return ((items > ft ? items : ft) + 63) / 64 * 64;
}

// Forward transforms of the staged lines (rows of SP complex values in buf,
// two real components each) and the unpacked half spectra, [line][kx][comp]
// with rows PS * C apart or [kx][line][comp] (a.planes). The caller has
// synchronized after its last write to buf.
template <typename T, int C, int N, int NL>
__device__ __forceinline__ void x_forward_lines(const Pipe<T>& a, int prob, int line0, int nvl, const c2<T>* tw,
                                                c2<T>* buf) {
  constexpr int M = Plan<N>::M;
  constexpr int G = N / M;
  constexpr int NP = (C + 1) / 2;
  constexpr int L = NL * NP;
  constexpr int H = N / 2 + 1;
  constexpr int SP = xstage_pitch(N);
  const int tid = threadIdx.x;
  const int nth = blockDim.x;
  const bool fw = tid < G * L;  // a thread of the line transforms
  const int l = tid % L;
  const int t = fw ? tid / L : 0;
  c2<T> r[M];
#pragma unroll
  for (int m = 0; m < M; ++m) r[m] = fw ? buf[l * SP + t + G * m] : mk(T(0), T(0));
  Plan<N>::run(r, t, tw, buf, L, l, fw);
  __syncthreads();
  if (fw) {
#pragma unroll
    for (int m = 0; m < M; ++m) buf[(t + G * m) * L + l] = r[m];
  }
  __syncthreads();

  // unpack the two real transforms of each complex line and write the block's
  // half spectra with 16-byte stores
  constexpr int V = 16 / sizeof(c2<T>);
  auto value = [&](int li, int k, int c) -> c2<T> {
    const int q = c >> 1;
    const c2<T> zk = buf[k * L + li * NP + q];
    const c2<T> zm = conjg(buf[((N - k) % N) * L + li * NP + q]);
    const c2<T> val = (c & 1) ? mul_mi(zk - zm) : (zk + zm);
    return cscale(val, T(0.5));
  };
  if (a.planes) {
    // the block's lines are contiguous in every plane of one kx
    const long long plane = (long long)a.ny * a.nz * C;
    c2<T>* spec = a.spec + (long long)prob * a.P * plane + (long long)line0 * C;
    constexpr int VP = C % 2 == 0 ? V : 1;  // pairs of components of one kx
    for (int i = tid; i < H * NL * C / VP; i += nth) {
      const int e = VP * i;
      const int k = e / (NL * C);
      const int rest = e - k * (NL * C);
      const int li = rest / C;
      const int c = rest - li * C;
      if (li >= nvl) continue;
      if constexpr (VP == 2) {
        const c2<T> u0 = value(li, k, c), u1 = value(li, k, c + 1);
        const nt_f4 t = {u0.x, u0.y, u1.x, u1.y};
        *reinterpret_cast<nt_f4*>(spec + k * plane + rest) = t;
      } else {
        spec[k * plane + rest] = value(li, k, c);
      }
    }
    return;
  }
  const int rowp = a.PS * C;
  c2<T>* spec = a.spec + (long long)prob * a.nz * a.ny * rowp + (long long)line0 * rowp;
  const int total = nvl * H * C;
  // rows are rowp apart; the (kx, comp) entries of one row are contiguous
  if constexpr (V == 2 && C % 2 == 0) {
    // pairs of components of one kx: 16-byte aligned stores (rowp * 8 is a
    // multiple of 128 and the pair starts at an even entry)
    for (int i = tid; i < total / 2; i += nth) {
      const int e = 2 * i;
      const int li = e / (H * C);
      const int rest = e - li * H * C;
      const int k = rest / C;
      const c2<T> u0 = value(li, k, rest - k * C), u1 = value(li, k, rest - k * C + 1);
      const nt_f4 t = {u0.x, u0.y, u1.x, u1.y};
      __builtin_nontemporal_store(t, reinterpret_cast<nt_f4*>(spec + li * rowp + rest));
    }
  } else {
    for (int e = tid; e < total; e += nth) {
      const int li = e / (H * C);
      const int rest = e - li * H * C;
      const int k = rest / C;
      stc(spec + li * rowp + rest, value(li, k, rest - k * C));
    }
  }
}

// Partial sums of an EVAL pass: |f|^2 of the field that is transformed.
template <typename T, int C>
__device__ __forceinline__ double x_load_field(const T* fb, long long nv, unsigned v, T (&out)[4][2 * ((C + 1) / 2)]) {
  double ff = 0.0;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const Q4<T> q = ld4(at(fb + c * nv, v));
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      out[j][c] = q.v[j];
      ff += (double)q.v[j] * (double)q.v[j];
    }
  }
  return ff;
}

// Fixed-point scheme (and single applications of the operator): the stress /
// flux field as it is.
template <typename T, int C, int N, int NL>
__global__ void __launch_bounds__((x_threads<N, NL, C>())) k_xfwd(Pipe<T> a) {
  constexpr int NP = (C + 1) / 2;
  constexpr int SP = xstage_pitch(N);
  static_assert(xfwd_lds_elems<N, NL, C>() - N >= NL * NP * SP, "x-forward LDS buffer too small");
  extern __shared__ __align__(16) unsigned char smem_raw[];
  c2<T>* tw = reinterpret_cast<c2<T>*>(smem_raw);
  c2<T>* buf = tw + N;
  const int nlines = a.ny * a.nz;
  const int bpp = (nlines + NL - 1) / NL;
  const int prob = blockIdx.x / bpp;
  const int line0 = (blockIdx.x % bpp) * NL;
  if (!pipeline_mode(a.ctl[prob].mode)) return;
  const int tid = threadIdx.x;
  for (int i = tid; i < N; i += blockDim.x) tw[i] = a.twx[i];
  const int nvl = min(NL, nlines - line0);
  const T* fb = a.f + (long long)prob * C * a.vs;
  for (int w = tid; w < NL * N / 4; w += blockDim.x) {
    const int e = 4 * w;
    const int li = e / N;
    const int xv = e - li * N;
    T out[4][2 * NP];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int c = 0; c < 2 * NP; ++c) out[j][c] = T(0);
    if (li < nvl) (void)x_load_field<T, C>(fb, a.vs, (unsigned)(line0 * N + e), out);
#pragma unroll
    for (int q = 0; q < NP; ++q)
#pragma unroll
      for (int j = 0; j < 4; ++j) buf[(li * NP + q) * SP + xv + j] = mk(out[j][2 * q], out[j][2 * q + 1]);
  }
  __syncthreads();
  x_forward_lines<T, C, N, NL>(a, prob, line0, nvl, tw, buf);
}

// Work-groups are dispatched to the 8 XCDs round-robin (work-group i to XCD
// i mod 8), each XCD with its own L2. This bijection of [0, n) gives every XCD
// a contiguous range of tiles, so neighbouring kx tiles, which share 128-byte
// lines when a tile row is not a whole number of lines, meet in one L2.
__device__ __forceinline__ int xcd_remap(int i, int n) {
  const int q = n >> 3, rem = n & 7;
  const int x = i & 7, k = i >> 3;
  return x * q + min(x, rem) + k;
}

// ---------------------------------------------------------------------------
// the Newton-CG state of a problem, driven by the first work-group of its y
// and z passes while the others transform. A work-group that starts late may
// already see the new mode: it skips a transform only where the problem has
// ended and nothing reads the spectrum any more.
// ---------------------------------------------------------------------------
// Sums of the first n partials of K quantities q0, q0 + 1, ...; in thread 0.
template <typename T, int K>
__device__ __forceinline__ void block_parts(const Pipe<T>& a, int prob, int q0, int n, double (&s)[K], double* red) {
#pragma unroll
  for (int k = 0; k < K; ++k) s[k] = 0.0;
  const double* pp = a.part + part_index(prob, q0, 0, a.maxblk);
#pragma unroll 4
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
#pragma unroll
    for (int k = 0; k < K; ++k) s[k] += pp[(long long)k * a.maxblk + i];
  }
  block_sum<K>(s, red);
}

// End of a fixed-point iteration: |Gamma0 sigma|^2 against |x|^2 of the field it
// gave (not a number if either is). Called by one thread.
__device__ __forceinline__ void basic_transition(Ctl& c, double dd, double xx, const Limits& lim) {
  c.pipelines += 1;
  const double err = xx == 0.0 ? 0.0 : sqrt(dd / xx);
  c.res = err;
  c.newton_it += 1;
  if (!isfinite(err)) {
    c.mode = M_FAIL;
    c.status = -4;
  } else if (err <= lim.tol) {
    c.mode = M_DONE;
    c.status = 1;
  } else if (c.newton_it >= lim.max_newton) {
    c.mode = M_FAIL;
    c.status = -3;
  }
}

// CG step length alpha = r.r / p.C p, or |f| of a residual evaluation, or the
// end of the fixed-point iteration before, from the partial sums of the x pass.
template <typename T>
__device__ __forceinline__ void cg_step_length(const Pipe<T>& a, int prob) {
  __shared__ double red[2 * 16];
  Ctl& c = a.ctl[prob];
  double s[2];
  block_parts<T, 2>(a, prob, 0, a.xblocks, s, red);
  if (threadIdx.x != 0) return;
  if (c.mode == M_CG) {
    const double pap = s[0];
    c.rr = s[1];
    c.cg_bad = !(pap > 0.0) || !isfinite(pap);
    c.alpha = c.cg_bad ? 0.0 : c.rr / pap;
  } else if (c.mode == M_BASIC) {
    if (c.pending) basic_transition(c, s[0], s[1], a.lim);
    c.pending = c.mode == M_BASIC;  // the x pass has an operator application to take in
  } else {
    c.fnorm = sqrt(s[0]);
  }
}

// End of an application of the operator, |v|^2 (Parseval sum s of the
// spectrum) being the squared norm of the residual or of A p: transitions of
// the state machine. Called by one thread.
__device__ __forceinline__ void newton_cg_transition(Ctl& c, double vv, const Limits& lim) {
  if (c.mode != M_CG && c.mode != M_EVAL) return;  // fixed point: at the step length's place
  c.pipelines += 1;
  if (c.mode == M_CG) {
    // |r - alpha A p|^2; rounding may leave a vanishing residual below zero
    const double rn = fmax(c.alpha * c.alpha * vv - c.rr, 0.0);
    c.beta = c.rr > 0.0 ? rn / c.rr : 0.0;
    c.cg_it += 1;
    c.krylov += 1;
    if (c.cg_bad || !isfinite(vv) || !isfinite(c.rr)) {
      c.mode = M_FAIL;
      c.status = -4;
    } else if (rn <= c.cg_target || c.cg_it >= lim.max_krylov) {
      c.mode = M_EVAL;
      c.pending = 1;
    }
  } else {
    // relative to the stress field; while that is zero, a prescribed mean stress
    // is all the residual there is: relative to itself (not a number if either is)
    const double rn = sqrt(vv), fn = c.fnorm == 0.0 ? rn : c.fnorm;
    const double res = fn == 0.0 ? 0.0 : rn / fn;
    c.res = res;
    c.newton_it += 1;
    c.pending = 0;
    if (!isfinite(res)) {
      c.mode = M_FAIL;
      c.status = -4;
    } else if (res <= lim.tol) {
      c.mode = M_DONE;
      c.status = 1;
    } else if (c.newton_it > lim.max_newton) {
      c.mode = M_FAIL;
      c.status = -3;
    } else {
      const double eta = lim.linear ? 0.0 : fmin(0.1, res);
      const double tgt = fmax(eta * rn, 0.5 * lim.tol * fn);
      c.cg_target = tgt * tgt;
      c.cg_it = 0;
      c.beta = 0.0;
      c.mode = M_CG;
    }
  }
}

template <typename T>
__device__ __forceinline__ void newton_cg_step(const Pipe<T>& a, int prob, double* red /* >= 16 doubles of LDS */) {
  double s[1];
  block_parts<T, 1>(a, prob, 2, a.zblocks, s, red);
  if (threadIdx.x == 0)
    newton_cg_transition(a.ctl[prob], s[0] / ((double)a.nx * a.ny * a.nz), a.lim);
}

// ---------------------------------------------------------------------------
// y pass (forward or inverse) on tiles of TX kx columns
// ---------------------------------------------------------------------------
template <typename T, int C, int N, int TX, int V>
__global__ void __launch_bounds__((N / Plan<N, V>::M) * TX * C) k_ypass(Pipe<T> a, int inverse) {
  constexpr int M = Plan<N, V>::M;
  constexpr int G = N / M;
  constexpr int L = TX * C;
  static_assert(tile_lds_elems<N, TX, C>() - N >= N * L, "tile LDS buffer too small");
  extern __shared__ __align__(16) unsigned char smem_raw[];
  c2<T>* tw = reinterpret_cast<c2<T>*>(smem_raw);
  c2<T>* buf = tw + N;
  const int P = a.P;
  const int nkb = (P + TX - 1) / TX;
  const int bpp = a.nz * nkb;
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  const int prob = bid / bpp;
  const int b = bid % bpp;
  if (!pipeline_mode(a.ctl[prob].mode)) return;
  // the exchange buffer is free until the first transform pass writes it
  if (inverse && a.xblocks > 0 && b == 0) newton_cg_step(a, prob, reinterpret_cast<double*>(buf));
  const int z = b / nkb;
  const int kb = b % nkb;
  const int tid = threadIdx.x;
  for (int i = tid; i < N; i += blockDim.x) tw[i] = a.twy[i];
  const int l = tid % L;
  const int t = tid / L;
  const int kx = kb * TX + l / C;
  const int c = l % C;
  const bool active = kx < P;
  const long long stride = (long long)a.PS * C;
  c2<T>* base = a.spec + (long long)prob * a.nz * a.ny * a.PS * C + ((long long)z * a.ny * a.PS + kx) * C + c;
  c2<T> r[M];
  __syncthreads();
#pragma unroll
  for (int m = 0; m < M; ++m) {
    c2<T> v = active ? base[(t + G * m) * stride] : mk(T(0), T(0));
    r[m] = inverse ? conjg(v) : v;
  }
  Plan<N, V>::run(r, t, tw, buf, L, l, active);
  if (active) {
#pragma unroll
    for (int m = 0; m < M; ++m) base[(t + G * m) * stride] = inverse ? conjg(r[m]) : r[m];
  }
}

// The Green operator of a pipeline at one frequency.
template <typename T>
struct GreenOp {
  const ProbInc& inc;
  T cs = T(1), hcn = T(0.5);
  bool rot;
  __device__ __forceinline__ GreenOp(const Pipe<T>& a, int prob) : inc(a.inc[prob]) {
    if (a.green == G_GAMMA0) {
      cs = T(1.0 / (2.0 * inc.mu0));
      hcn = T(0.5 * (inc.lam0 + inc.mu0) / (inc.mu0 * (inc.lam0 + 2.0 * inc.mu0)));
    } else if (a.green == G_GAMMA_TH) {
      cs = T(1.0 / inc.kappa0);
    }
    rot = (a.green == G_PROJ_ROT || a.green == G_GRADPROJ_ROT);
    eval = a.ctl[prob].mode == M_EVAL;
  }
  bool eval;
  // v: the components at frequency (kx, ky, kz); fa, fb: the x and y parts of
  // the frequency vector; twx, twy, twz: forward twiddles of the axes
  template <int C>
  __device__ __forceinline__ void apply(const Pipe<T>& a, c2<T>* v, int kx, int ky, int kz, T fa, T fb,
                                        const c2<T>* twx, const c2<T>* twy, const c2<T>* twz) const {
    T n0 = T(0), n1 = T(0), n2 = T(0);
    c2<T> nc[3];
    bool zero;
    if (rot) {
      rotated_direction<T>(twx[kx], twy[ky], twz[kz], a.nx, a.ny, a.nz, a.len, nc, zero);
    } else {
      const T fc = frequency_component<T>(kz, a.nz, T(a.ilen[2]));
      const T m2 = fc * fc + (fa * fa + fb * fb);
      zero = !(m2 > T(0));
      const T inv = zero ? T(0) : inv_norm(m2);
      n0 = fa * inv;
      n1 = fb * inv;
      n2 = fc * inv;
    }
    if (zero) {
      // the mean: removed, except for the stress-controlled components of
      // mixed conditions, whose mean strain is an unknown of the iteration
      // (the projector's zero-frequency block is the mask). A residual
      // evaluation compares the mean stress with the prescribed one (the
      // spectrum is unnormalized: the mean mode holds nvox <sigma>).
      const bool mean = (kx == 0 && ky == 0 && kz == 0);
#pragma unroll
      for (int cc = 0; cc < C; ++cc) {
        if (C == 6 && mean && ((inc.smask >> cc) & 1))
          v[cc] = mk(v[cc].x - (eval ? T((double)a.nvox * inc.S[cc]) : T(0)), T(0));
        else
          v[cc] = mk(T(0), T(0));
      }
    } else if (rot) {
      if constexpr (C == 6)
        green_mech_herm<T>(v, nc);
      else
        green_grad_herm<T>(v, nc);
    } else {
      if constexpr (C == 6)
        green_mech<T>(v, n0, n1, n2, cs, hcn);
      else
        green_grad<T>(v, n0, n1, n2, cs);
    }
  }
};

// ---------------------------------------------------------------------------
// z forward + Green operator + z inverse on tiles of TX kx columns
// ---------------------------------------------------------------------------
template <typename T, int C, int N, int TX, int V>
__global__ void __launch_bounds__((N / Plan<N, V>::M) * TX * C)
    __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 5 : 1))) k_zgreen(Pipe<T> a) {
  constexpr int M = Plan<N, V>::M;
  constexpr int G = N / M;
  constexpr int L = TX * C;
  static_assert(tile_lds_elems<N, TX, C>() - N >= N * L, "tile LDS buffer too small");
  extern __shared__ __align__(16) unsigned char smem_raw[];
  c2<T>* tw = reinterpret_cast<c2<T>*>(smem_raw);
  c2<T>* buf = tw + N;
  const int P = a.P;
  const int nkb = (P + TX - 1) / TX;
  const int bpp = a.ny * nkb;
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  const int prob = bid / bpp;
  const int b = bid % bpp;
  if (!pipeline_mode(a.ctl[prob].mode)) return;
  const int ky = b / nkb;
  const int kb = b % nkb;
  const int tid = threadIdx.x;
  const int nth = blockDim.x;
  if (a.xblocks > 0 && b == 0) cg_step_length(a, prob);
  for (int i = tid; i < N; i += nth) tw[i] = a.twz[i];
  const int l = tid % L;
  const int t = tid / L;
  const int kx = kb * TX + l / C;
  const int c = l % C;
  const bool active = kx < P;
  const long long stride = (long long)a.ny * a.PS * C;
  c2<T>* base = a.spec + (long long)prob * a.nz * a.ny * a.PS * C + ((long long)ky * a.PS + kx) * C + c;
  c2<T> r[M];
  __syncthreads();
#pragma unroll
  for (int m = 0; m < M; ++m) r[m] = active ? base[(t + G * m) * stride] : mk(T(0), T(0));
  Plan<N, V>::run(r, t, tw, buf, L, l, active);
  __syncthreads();
#pragma unroll
  for (int m = 0; m < M; ++m) buf[(t + G * m) * L + l] = r[m];
  __syncthreads();

  GreenOp<T> op(a, prob);
  // every index of this thread has the same kx (nth is a multiple of TX):
  // the x and y parts of the frequency are fixed, the z part varies
  const int kxx = kb * TX + tid % TX;
  const T fa = frequency_component<T>(kxx, a.nx, T(a.ilen[0]));
  const T fb = frequency_component<T>(ky, a.ny, T(a.ilen[1]));
  static_assert(((N / Plan<N, V>::M) * TX * C) % TX == 0, "thread count must be a multiple of TX");
  // Parseval sum of the operator's result; a half spectrum stands for its
  // mirror image too, except at kx = 0 and the Nyquist index
  const double pw = (kxx == 0 || 2 * kxx == a.nx) ? 1.0 : 2.0;
  double norm = 0.0;
  for (int idx = tid; idx < N * TX; idx += nth) {
    const int kz = idx / TX;
    const int kxi = idx - kz * TX;
    if (kxx >= P) break;
    c2<T> v[C];
#pragma unroll
    for (int cc = 0; cc < C; ++cc) v[cc] = buf[kz * L + kxi * C + cc];
    op.template apply<C>(a, v, kxx, ky, kz, fa, fb, a.twx, a.twy, tw);
#pragma unroll
    for (int cc = 0; cc < C; ++cc) {
      buf[kz * L + kxi * C + cc] = v[cc];
      norm += (double)v[cc].x * (double)v[cc].x + (double)v[cc].y * (double)v[cc].y;
    }
  }
  if (a.xblocks > 0) {
    __shared__ double nred[16];
    double s[1] = {pw * norm};
    block_sum<1>(s, nred);
    if (tid == 0) a.part[part_index(prob, 2, b, a.maxblk)] = s[0];
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < M; ++m) r[m] = conjg(buf[(t + G * m) * L + l]);
  Plan<N, V>::run(r, t, tw, buf, L, l, active);
  if (active) {
#pragma unroll
    for (int m = 0; m < M; ++m) base[(t + G * m) * stride] = conjg(r[m]);
  }
}

// ---------------------------------------------------------------------------
// y and z transforms, Green operator and back, on a whole plane of one kx
// ---------------------------------------------------------------------------
// Where a plane of all components fits into LDS, one work-group transforms it
// along z (from and to memory, contiguous accesses) and along y (in LDS) both
// ways, with the Green operator between: one pass over the spectra instead of
// three. A line's exchange takes place in the line's own LDS elements.
// The work-group's vector instructions bound it (no packed FP32; lines spread
// over the four lanes of a quad with the exchange in registers and a sixth of
// the barriers took 1.0 to 1.3 times as long, because they take more of them).
template <int N>
constexpr int plane_plan = N == 96 ? 1 : 0;  // 12 instead of 24 elements a thread
template <typename T, int C, int NY, int NZ>
struct PlaneCfg {
  using PY = Plan<NY, plane_plan<NY>>;
  using PZ = Plan<NZ, plane_plan<NZ>>;
  static constexpr int GY = NY / PY::M, GZ = NZ / PZ::M;
  static constexpr int LY = NZ * C, LZ = NY * C;  // lines along y and z
  // threads: all lines at once if the registers of a thread's elements allow
  // it, else in rounds of whole lines
  static constexpr int MOST = sizeof(T) == 8 ? 512 : 1024;
  static constexpr int rounds(int lines, int g, int threads) { return (lines + threads / g - 1) / (threads / g); }
  static constexpr int need(int lines, int g) {
    return g * ((lines + rounds(lines, g, MOST) - 1) / rounds(lines, g, MOST));
  }
  static constexpr int THREADS = ((need(LY, GY) > need(LZ, GZ) ? need(LY, GY) : need(LZ, GZ)) + 63) / 64 * 64;
  static constexpr int RY = rounds(LY, GY, THREADS), RZ = rounds(LZ, GZ, THREADS);
  static constexpr int NLY = (LY + RY - 1) / RY, NLZ = (LZ + RZ - 1) / RZ;  // lines of a round
  static constexpr int SZ = plane_row(NY, C);                               // LDS row of one z
  // thread tid's place in round i: line and position in it (off lines: idle)
  static __device__ __forceinline__ bool y_line(int tid, int i, int& t, int& l) {
    t = tid / NLY;
    l = tid - t * NLY + i * NLY;
    const bool on = t < GY && l < LY;
    t = on ? t : 0;
    l = on ? l : 0;
    return on;
  }
  static __device__ __forceinline__ bool z_line(int tid, int i, int& t, int& l) {
    t = tid / NLZ;
    l = tid - t * NLZ + i * NLZ;
    const bool on = t < GZ && l < LZ;
    t = on ? t : 0;
    l = on ? l : 0;
    return on;
  }
};

template <typename T, int C, int NY, int NZ>
__global__ void __launch_bounds__((PlaneCfg<T, C, NY, NZ>::THREADS)) k_yzplane(Pipe<T> a) {
  using Cfg = PlaneCfg<T, C, NY, NZ>;
  using PY = typename Cfg::PY;
  using PZ = typename Cfg::PZ;
  constexpr int GY = Cfg::GY, GZ = Cfg::GZ, SZ = Cfg::SZ, NTH = Cfg::THREADS, LZ = Cfg::LZ;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  c2<T>* twy = reinterpret_cast<c2<T>*>(smem_raw);
  c2<T>* twz = twy + NY;
  c2<T>* S = twz + NZ;
  __shared__ double red[2 * 16];
  __shared__ int last;
  const int P = a.P;
  const bool drive = a.xblocks > 0;  // Newton-CG: one more work-group a problem forms the step length
  const int bpp = drive ? P + 1 : P;
  const int prob = blockIdx.x / bpp;
  const int kx = blockIdx.x - prob * bpp;
  Ctl& ctl = a.ctl[prob];
  const int mode = ctl.mode;
  if (!pipeline_mode(mode)) return;
  const int tid = threadIdx.x;
  double norm = 0.0;
  c2<T>* base = a.spec + ((long long)prob * P + min(kx, P - 1)) * (NY * NZ * C);
  if (kx < P) {
    c2<T> rz[Cfg::RZ][PZ::M];
#pragma unroll
    for (int i = 0; i < Cfg::RZ; ++i) {
      int t, l;
      const bool on = Cfg::z_line(tid, i, t, l);
#pragma unroll
      for (int m = 0; m < PZ::M; ++m) rz[i][m] = on ? base[(t + GZ * m) * LZ + l] : mk(T(0), T(0));
    }
    for (int i = tid; i < NY; i += NTH) twy[i] = a.twy[i];
    for (int i = tid; i < NZ; i += NTH) twz[i] = a.twz[i];
    __syncthreads();
    // z forward
#pragma unroll
    for (int i = 0; i < Cfg::RZ; ++i) {
      int t, l;
      const bool on = Cfg::z_line(tid, i, t, l);
      PZ::run(rz[i], t, twz, S, SZ, l, on);
      __syncthreads();
      if (on) {
#pragma unroll
        for (int m = 0; m < PZ::M; ++m) S[(t + GZ * m) * SZ + l] = rz[i][m];
      }
    }
    __syncthreads();
    // y forward
#pragma unroll
    for (int i = 0; i < Cfg::RY; ++i) {
      int t, l;
      const bool on = Cfg::y_line(tid, i, t, l);
      const int z = l / C, off = z * SZ + (l - z * C);
      c2<T> r[PY::M];
#pragma unroll
      for (int m = 0; m < PY::M; ++m) r[m] = S[off + (t + GY * m) * C];
      PY::run(r, t, twy, S, C, off, on);
      __syncthreads();
      if (on) {
#pragma unroll
        for (int m = 0; m < PY::M; ++m) S[off + (t + GY * m) * C] = r[m];
      }
    }
    __syncthreads();
    {
      const GreenOp<T> op(a, prob);
      const T fa = frequency_component<T>(kx, a.nx, T(a.ilen[0]));
      for (int i = tid; i < NY * NZ; i += NTH) {
        const int kz = i / NY, ky = i - kz * NY;
        c2<T>* q = S + kz * SZ + ky * C;
        c2<T> v[C];
#pragma unroll
        for (int c = 0; c < C; ++c) v[c] = q[c];
        op.template apply<C>(a, v, kx, ky, kz, fa, frequency_component<T>(ky, NY, T(a.ilen[1])), a.twx, twy, twz);
#pragma unroll
        for (int c = 0; c < C; ++c) {
          q[c] = v[c];
          norm += (double)v[c].x * (double)v[c].x + (double)v[c].y * (double)v[c].y;
        }
      }
      // Parseval weight: a half spectrum stands for its mirror image too
      if (kx != 0 && 2 * kx != a.nx) norm *= 2.0;
    }
  }
  if (drive && mode == M_BASIC) {  // no norm and nothing to wait for (16^3 in FP64 6.3 us, 8.0 with the ticket)
    if (kx == P) cg_step_length(a, prob);
  } else if (drive) {
    if (kx == P) cg_step_length(a, prob);
    double s[1] = {norm};
    block_sum<1>(s, red);
    if (tid == 0) {
      // the last work-group of the problem has every partial sum and the step
      // length, and moves the solver's state while the others transform back
      double* pp = a.part + part_index(prob, 2, 0, a.maxblk);
      if (kx < P) __hip_atomic_store(pp + kx, s[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int before = __hip_atomic_fetch_add(&ctl.ticket, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
      last = before == P;
    }
    __syncthreads();
    if (last && tid < 64) {
      const double* pp = a.part + part_index(prob, 2, 0, a.maxblk);
      double v = 0.0;
      for (int i = tid; i < P; i += 64) v += __hip_atomic_load(pp + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
      if (tid == 0) {
        ctl.ticket = 0;
        newton_cg_transition(ctl, v / ((double)a.nx * a.ny * a.nz), a.lim);
      }
    }
  }
  if (kx >= P) return;
  __syncthreads();
  // y inverse
#pragma unroll
  for (int i = 0; i < Cfg::RY; ++i) {
    int t, l;
    const bool on = Cfg::y_line(tid, i, t, l);
    const int z = l / C, off = z * SZ + (l - z * C);
    c2<T> r[PY::M];
#pragma unroll
    for (int m = 0; m < PY::M; ++m) r[m] = conjg(S[off + (t + GY * m) * C]);
    PY::run(r, t, twy, S, C, off, on);
    __syncthreads();
    if (on) {
#pragma unroll
      for (int m = 0; m < PY::M; ++m) S[off + (t + GY * m) * C] = conjg(r[m]);
    }
  }
  __syncthreads();
  // z inverse
#pragma unroll
  for (int i = 0; i < Cfg::RZ; ++i) {
    int t, l;
    const bool on = Cfg::z_line(tid, i, t, l);
    c2<T> r[PZ::M];
#pragma unroll
    for (int m = 0; m < PZ::M; ++m) r[m] = conjg(S[(t + GZ * m) * SZ + l]);
    PZ::run(r, t, twz, S, SZ, l, on);
    if (on) {
#pragma unroll
      for (int m = 0; m < PZ::M; ++m) base[(t + GZ * m) * LZ + l] = conjg(r[m]);
    }
  }
}

// ---------------------------------------------------------------------------
// x inverse: packed complex-to-real transforms (+ post-operation + partial sums)
// ---------------------------------------------------------------------------
// Staging access of x_inverse_lines: a pair of FP32 complex values, else one
// complex value.
template <typename T, int V>
struct x_access;
template <>
struct x_access<float, 2> {
  using type = nt_f4;
};
template <>
struct x_access<float, 1> {
  using type = nt_f2;
};
template <>
struct x_access<double, 1> {
  using type = nt_d2;
};
// The half spectra of a work-group's lines, transformed back: rows of SP
// complex values in buf (unscaled), two real components each. The launch has
// NTH threads. Ends synchronized.
template <typename T, int C, int N, int NL, int NTH>
__device__ __forceinline__ void x_inverse_lines(const Pipe<T>& a, int prob, int line0, int nvl, const c2<T>* tw,
                                                c2<T>* buf) {
  constexpr int M = Plan<N>::M;
  constexpr int G = N / M;
  constexpr int NP = (C + 1) / 2;
  constexpr int L = NL * NP;
  constexpr int H = N / 2 + 1;
  constexpr int SP = xstage_pitch(N);
  static_assert(xinv_lds_elems<N, NL, C>() - N >= L * SP && xinv_lds_elems<N, NL, C>() - N >= NL * H * C &&
                    L * SP >= N * L,
                "x-inverse LDS buffer too small");
  const int tid = threadIdx.x;
  // stage the block's half spectra: [line][kx][comp], rows rowp apart in
  // memory and packed in LDS, or [kx][line][comp] (a.planes). All of a
  // thread's loads are issued before the LDS writes, with indices clamped in
  // range and no branch between them; a clamped thread rewrites the last
  // element's own value (else the compiler sinks each load into its write's
  // branch).
  constexpr int V = (sizeof(c2<T>) == 8 && C % 2 == 0) ? 2 : 1;
  constexpr int K = (NL * H * C / V + NTH - 1) / NTH;
  using acc_t = typename x_access<T, V>::type;
  acc_t t4[K];
  acc_t* d4 = reinterpret_cast<acc_t*>(buf);
  int tot;
  if (a.planes) {
    const long long plane = (long long)a.ny * a.nz * C;
    const c2<T>* spec = a.spec + (long long)prob * a.P * plane + (long long)line0 * C;
    tot = NL * H * C / V;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int e = V * min(tid + k * NTH, tot - 1);
      const int kk = e / (NL * C);
      const int rest = min(e - kk * (NL * C), nvl * C - V);
      t4[k] = *reinterpret_cast<const acc_t*>(spec + kk * plane + rest);
    }
  } else {
    const int rowp = a.PS * C;
    const c2<T>* spec = a.spec + (long long)prob * a.nz * a.ny * rowp + (long long)line0 * rowp;
    tot = nvl * H * C / V;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int e = V * min(tid + k * NTH, tot - 1);
      const int li = e / (H * C);
      t4[k] = __builtin_nontemporal_load(reinterpret_cast<const acc_t*>(spec + li * rowp + (e - li * H * C)));
    }
  }
#pragma unroll
  for (int k = 0; k < K; ++k) d4[min(tid + k * NTH, tot - 1)] = t4[k];
  const int sl = a.planes ? C : H * C;   // LDS strides of a line and of a kx
  const int sk = a.planes ? NL * C : C;
  if (!a.planes)
    for (int e = nvl * H * C + tid; e < NL * H * C; e += NTH) buf[e] = mk(T(0), T(0));
  __syncthreads();
  const bool fw = NTH == G * L || tid < G * L;  // a thread of the line transforms
  const int l = tid % L;
  const int t = fw ? tid / L : 0;
  const int li = l / NP;
  const int q = l - li * NP;
  c2<T> r[M];
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const int p = t + G * m;
    const bool lo = p <= N / 2;
    const int kk = lo ? p : N - p;
    c2<T> A = buf[li * sl + kk * sk + 2 * q];
    c2<T> B = (2 * q + 1 < C) ? buf[li * sl + kk * sk + 2 * q + 1] : mk(T(0), T(0));
    if (!lo) {
      A = conjg(A);
      B = conjg(B);
    }
    // Z = A + i B, transformed as conj(DFT(conj(Z)))
    r[m] = mk(A.x - B.y, -(A.y + B.x));
  }
  Plan<N>::run(r, t, tw, buf, L, l, fw);
  __syncthreads();
  if (fw) {
#pragma unroll
    for (int m = 0; m < M; ++m) buf[l * SP + t + G * m] = conjg(r[m]);
  }
  __syncthreads();
}

template <typename T, int C, int N, int NL>
__global__ void __launch_bounds__((x_threads<N, NL, C>())) k_xinv(Pipe<T> a) {
  constexpr int NP = (C + 1) / 2;
  constexpr int SP = xstage_pitch(N);
  extern __shared__ __align__(16) unsigned char smem_raw[];
  c2<T>* tw = reinterpret_cast<c2<T>*>(smem_raw);
  c2<T>* buf = tw + N;  // holds the staged half spectra first, then the line FFTs
  __shared__ double red[2 * 16];

  const int nlines = a.ny * a.nz;
  const int bpp = (nlines + NL - 1) / NL;
  const int prob = blockIdx.x / bpp;
  const int blk = blockIdx.x % bpp;
  const int line0 = blk * NL;
  const int mode = a.ctl[prob].mode;
  if (!pipeline_mode(mode)) return;
  const int tid = threadIdx.x;
  const int nth = blockDim.x;
  for (int i = tid; i < N; i += nth) tw[i] = a.twx[i];
  const int nvl = min(NL, nlines - line0);
  x_inverse_lines<T, C, N, NL, x_threads<N, NL, C>()>(a, prob, line0, nvl, tw, buf);

  const long long nv = a.vs;  // stride of the per-voxel arrays (component, problem)
  const long long fo = (long long)prob * C * nv;
  const T scale = T(1.0 / ((double)a.nx * a.ny * a.nz));
  double s0 = 0.0, s1 = 0.0;
  const unsigned v0 = (unsigned)(line0 * N);
  const T* sb = (mode == M_EVAL ? a.f : a.x) + fo;  // uniform bases
  T* db = (mode == M_BASIC ? a.x : a.r) + fo;
  for (int w = tid; w < nvl * N / 4; w += nth) {
    const int e = 4 * w;
    const int lj = e / N;
    const int xv = e - lj * N;
    const unsigned v = v0 + (unsigned)e;
    // the work item's global operand for every component first (one memory
    // round trip), then the transformed values from LDS, then the stores
    Q4<T> q[C];
#pragma unroll
    for (int c = 0; c < C; ++c) q[c] = ld4(at(sb + c * nv, v));
#pragma unroll
    for (int c = 0; c < C; ++c) {
      T g[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const c2<T> z = buf[(lj * NP + (c >> 1)) * SP + xv + j];
        g[j] = ((c & 1) ? z.y : z.x) * scale;
      }
      T* o = at(db + c * nv, v);
      T out[4];
      if (mode == M_EVAL) {  // a single application of the operator: r = -Gamma f
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          out[j] = -g[j];
          s0 += (double)g[j] * (double)g[j];
          s1 += (double)q[c].v[j] * (double)q[c].v[j];
        }
        st4(o, out);
      } else {  // basic scheme: x -= Gamma0 sigma
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          out[j] = q[c].v[j] - g[j];
          s0 += (double)g[j] * (double)g[j];
          s1 += (double)out[j] * (double)out[j];
        }
        st4(o, out);
      }
    }
  }
  double s[2] = {s0, s1};
  block_sum<2>(s, red);
  if (tid == 0) {
    a.part[part_index(prob, 0, blk, a.maxblk)] = s[0];
    a.part[part_index(prob, 1, blk, a.maxblk)] = s[1];
  }
}

// ---------------------------------------------------------------------------
// x middle: one pass of a Newton-CG iteration over the fields
// ---------------------------------------------------------------------------
template <int N, int NL, int C>
constexpr int xmid_lds_elems() {
  return xinv_lds_elems<N, NL, C>() > xfwd_lds_elems<N, NL, C>() ? xinv_lds_elems<N, NL, C>()
                                                                  : xfwd_lds_elems<N, NL, C>();
}

// Bound by HBM at 128^3 and above (two spectra and six field accesses, 207
// bytes a voxel in FP32), by the latency of its chain of loads, exchanges and
// stores below. In the place of a forward pass, an inverse pass and a
// reduction kernel, which moved the residual twice more and stood one behind
// the other: an increment of the 256^3 fibre composite 140.4 -> 134.8 ms, of
// a 64^3 cell 6.72 -> 5.77 ms, a 32^3 cell with its four tangents 28.0 ->
// 22.7 ms, 96 x 24 x 48 in FP64 19.7 -> 17.5 ms.
// FP32: at most 128 VGPRs, four waves per SIMD (it takes 107)
template <typename T, int C, int N, int NL>
__global__ void __launch_bounds__((x_threads<N, NL, C>()))
    __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 1))) k_xmid(Pipe<T> a) {
  constexpr int NP = (C + 1) / 2;
  constexpr int SP = xstage_pitch(N);
  extern __shared__ __align__(16) unsigned char smem_raw[];
  c2<T>* tw = reinterpret_cast<c2<T>*>(smem_raw);
  c2<T>* buf = tw + N;
  __shared__ double red[2 * 16];
  const int nlines = a.ny * a.nz;
  const int bpp = (nlines + NL - 1) / NL;
  const int prob = blockIdx.x / bpp;
  const int blk = blockIdx.x % bpp;
  const int line0 = blk * NL;
  const Ctl& ctl = a.ctl[prob];
  const int mode = ctl.mode;
  if (mode != M_EVAL && mode != M_CG) return;
  const int tid = threadIdx.x;
  const int nth = blockDim.x;
  for (int i = tid; i < N; i += nth) tw[i] = a.twx[i];
  const long long nv = a.vs;  // stride of the per-voxel arrays (component, problem)
  const long long fo = (long long)prob * C * nv;
  const int cell = prob / a.div;  // whose phases and tangents the problem has
  const uint8_t* phase = a.phase + (long long)cell * nv;
  const ProbInc& inc = a.inc[prob];
  const bool cg = (mode == M_CG);
  const bool first = (ctl.cg_it == 0);
  const T beta = T(ctl.beta);
  const T alpha = T(ctl.alpha);  // step length of the direction p in memory
  __shared__ T ptab[MAX_PHASES];  // 3K (mechanics) or kappa (conduction) per phase
  if (tid < MAX_PHASES) ptab[tid] = T(C == 6 ? inc.ph[tid].K3 : inc.ph[tid].kappa);
  const int nvl = min(NL, nlines - line0);
  if (cg)  // uniform over the work-group
    x_inverse_lines<T, C, N, NL, x_threads<N, NL, C>()>(a, prob, line0, nvl, tw, buf);

  // four consecutive voxels of one line per work item, 16-byte accesses;
  // uniform per-component bases and a 32-bit voxel offset: loads and stores
  // take the scalar-base + 32-bit-offset form
  const unsigned v0 = (unsigned)(line0 * N);
  const T scale = T(1.0 / ((double)a.nx * a.ny * a.nz));
  T* rb = a.r + fo;
  T* pb = a.p + fo;
  T* xb = a.x + fo;
  const T* tb = a.tab + (long long)cell * 2 * nv;
  const T* nb = a.tn + (long long)cell * 6 * nv;
  double s0 = 0.0, s1 = 0.0;  // CG: p . C p and r . r; evaluation: f . f
  const int w = tid;
  if (w < NL * N / 4) {
    const int e = 4 * w;
    const int li = e / N;
    const int xv = e - li * N;
    T out[4][2 * NP];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int c = 0; c < 2 * NP; ++c) out[j][c] = T(0);
    if (li < nvl) {
      const unsigned v = v0 + (unsigned)e;
      if (!cg) {
        s0 = x_load_field<T, C>(a.f + fo, nv, v, out);
      } else {
        // r -= alpha A p, p = r + beta p, and the deferred step x += alpha p.
        // Every load of the work item is issued before the first store (one
        // memory round trip instead of one per component).
        Q4<T> rq[C], pq[C], xq[C];
        if (!first) {  // uniform over the block
#pragma unroll
          for (int c = 0; c < C; ++c) {
            rq[c] = ld4(at(rb + c * nv, v));
            pq[c] = ld4(at(pb + c * nv, v));
            xq[c] = ld4(at(xb + c * nv, v));
          }
        }
        Q4<T> ca, cb;
        if constexpr (C == 6) {
          ca = ld4(at(tb, v));
          cb = ld4(at(tb + nv, v));
        }
        const uchar4 ph = *reinterpret_cast<const uchar4*>(at(phase, v));
        T pv[C][4];
#pragma unroll
        for (int c = 0; c < C; ++c) {
          T g[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const c2<T> z = buf[(li * NP + (c >> 1)) * SP + xv + j];
            g[j] = ((c & 1) ? z.y : z.x) * scale;
          }
          T rn[4];
          if (first) {  // g is the projected residual stress
#pragma unroll
            for (int j = 0; j < 4; ++j) pv[c][j] = rn[j] = -g[j];
          } else {
            T xn[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              rn[j] = rq[c].v[j] - alpha * g[j];
              pv[c][j] = rn[j] + beta * pq[c].v[j];
              xn[j] = xq[c].v[j] + alpha * pq[c].v[j];
            }
            st4(at(xb + c * nv, v), xn);
          }
          st4(at(rb + c * nv, v), rn);
          st4(at(pb + c * nv, v), pv[c]);
#pragma unroll
          for (int j = 0; j < 4; ++j) s1 += (double)rn[j] * (double)rn[j];
        }
        const int phs[4] = {ph.x, ph.y, ph.z, ph.w};
        if constexpr (C == 6) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const T tr3 = (pv[0][j] + pv[1][j] + pv[2][j]) * T(1.0 / 3.0);
            const T sph = (ptab[phs[j]] - ca.v[j]) * tr3;
#pragma unroll
            for (int c = 0; c < 6; ++c) out[j][c] = ca.v[j] * pv[c][j];
            out[j][0] += sph;
            out[j][1] += sph;
            out[j][2] += sph;
          }
          if (cb.v[0] != T(0) || cb.v[1] != T(0) || cb.v[2] != T(0) || cb.v[3] != T(0)) {
            T nd[6][4];
#pragma unroll
            for (int c = 0; c < 6; ++c) {
              const Q4<T> q = ld4(at(nb + c * nv, v));
#pragma unroll
              for (int j = 0; j < 4; ++j) nd[c][j] = q.v[j];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              if (cb.v[j] == T(0)) continue;
              T dot = T(0);
#pragma unroll
              for (int c = 0; c < 6; ++c) dot += nd[c][j] * pv[c][j];
#pragma unroll
              for (int c = 0; c < 6; ++c) out[j][c] += cb.v[j] * dot * nd[c][j];
            }
          }
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const T kap = ptab[phs[j]];
#pragma unroll
            for (int c = 0; c < C; ++c) out[j][c] = kap * pv[c][j];
          }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int c = 0; c < C; ++c) s0 += (double)pv[c][j] * (double)out[j][c];
      }
    }
    // each work item overwrites the staged values that it alone has read
#pragma unroll
    for (int q = 0; q < NP; ++q)
#pragma unroll
      for (int j = 0; j < 4; ++j) buf[(li * NP + q) * SP + xv + j] = mk(out[j][2 * q], out[j][2 * q + 1]);
  }
  double s[2] = {s0, s1};
  block_sum<2>(s, red);
  if (tid == 0) {
    a.part[part_index(prob, 0, blk, a.maxblk)] = s[0];
    a.part[part_index(prob, 1, blk, a.maxblk)] = s[1];
  }
  __syncthreads();
  x_forward_lines<T, C, N, NL>(a, prob, line0, nvl, tw, buf);
}

// ---------------------------------------------------------------------------
// x middle pass of the fixed-point scheme without internal variables: inverse
// transform, x -= Gamma0 sigma, the law, forward transform
// ---------------------------------------------------------------------------
// Bound like the middle pass above. In the place of the evaluation, a forward
// pass, an inverse pass and a reduction kernel (the end of an iteration is found
// by the next one's z or plane pass): elastic increments of 16^3 in FP64 3.54 ->
// 2.16 ms, 32^3 FP64 5.56 -> 4.05, FP32 3.13 -> 2.18, 64^3 FP32 5.34 -> 4.00,
// 128^3 FP32 16.2 -> 12.7 ms. Laws with internal variables keep the pointwise
// evaluation: theirs takes 130 registers and reads the state.
template <typename T, int C, int N, int NL>
__global__ void __launch_bounds__((x_threads<N, NL, C>())) k_xbasic(Pipe<T> a) {
  constexpr int NP = (C + 1) / 2;
  constexpr int SP = xstage_pitch(N);
  extern __shared__ __align__(16) unsigned char smem_raw[];
  c2<T>* tw = reinterpret_cast<c2<T>*>(smem_raw);
  c2<T>* buf = tw + N;
  __shared__ double red[2 * 16];
  __shared__ double ptab[MAX_PHASES][3];  // 3K, 2G, thermal strain (mechanics) or kappa (conduction) per phase
  const int nlines = a.ny * a.nz;
  const int bpp = (nlines + NL - 1) / NL;
  const int prob = blockIdx.x / bpp;
  const int blk = blockIdx.x % bpp;
  const int line0 = blk * NL;
  const Ctl& ctl = a.ctl[prob];
  if (ctl.mode != M_BASIC) return;
  const bool pending = ctl.pending != 0;  // an application of the operator is in the spectrum
  const int tid = threadIdx.x;
  const int nth = blockDim.x;
  for (int i = tid; i < N; i += nth) tw[i] = a.twx[i];
  const ProbInc& inc = a.inc[prob];
  if (tid < MAX_PHASES) {
    ptab[tid][0] = C == 6 ? inc.ph[tid].K3 : inc.ph[tid].kappa;
    ptab[tid][1] = inc.ph[tid].G2;
    ptab[tid][2] = inc.ph[tid].alpha_dth;
  }
  const int nvl = min(NL, nlines - line0);
  if (pending)  // uniform over the work-group
    x_inverse_lines<T, C, N, NL, x_threads<N, NL, C>()>(a, prob, line0, nvl, tw, buf);
  else
    __syncthreads();
  const long long nv = a.vs;  // stride of the per-voxel arrays (component, problem)
  const long long fo = (long long)prob * C * nv;
  const uint8_t* phase = a.phase + (long long)prob * nv;
  const T scale = T(1.0 / ((double)a.nx * a.ny * a.nz));
  T* xb = a.x + fo;
  T* fb = a.f + fo;
  // sigma = 3K (tr/3 - alpha dtheta) 1 + 2G dev of voxel j, as the pointwise evaluation forms it
  const auto law = [&](const T (&x)[C][4], int j, int ph, T (&f)[C]) {
    if constexpr (C == 6) {
      const double K3 = ptab[ph][0], G2 = ptab[ph][1];
      const double tr3 = ((double)x[0][j] + (double)x[1][j] + (double)x[2][j]) * (1.0 / 3.0);
      const double sph = K3 * (tr3 - ptab[ph][2]) - G2 * tr3;
#pragma unroll
      for (int c = 0; c < 6; ++c) f[c] = T(G2 * (double)x[c][j] + (c < 3 ? sph : 0.0));
    } else {
      const T kap = T(ptab[ph][0]);
#pragma unroll
      for (int c = 0; c < C; ++c) f[c] = kap * x[c][j];
    }
  };
  double s0 = 0.0, s1 = 0.0;
  const int w = tid;
  if (w < NL * N / 4) {
    const int e = 4 * w;
    const int li = e / N;
    const int xv = e - li * N;
    T out[4][2 * NP];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int c = 0; c < 2 * NP; ++c) out[j][c] = T(0);
    if (li < nvl) {
      const unsigned v = (unsigned)(line0 * N + e);
      Q4<T> q[C];
#pragma unroll
      for (int c = 0; c < C; ++c) q[c] = ld4(at(xb + c * nv, v));
      const uchar4 ph = *reinterpret_cast<const uchar4*>(at(phase, v));
      const int phs[4] = {ph.x, ph.y, ph.z, ph.w};
      T x[C][4];
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int j = 0; j < 4; ++j) x[c][j] = q[c].v[j];
      if constexpr (C == 6) {  // the stress field that goes with this iteration: of the strain it starts from
        T f[C][4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          T fj[C];
          law(x, j, phs[j], fj);
#pragma unroll
          for (int c = 0; c < C; ++c) f[c][j] = fj[c];
        }
#pragma unroll
        for (int c = 0; c < C; ++c) st4(at(fb + c * nv, v), f[c]);
      }
      if (pending) {
#pragma unroll
        for (int c = 0; c < C; ++c) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const c2<T> z = buf[(li * NP + (c >> 1)) * SP + xv + j];
            const T g = ((c & 1) ? z.y : z.x) * scale;
            x[c][j] -= g;
            s0 += (double)g * (double)g;
            s1 += (double)x[c][j] * (double)x[c][j];
          }
          st4(at(xb + c * nv, v), x[c]);
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        T fj[C];
        law(x, j, phs[j], fj);
#pragma unroll
        for (int c = 0; c < C; ++c) out[j][c] = fj[c];
      }
    }
    // each work item overwrites the staged values that it alone has read
#pragma unroll
    for (int q = 0; q < NP; ++q)
#pragma unroll
      for (int j = 0; j < 4; ++j) buf[(li * NP + q) * SP + xv + j] = mk(out[j][2 * q], out[j][2 * q + 1]);
  }
  double s[2] = {s0, s1};
  block_sum<2>(s, red);
  if (tid == 0) {
    a.part[part_index(prob, 0, blk, a.maxblk)] = s[0];
    a.part[part_index(prob, 1, blk, a.maxblk)] = s[1];
  }
  __syncthreads();
  x_forward_lines<T, C, N, NL>(a, prob, line0, nvl, tw, buf);
}

}  // namespace hom
