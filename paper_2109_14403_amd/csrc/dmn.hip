// Direct deep material network (see dmn.h): offline training kernels and
// the online evaluation of many macroscopic points.
//
// Laminate of two phases with stiffnesses C1, C2, fractions c1, c2 = 1 - c1
// and normal n (the exact laminate rule; the paper writes it with the
// auxiliary parameter lambda of Sec. 3.2, which gives the same stiffness):
// the phase strains are eps1 = eps + c2 N a, eps2 = eps - c1 N a with
// N a = sym(a (x) n) (Mandel, 6 x 3), the jump a makes the traction
// continuous, N^T (sigma1 - sigma2) = 0, so
//   M = N^T (c2 C1 + c1 C2) N,  a = -M^-1 N^T (C1 - C2) eps,
//   C = c1 C1 + c2 C2 - c1 c2 (C1 - C2) N M^-1 N^T (C1 - C2).
// The online Newton step eliminates the jumps of the whole tree the same way,
// from the leaves to the root, with each subtree's condensed tangent and
// stress offset: one 3 x 3 solve per laminate instead of the dense system.
#include <math.h>

#include <algorithm>
#include <cstring>
#include <random>
#include <string>
#include <type_traits>
#include <unordered_map>
#include <utility>

#include "dmn.h"
#include "pa66.h"
#include "pipeline.h"
#include "runtime.h"

namespace hom {

namespace {

constexpr double SQ2H = 0.70710678118654752440;  // sqrt(2) / 2

// N (6 x 3, Mandel) of a -> sym(a (x) n)
__device__ __forceinline__ void nmat(const double* n, double N[6][3]) {
#pragma unroll
  for (int i = 0; i < 6; ++i)
#pragma unroll
    for (int k = 0; k < 3; ++k) N[i][k] = 0.0;
  N[0][0] = n[0];
  N[1][1] = n[1];
  N[2][2] = n[2];
  N[3][1] = SQ2H * n[2];
  N[3][2] = SQ2H * n[1];
  N[4][0] = SQ2H * n[2];
  N[4][2] = SQ2H * n[0];
  N[5][0] = SQ2H * n[1];
  N[5][1] = SQ2H * n[0];
}

// adjoint of N with respect to n
__device__ __forceinline__ void nmat_adj(const double Nb[6][3], double* nb) {
  nb[0] = Nb[0][0] + SQ2H * (Nb[4][2] + Nb[5][1]);
  nb[1] = Nb[1][1] + SQ2H * (Nb[3][2] + Nb[5][0]);
  nb[2] = Nb[2][2] + SQ2H * (Nb[3][1] + Nb[4][0]);
}

// inverse of a 3 x 3 matrix by the adjugate; false if singular
__device__ __forceinline__ bool inv3(const double M[3][3], double R[3][3]) {
  const double c00 = M[1][1] * M[2][2] - M[1][2] * M[2][1];
  const double c01 = M[1][2] * M[2][0] - M[1][0] * M[2][2];
  const double c02 = M[1][0] * M[2][1] - M[1][1] * M[2][0];
  const double det = M[0][0] * c00 + M[0][1] * c01 + M[0][2] * c02;
  double scale = 0.0;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) scale = fmax(scale, fabs(M[i][j]));
  if (!(fabs(det) > 1e-13 * scale * scale * scale)) return false;
  const double id = 1.0 / det;
  R[0][0] = c00 * id;
  R[1][0] = c01 * id;
  R[2][0] = c02 * id;
  R[0][1] = (M[0][2] * M[2][1] - M[0][1] * M[2][2]) * id;
  R[1][1] = (M[0][0] * M[2][2] - M[0][2] * M[2][0]) * id;
  R[2][1] = (M[0][1] * M[2][0] - M[0][0] * M[2][1]) * id;
  R[0][2] = (M[0][1] * M[1][2] - M[0][2] * M[1][1]) * id;
  R[1][2] = (M[0][2] * M[1][0] - M[0][0] * M[1][2]) * id;
  R[2][2] = (M[0][0] * M[1][1] - M[0][1] * M[1][0]) * id;
  return true;
}

__device__ __forceinline__ void unit(const double* m, double* n, double& len) {
  len = sqrt(m[0] * m[0] + m[1] * m[1] + m[2] * m[2]);
  const double il = len > 0.0 ? 1.0 / len : 0.0;
  n[0] = m[0] * il;
  n[1] = m[1] * il;
  n[2] = m[2] * il;
}

// parameter index of the direction of heap node h at depth level k (2^(k-1) <= h < 2^k)
__device__ __forceinline__ int param_of(int h, int nleaf) {
  const int cnt = 1 << (31 - __clz(h));  // 2^(k-1)
  return nleaf - 2 * cnt + (h - cnt);
}

// ---------------------------------------------------------------------------
// offline: laminate forward and backward, eight lanes a laminate
// ---------------------------------------------------------------------------
// Lane r < 6 of a group of eight owns row r of the 6 x 6 matrices (lanes 6 and
// 7 repeat row 5 and add nothing to sums). With one thread a laminate a tree of
// depth 8 was a chain of sixteen levels of 7 to 20 us each (1500 FP64
// operations, uncoalesced rows, spills): 60 us forward and 180 us backward for
// 32 samples, now 49 us for both; the update 25 -> 13 us. What is left is the
// latency of the levels, of which the upper ones hold few laminates.

// sum over the eight lanes of a group, in all of them
__device__ __forceinline__ double dpp_add(double v, int lo, int hi) { return v + __hiloint2double(hi, lo); }
#define HOM_DPP_ADD(v, ctrl)                                                                       \
  dpp_add(v, __builtin_amdgcn_mov_dpp(__double2loint(v), ctrl, 0xf, 0xf, true),                    \
          __builtin_amdgcn_mov_dpp(__double2hiint(v), ctrl, 0xf, 0xf, true))
__device__ __forceinline__ double sum8(double v) {
  v = HOM_DPP_ADD(v, 0xB1);   // quad_perm [1,0,3,2]
  v = HOM_DPP_ADD(v, 0x4E);   // quad_perm [2,3,0,1]
  return HOM_DPP_ADD(v, 0x141);  // row_half_mirror: the other quad of the eight
}
#undef HOM_DPP_ADD

// d^T N and x . N_j of N (6 x 3, Mandel, a -> sym(a (x) n)), without its zeros
__device__ __forceinline__ void row_times_n(const double* d, const double* n, double* g) {
  g[0] = d[0] * n[0] + SQ2H * (d[4] * n[2] + d[5] * n[1]);
  g[1] = d[1] * n[1] + SQ2H * (d[3] * n[2] + d[5] * n[0]);
  g[2] = d[2] * n[2] + SQ2H * (d[3] * n[1] + d[4] * n[0]);
}
__device__ __forceinline__ void n_rows_dot(const double* x, const double* n, double* y) {
  y[0] = x[0] * n[0];
  y[1] = x[1] * n[1];
  y[2] = x[2] * n[2];
  y[3] = SQ2H * (x[1] * n[2] + x[2] * n[1]);
  y[4] = SQ2H * (x[0] * n[2] + x[2] * n[0]);
  y[5] = SQ2H * (x[0] * n[1] + x[1] * n[0]);
}
// row r of N
__device__ __forceinline__ void n_row(int r, const double* n, double* nr) {
  const double s0 = SQ2H * n[0], s1 = SQ2H * n[1], s2 = SQ2H * n[2];
  nr[0] = r == 0 ? n[0] : (r == 4 ? s2 : (r == 5 ? s1 : 0.0));
  nr[1] = r == 1 ? n[1] : (r == 3 ? s2 : (r == 5 ? s0 : 0.0));
  nr[2] = r == 2 ? n[2] : (r == 3 ? s1 : (r == 4 ? s0 : 0.0));
}

// What both directions form first: row r of C1, C2, of G = (C1 - C2) N and of
// HN = (c2 C1 + c1 C2) N, and M^-1 of M = N^T HN.
struct Lam8 {
  double a[6], b[6], G[3], HN[3], nr[3], Mi[3][3];
  __device__ __forceinline__ void form(const double* C1, const double* C2, double c1, const double* n, int row,
                                       bool own) {
    const double c2 = 1.0 - c1;
    double d[6], e[6];
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      a[j] = C1[6 * row + j];
      b[j] = C2[6 * row + j];
      d[j] = a[j] - b[j];
      e[j] = c2 * a[j] + c1 * b[j];
    }
    row_times_n(d, n, G);
    row_times_n(e, n, HN);
    n_row(row, n, nr);
    double M[3][3];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int l = 0; l < 3; ++l) M[k][l] = sum8(own ? nr[k] * HN[l] : 0.0);
    if (!inv3(M, Mi)) {
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int l = 0; l < 3; ++l) Mi[k][l] = 0.0;
    }
  }
};

__device__ __forceinline__ void times_mi(const double* g, const double Mi[3][3], double* gm) {
#pragma unroll
  for (int k = 0; k < 3; ++k) gm[k] = g[0] * Mi[0][k] + g[1] * Mi[1][k] + g[2] * Mi[2][k];
}

// the rows v (3 values) of the six lanes, through the group's scratch in LDS;
// the lanes are in one wave, whose LDS accesses are in order
__device__ __forceinline__ void share_rows(const double* v, double* scr, int row, double (&all)[6][3]) {
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int k = 0; k < 3; ++k) scr[3 * row + k] = v[k];
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int j = 0; j < 6; ++j)
#pragma unroll
    for (int k = 0; k < 3; ++k) all[j][k] = scr[3 * j + k];
  __builtin_amdgcn_wave_barrier();
}

constexpr int SCR8 = 18;  // scratch of a group

__device__ __forceinline__ void lam_fwd8(const double* C1, const double* C2, double c1, const double* n, double* C,
                                         int row, bool own, double* scr) {
  const double c2 = 1.0 - c1;
  Lam8 m;
  m.form(C1, C2, c1, n, row, own);
  double GM[3], G[6][3];
  times_mi(m.G, m.Mi, GM);
  share_rows(m.G, scr, row, G);
  const double cc = c1 * c2;
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    const double v = c1 * m.a[j] + c2 * m.b[j] - cc * (GM[0] * G[j][0] + GM[1] * G[j][1] + GM[2] * G[j][2]);
    if (own) C[6 * row + j] = v;
  }
}

// Reverse mode of lam_fwd8: given Cb = dJ/dC, writes dJ/dC1, dJ/dC2 (if the
// pointers are non-null; they may be C1 and C2), dJ/dc1 and dJ/dn.
__device__ __forceinline__ void lam_bwd8(const double* C1, const double* C2, double c1, const double* n,
                                         const double* Cb, double* C1b, double* C2b, double& c1b, double* nb, int row,
                                         bool own, double* scr) {
  const double c2 = 1.0 - c1;
  const double cc = c1 * c2;
  Lam8 m;
  m.form(C1, C2, c1, n, row, own);
  double cr[6], ck[6], dk[6];  // row and column of Cb, column of C1 - C2
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    cr[j] = Cb[6 * row + j];
    ck[j] = Cb[6 * j + row];
    dk[j] = C1[6 * j + row] - C2[6 * j + row];
  }
  // C = c1 C1 + c2 C2 - cc X, X = G Mi G^T = GM G^T. With T = Cb G:
  //   <Cb, X> = <GM, T>, dJ/dMi = -cc G^T T, dJ/dG = -cc (Cb + Cb^T) GM
  double GM[3], T[3], Gb[3], all[6][3];
  times_mi(m.G, m.Mi, GM);
  share_rows(m.G, scr, row, all);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    double t = 0.0;
#pragma unroll
    for (int j = 0; j < 6; ++j) t += cr[j] * all[j][k];
    T[k] = t;
  }
  share_rows(GM, scr, row, all);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    double u = 0.0;
#pragma unroll
    for (int j = 0; j < 6; ++j) u += (cr[j] + ck[j]) * all[j][k];
    Gb[k] = -cc * u;
  }
  double dd = 0.0;
#pragma unroll
  for (int j = 0; j < 6; ++j) dd += cr[j] * (m.a[j] - m.b[j]);
  dd = sum8(own ? dd : 0.0);                                                   // <Cb, C1 - C2>
  const double dx = sum8(own ? GM[0] * T[0] + GM[1] * T[1] + GM[2] * T[2] : 0.0);  // <Cb, X>
  double Mib[3][3];
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int l = 0; l < 3; ++l) Mib[k][l] = -cc * sum8(own ? m.G[k] * T[l] : 0.0);
  // Mi = M^-1: Mb = -Mi Mib Mi (Mi symmetric)
  double W[3][3], Mb[3][3];
#pragma unroll
  for (int k = 0; k < 3; ++k) times_mi(Mib[k], m.Mi, W[k]);
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int l = 0; l < 3; ++l)
      Mb[k][l] = -(m.Mi[k][0] * W[0][l] + m.Mi[k][1] * W[1][l] + m.Mi[k][2] * W[2][l]);
  // M = N^T H N, H = c2 C1 + c1 C2: Hb = N Mb N^T, Nb = HN (Mb + Mb^T);
  // G = (C1 - C2) N: Nb += (C1 - C2)^T Gb, (C1 - C2)b = Gb N^T
  share_rows(Gb, scr, row, all);
  double Nb[3], NM[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    double s = 0.0;
#pragma unroll
    for (int l = 0; l < 3; ++l) s += m.HN[l] * (Mb[k][l] + Mb[l][k]);
#pragma unroll
    for (int i = 0; i < 6; ++i) s += dk[i] * all[i][k];
    Nb[k] = s;
    NM[k] = m.nr[0] * Mb[0][k] + m.nr[1] * Mb[1][k] + m.nr[2] * Mb[2][k];
  }
  double hb[6], db[6], dh = 0.0;  // <Hb, C2 - C1>
  n_rows_dot(NM, n, hb);
  n_rows_dot(Gb, n, db);
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    dh += hb[j] * (m.b[j] - m.a[j]);
    if (own) {
      if (C1b) C1b[6 * row + j] = c1 * cr[j] + c2 * hb[j] + db[j];
      if (C2b) C2b[6 * row + j] = c2 * cr[j] + c1 * hb[j] - db[j];
    }
  }
  c1b = dd - (1.0 - 2.0 * c1) * dx + sum8(own ? dh : 0.0);
  // adjoint of N with respect to n: every row adds where n enters it
  nb[0] = sum8(!own ? 0.0 : (row == 0 ? Nb[0] : (row == 4 ? SQ2H * Nb[2] : (row == 5 ? SQ2H * Nb[1] : 0.0))));
  nb[1] = sum8(!own ? 0.0 : (row == 1 ? Nb[1] : (row == 3 ? SQ2H * Nb[2] : (row == 5 ? SQ2H * Nb[0] : 0.0))));
  nb[2] = sum8(!own ? 0.0 : (row == 2 ? Nb[2] : (row == 3 ? SQ2H * Nb[1] : (row == 4 ? SQ2H * Nb[0] : 0.0))));
}

// threads of an offline work-group (one sample): 64 laminates at a time, half
// the bottom level of a depth-8 tree
constexpr int OFF_THREADS = 512;

struct OffArgs {
  int K, nleaf;
  const double* p;     // m [nnode][3], v [nleaf]
  const double* C1;    // [S][36]
  const double* C2;
  const double* Cb;    // [S][36] targets, or null
  int first;           // number of the launch's first block
  const int* idx;      // [B] sample of each block, or null (block = sample)
  double* Cnode;       // [B][nleaf][36] (heap index 1 .. nleaf - 1) of trees that do not fit into LDS
  double* D;           // [B][36] prediction, or null
  double q;            // exponent of the loss
  double* err;         // [2][B] relative l1 errors e: e^q, then e^(q - 1); then the sum of the weights
  int B;
  double* grad;        // [B][nparam] gradients of every sample's error, or null (forward only)
};

// Trees up to this depth keep their nodes' stiffnesses in LDS (72 KB at 8).
constexpr int OFF_LDS_K = 8;
constexpr size_t off_lds(int nleaf, bool nodes) {
  return sizeof(double) * ((size_t)4 * nleaf + (OFF_THREADS / 8) * SCR8 + (nodes ? (size_t)nleaf * 36 : 0));
}

// Forward and, with a.grad, reverse mode of one sample: the effective
// stiffness and its error e_s = |T - C|_1 / |T|_1, then de_s / dparameters
// (the batch's loss weighs them by dJ/de_s, which needs all errors, in the
// update kernel). A node's adjoint takes the place of its stiffness, which its
// parent's reverse step is the last to read.
template <bool NODES>
__global__ void __launch_bounds__(OFF_THREADS) k_dmn_sample(OffArgs a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* wsub = reinterpret_cast<double*>(smem_raw);  // subtree weights, heap order
  double* wbar = wsub + 2 * a.nleaf;
  double* scr = wbar + 2 * a.nleaf + (threadIdx.x >> 3) * SCR8;
  double* node = NODES ? wbar + 2 * a.nleaf + (OFF_THREADS / 8) * SCR8
                       : a.Cnode + (long long)(a.first + blockIdx.x) * a.nleaf * 36;
  __shared__ double den_s, err_s;
  const int s = a.first + blockIdx.x;
  const int sample = a.idx ? a.idx[s] : s;
  const int nleaf = a.nleaf;
  const int tid = threadIdx.x, nth = blockDim.x;
  const int row = min(tid & 7, 5);
  const bool own = (tid & 7) < 6;
  const double* v = a.p + 3 * (nleaf - 1);
  for (int l = tid; l < nleaf; l += nth) wsub[nleaf + l] = fmax(v[l], 0.0);
  __syncthreads();
  for (int cnt = nleaf >> 1; cnt >= 1; cnt >>= 1) {
    for (int j = tid; j < cnt; j += nth) wsub[cnt + j] = wsub[2 * (cnt + j)] + wsub[2 * (cnt + j) + 1];
    __syncthreads();
  }
  const auto child = [&](int h) -> const double* {
    if (h >= nleaf) return (((h - nleaf) & 1) ? a.C2 : a.C1) + (long long)sample * 36;
    return node + h * 36;
  };
  const auto fraction = [&](int h) {
    const double wl = wsub[2 * h], sw = wl + wsub[2 * h + 1];
    return sw > 0.0 ? wl / sw : 0.5;
  };
  for (int cnt = nleaf >> 1; cnt >= 1; cnt >>= 1) {
    for (int j = tid >> 3; j < cnt; j += nth >> 3) {
      const int h = cnt + j;
      double n[3], len;
      unit(a.p + 3 * param_of(h, nleaf), n, len);
      lam_fwd8(child(2 * h), child(2 * h + 1), fraction(h), n, node + h * 36, row, own, scr);
    }
    __syncthreads();
  }
  double* root = node + 36;
  if (a.D && tid < 36) a.D[(long long)s * 36 + tid] = root[tid];
  const double* Tg = a.Cb ? a.Cb + (long long)sample * 36 : nullptr;
  if (Tg && tid == 0) {
    double num = 0.0, den = 0.0;
    for (int i = 0; i < 36; ++i) {
      num += fabs(Tg[i] - root[i]);
      den += fabs(Tg[i]);
    }
    err_s = num / den;
    den_s = den;
    if (s == 0) a.err[2 * a.B] = wsub[1];
    wbar[1] = 0.0;  // the mixing penalty is added once per batch by the update kernel
  }
  if (!a.grad) return;
  __syncthreads();
  if (tid == nth - 1) {  // of the last wave, which waits through the first levels below
    a.err[s] = pow(err_s, a.q);
    a.err[a.B + s] = pow(err_s, a.q - 1.0);
  }
  if (tid < 36) {
    const double d = Tg[tid] - root[tid];
    root[tid] = d > 0.0 ? -1.0 / den_s : (d < 0.0 ? 1.0 / den_s : 0.0);
  }
  __syncthreads();
  double* grad = a.grad + (long long)s * (3 * (nleaf - 1) + nleaf);
  for (int cnt = 1; cnt < nleaf; cnt <<= 1) {
    for (int j = tid >> 3; j < cnt; j += nth >> 3) {
      const int h = cnt + j;
      const int pi = param_of(h, nleaf);
      double n[3], len;
      unit(a.p + 3 * pi, n, len);
      const bool inner = 2 * h < nleaf;
      double c1b, nb[3];
      lam_bwd8(child(2 * h), child(2 * h + 1), fraction(h), n, node + h * 36, inner ? node + 2 * h * 36 : nullptr,
               inner ? node + (2 * h + 1) * 36 : nullptr, c1b, nb, row, own, scr);
      if ((tid & 7) == 0) {
        // n = m / |m|
        const double dn = nb[0] * n[0] + nb[1] * n[1] + nb[2] * n[2];
        const double il = len > 0.0 ? 1.0 / len : 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) grad[3 * pi + k] = (nb[k] - dn * n[k]) * il;
        // c1 = wl / (wl + wr); the node weight wl + wr passes its adjoint down
        const double wl = wsub[2 * h], wr = wsub[2 * h + 1], sw = wl + wr;
        double gl = wbar[h], gr = wbar[h];
        if (sw > 0.0) {
          gl += c1b * wr / (sw * sw);
          gr -= c1b * wl / (sw * sw);
        }
        wbar[2 * h] = gl;
        wbar[2 * h + 1] = gr;
      }
    }
    __syncthreads();
  }
  for (int l = tid; l < nleaf; l += nth) grad[3 * (nleaf - 1) + l] = v[l] > 0.0 ? wbar[nleaf + l] : 0.0;
}

struct StepArgs {
  int nparam, nnode, nleaf, B;
  double* p;
  double *a1, *a2, *a2max;
  const double* grad;   // [B][nparam] of the samples' errors
  const double* err;    // [2][B] e^q and e^(q - 1) of the samples, then the sum of the weights
  double* gout;         // [nparam] summed gradient (or null)
  double* loss;         // loss of this batch (or null)
  double* loss_acc;     // accumulated batch losses (or null)
  double lr, q, penalty, beta1, beta2, eps;
  double bc1, bc2;      // bias corrections of this step
  int update;
};

// loss value J = (1/B) (sum_s e_s^q)^(1/q) + penalty (sum w - 1)^2, its gradient
// (the per-sample gradients weighed by dJ/de_s = (1/B) (sum e^q)^(1/q - 1)
// e_s^(q - 1) and summed in a fixed order, plus the mixing penalty) and the
// AMSGrad update, a parameter a thread. Latency-bound: 5.7 us for 1021
// parameters of 32 samples; on one work-group that formed the powers and the
// sum of the weights first, 13.4 us.
constexpr int STEP_THREADS = 256;
__global__ void __launch_bounds__(STEP_THREADS) k_dmn_step(StepArgs a) {
  __shared__ double red[16];
  __shared__ double tot;
  const double* v = a.p + 3 * a.nnode;
  const int i = blockIdx.x * STEP_THREADS + threadIdx.x;
  double g = 0.0;
  if (i < a.nparam) {
#pragma unroll 8
    for (int b = 0; b < a.B; ++b) g += a.err[a.B + b] * a.grad[(long long)b * a.nparam + i];
  }
  double r[1] = {0.0};
  for (int b = threadIdx.x; b < a.B; b += STEP_THREADS) r[0] += a.err[b];
  block_sum<1>(r, red);
  if (threadIdx.x == 0) tot = r[0];
  __syncthreads();
  const double sq = tot, off = a.err[2 * a.B] - 1.0;
  if (i == 0 && (a.loss || a.loss_acc)) {
    const double J = pow(sq, 1.0 / a.q) / a.B + a.penalty * off * off;
    if (a.loss) *a.loss = J;
    if (a.loss_acc) *a.loss_acc += J;
  }
  if (i >= a.nparam) return;
  g = sq > 0.0 ? pow(sq, 1.0 / a.q - 1.0) / a.B * g : 0.0;
  if (i >= 3 * a.nnode && v[i - 3 * a.nnode] > 0.0) g += 2.0 * a.penalty * off;
  if (a.gout) a.gout[i] = g;
  if (!a.update) return;
  const double m1 = a.beta1 * a.a1[i] + (1.0 - a.beta1) * g;
  const double m2 = a.beta2 * a.a2[i] + (1.0 - a.beta2) * g * g;
  const double mx = fmax(a.a2max[i], m2);
  a.a1[i] = m1;
  a.a2[i] = m2;
  a.a2max[i] = mx;
  a.p[i] -= a.lr * (m1 / a.bc1) / (sqrt(mx / a.bc2) + a.eps);
}

template <typename U>
U* dalloc_into(std::vector<void*>& allocs, size_t count) {
  void* ptr = nullptr;
  hip_check(hipMalloc(&ptr, count * sizeof(U) + 256), "hipMalloc");
  allocs.push_back(ptr);
  hip_check(hipMemset(ptr, 0, count * sizeof(U)), "hipMemset");
  return static_cast<U*>(ptr);
}

// One launch, or several where one would have 2^32 threads or more (from 2^23
// samples of depth 7 on), which a launch does not run.
void launch_samples(OffArgs a, int B, hipStream_t stream) {
  const int threads = std::min(OFF_THREADS, std::max(64, 4 * a.nleaf));  // eight lanes a laminate
  const bool nodes = a.K <= OFF_LDS_K;
  const size_t lds = off_lds(a.nleaf, nodes);
  if (nodes && lds > 65536)
    hip_check(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_dmn_sample<true>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds),
              "hipFuncSetAttribute");
  constexpr int kMost = 1 << 22;
  for (a.first = 0;; a.first += kMost) {
    const dim3 groups(std::min(B - a.first, kMost));
    if (nodes)
      hipLaunchKernelGGL(k_dmn_sample<true>, groups, dim3(threads), lds, stream, a);
    else
      hipLaunchKernelGGL(k_dmn_sample<false>, groups, dim3(threads), lds, stream, a);
    hip_check(hipGetLastError(), "k_dmn_sample");
    if (B - a.first <= kMost) return;
  }
}
// node stiffnesses in memory, for the trees that do not fit into LDS
size_t node_doubles(int K, long long B) { return K <= OFF_LDS_K ? 1 : (size_t)B * ((size_t)1 << K) * 36; }
void launch_step(const StepArgs& s, hipStream_t stream) {
  hipLaunchKernelGGL(k_dmn_step, dim3((s.nparam + STEP_THREADS - 1) / STEP_THREADS), dim3(STEP_THREADS), 0, stream, s);
  hip_check(hipGetLastError(), "k_dmn_step");
}

}  // namespace

// ---------------------------------------------------------------------------
// Dmn host object
// ---------------------------------------------------------------------------
Dmn::Dmn(int K_, uint64_t seed) : K(K_) {
  if (K < 1 || K > DMN_MAX_K) fail(HOM_E_ARG, "DMN depth must be in [1, 10]");
  nleaf = 1 << K;
  nnode = nleaf - 1;
  nparam = 3 * nnode + nleaf;
  p = dalloc_into<double>(allocs, nparam);
  a1 = dalloc_into<double>(allocs, nparam);
  a2 = dalloc_into<double>(allocs, nparam);
  a2max = dalloc_into<double>(allocs, nparam);
  // directions uniform on the unit sphere, weights uniform on [0, 1] rescaled
  // to sum to one (the paper's initialization)
  std::mt19937_64 rng(seed);
  std::normal_distribution<double> nd(0.0, 1.0);
  std::uniform_real_distribution<double> ud(0.0, 1.0);
  std::vector<double> h(nparam);
  for (int i = 0; i < nnode; ++i) {
    double x, y, z, r;
    do {
      x = nd(rng);
      y = nd(rng);
      z = nd(rng);
      r = std::sqrt(x * x + y * y + z * z);
    } while (r < 1e-12);
    h[3 * i] = x / r;
    h[3 * i + 1] = y / r;
    h[3 * i + 2] = z / r;
  }
  double sw = 0.0;
  for (int l = 0; l < nleaf; ++l) sw += (h[3 * nnode + l] = ud(rng));
  for (int l = 0; l < nleaf; ++l) h[3 * nnode + l] /= sw;
  hip_check(hipMemcpy(p, h.data(), nparam * sizeof(double), hipMemcpyHostToDevice), "hipMemcpy");
}

Dmn::~Dmn() {
  for (void* ptr : allocs) (void)hipFree(ptr);
}

void Dmn::get(double* m, double* v) const {
  std::vector<double> h(nparam);
  hip_check(hipMemcpy(h.data(), p, nparam * sizeof(double), hipMemcpyDeviceToHost), "hipMemcpy");
  if (m) std::memcpy(m, h.data(), 3 * nnode * sizeof(double));
  if (v) std::memcpy(v, h.data() + 3 * nnode, nleaf * sizeof(double));
}

void Dmn::set(const double* m, const double* v) {
  std::vector<double> h(nparam);
  get(h.data(), h.data() + 3 * nnode);
  if (m) std::memcpy(h.data(), m, 3 * nnode * sizeof(double));
  if (v) std::memcpy(h.data() + 3 * nnode, v, nleaf * sizeof(double));
  for (int i = 0; i < nnode; ++i)
    if (!(h[3 * i] * h[3 * i] + h[3 * i + 1] * h[3 * i + 1] + h[3 * i + 2] * h[3 * i + 2] > 0.0))
      fail(HOM_E_ARG, "direction " + std::to_string(i) + " is zero");
  for (double x : h)
    if (!std::isfinite(x)) fail(HOM_E_ARG, "parameters must be finite");
  hip_check(hipMemcpy(p, h.data(), nparam * sizeof(double), hipMemcpyHostToDevice), "hipMemcpy");
  steps = 0;
  hip_check(hipMemset(a1, 0, nparam * sizeof(double)), "hipMemset");
  hip_check(hipMemset(a2, 0, nparam * sizeof(double)), "hipMemset");
  hip_check(hipMemset(a2max, 0, nparam * sizeof(double)), "hipMemset");
}

namespace {
void check_samples(long long n, const double* C1, const double* C2) {
  if (n < 1) fail(HOM_E_ARG, "need at least one sample");
  if (!C1 || !C2) fail(HOM_E_ARG, "null stiffness array");
  for (long long i = 0; i < 36 * n; ++i)
    if (!std::isfinite(C1[i]) || !std::isfinite(C2[i])) fail(HOM_E_ARG, "stiffnesses must be finite");
}

struct DevSamples {
  std::vector<void*> allocs;
  double *C1 = nullptr, *C2 = nullptr, *Cb = nullptr;
  DevSamples(long long n, const double* c1, const double* c2, const double* cb) {
    C1 = dalloc_into<double>(allocs, 36 * n);
    C2 = dalloc_into<double>(allocs, 36 * n);
    hip_check(hipMemcpy(C1, c1, 36 * n * sizeof(double), hipMemcpyHostToDevice), "hipMemcpy");
    hip_check(hipMemcpy(C2, c2, 36 * n * sizeof(double), hipMemcpyHostToDevice), "hipMemcpy");
    if (cb) {
      Cb = dalloc_into<double>(allocs, 36 * n);
      hip_check(hipMemcpy(Cb, cb, 36 * n * sizeof(double), hipMemcpyHostToDevice), "hipMemcpy");
    }
  }
  ~DevSamples() {
    for (void* p : allocs) (void)hipFree(p);
  }
};
}  // namespace

void Dmn::homogenize(long long n, const double* C1, const double* C2, double* Cout) {
  check_samples(n, C1, C2);
  if (!Cout) fail(HOM_E_ARG, "null output");
  DevSamples d(n, C1, C2, nullptr);
  std::vector<void*> tmp;
  OffArgs a{};
  a.K = K;
  a.nleaf = nleaf;
  a.p = p;
  a.C1 = d.C1;
  a.C2 = d.C2;
  a.Cnode = dalloc_into<double>(tmp, node_doubles(K, n));
  a.D = dalloc_into<double>(tmp, (size_t)n * 36);
  launch_samples(a, (int)n, nullptr);
  hip_check(hipMemcpy(Cout, a.D, 36 * n * sizeof(double), hipMemcpyDeviceToHost), "hipMemcpy");
  for (void* ptr : tmp) (void)hipFree(ptr);
}

double Dmn::loss_grad(long long n, const double* C1, const double* C2, const double* Cb, double* gm, double* gv,
                      const DmnSchedule& sc) {
  check_samples(n, C1, C2);
  if (!Cb) fail(HOM_E_ARG, "null targets");
  DevSamples d(n, C1, C2, Cb);
  std::vector<void*> tmp;
  OffArgs a{};
  a.K = K;
  a.nleaf = nleaf;
  a.p = p;
  a.C1 = d.C1;
  a.C2 = d.C2;
  a.Cb = d.Cb;
  a.Cnode = dalloc_into<double>(tmp, node_doubles(K, n));
  a.q = sc.q;
  a.B = (int)n;
  a.err = dalloc_into<double>(tmp, 2 * (size_t)n + 1);
  a.grad = dalloc_into<double>(tmp, (size_t)n * nparam);
  launch_samples(a, (int)n, nullptr);
  StepArgs s{};
  s.nparam = nparam;
  s.nnode = nnode;
  s.nleaf = nleaf;
  s.B = (int)n;
  s.p = p;
  s.grad = a.grad;
  s.err = a.err;
  s.gout = dalloc_into<double>(tmp, nparam);
  s.loss = dalloc_into<double>(tmp, 1);
  s.q = sc.q;
  s.penalty = sc.penalty;
  s.update = 0;
  s.beta1 = sc.beta1;
  s.beta2 = sc.beta2;
  launch_step(s, nullptr);
  std::vector<double> g(nparam);
  double J = 0.0;
  hip_check(hipMemcpy(g.data(), s.gout, nparam * sizeof(double), hipMemcpyDeviceToHost), "hipMemcpy");
  hip_check(hipMemcpy(&J, s.loss, sizeof(double), hipMemcpyDeviceToHost), "hipMemcpy");
  if (gm) std::memcpy(gm, g.data(), 3 * nnode * sizeof(double));
  if (gv) std::memcpy(gv, g.data() + 3 * nnode, nleaf * sizeof(double));
  for (void* ptr : tmp) (void)hipFree(ptr);
  return J;
}

void Dmn::train(long long n, const double* C1, const double* C2, const double* Cb, int epochs, int batch,
                uint64_t seed, double* loss_hist, const DmnSchedule& sc) {
  check_samples(n, C1, C2);
  if (!Cb) fail(HOM_E_ARG, "null targets");
  if (batch < 1 || batch > n) fail(HOM_E_ARG, "batch must be in [1, n]");
  if (epochs < 0) fail(HOM_E_ARG, "epochs must be >= 0");
  DevSamples d(n, C1, C2, Cb);
  std::vector<void*> tmp;
  OffArgs a{};
  a.K = K;
  a.nleaf = nleaf;
  a.p = p;
  a.C1 = d.C1;
  a.C2 = d.C2;
  a.Cb = d.Cb;
  a.Cnode = dalloc_into<double>(tmp, node_doubles(K, batch));
  a.q = sc.q;
  a.B = batch;
  a.err = dalloc_into<double>(tmp, 2 * (size_t)batch + 1);
  a.grad = dalloc_into<double>(tmp, (size_t)batch * nparam);
  const long long nb = n / batch;  // incomplete batches are dropped
  int* idx = dalloc_into<int>(tmp, (size_t)nb * batch);
  double* lacc = dalloc_into<double>(tmp, std::max(epochs, 1));
  std::vector<int> perm(n);
  std::mt19937_64 rng(seed);
  StepArgs s{};
  s.nparam = nparam;
  s.nnode = nnode;
  s.nleaf = nleaf;
  s.B = batch;
  s.p = p;
  s.a1 = a1;
  s.a2 = a2;
  s.a2max = a2max;
  s.grad = a.grad;
  s.err = a.err;
  s.q = sc.q;
  s.penalty = sc.penalty;
  s.beta1 = sc.beta1;
  s.beta2 = sc.beta2;
  s.eps = sc.eps;
  s.update = 1;
  const double pi = 3.14159265358979323846;
  for (int e = 0; e < epochs; ++e) {
    for (long long i = 0; i < n; ++i) perm[i] = (int)i;
    std::shuffle(perm.begin(), perm.end(), rng);
    hip_check(hipMemcpy(idx, perm.data(), nb * batch * sizeof(int), hipMemcpyHostToDevice), "hipMemcpy");
    // harmonic modulation with geometric decay (the paper's warm restarts)
    s.lr = std::pow(sc.decay, e) *
           (sc.lr_min + 0.5 * (sc.lr_max - sc.lr_min) * (1.0 + std::cos(pi * e / sc.half_period)));
    s.loss_acc = lacc + e;
    for (long long b = 0; b < nb; ++b) {
      a.idx = idx + b * batch;
      launch_samples(a, batch, nullptr);
      ++steps;
      s.bc1 = 1.0 - std::pow(sc.beta1, (double)steps);
      s.bc2 = 1.0 - std::pow(sc.beta2, (double)steps);
      launch_step(s, nullptr);
    }
  }
  hip_check(hipDeviceSynchronize(), "dmn training");
  if (loss_hist && epochs > 0) {
    hip_check(hipMemcpy(loss_hist, lacc, epochs * sizeof(double), hipMemcpyDeviceToHost), "hipMemcpy");
    for (int e = 0; e < epochs; ++e) loss_hist[e] /= (double)nb;
  }
  for (void* ptr : tmp) (void)hipFree(ptr);
}

// ---------------------------------------------------------------------------
// online evaluation (paper Sec. 3.3): Newton's method on the jumps of the
// whole tree for many macroscopic points, one wave per point.
//
// Lane t of a point owns the subtree of R = K - S levels below the depth-S
// node 2^S + t (S = min(K, 6)), i.e. 2^R leaves whose data stay in its
// registers. The S levels above are combined across lanes with shuffles: the
// depth-d node j (heap 2^d + j) belongs to lane j 2^(S-d), its right child to
// lane j 2^(S-d) + 2^(S-d-1). Per-node data (the jumps, the elimination factors
// G, d0 and the last Newton step) are touched only by the owning lane: those of
// the 2^S - 1 nodes above depth S are in LDS during the call, those of the
// lane's own subtree in memory, 64 lanes to a line.
//
// A wave's time is a chain of latencies (four rounds of one wave per SIMD at
// 4096 points of depth 8; vector instructions fill half of it). With the nodes'
// fields of a lane side by side in memory (64 lines an access) and every level
// reading its node when it got there, a call of 4096 points of depth 8 took
// 1.55 ms and one of 300 points 0.34 ms; now, with the upper nodes in LDS, the
// lane's own factors loaded ahead of the shuffle levels and the leaf states held
// in registers, 1.14 and 0.29 ms. Two waves per SIMD at half the registers,
// without the LDS: 1.67 ms, bound by 8 GB of traffic.
//
// One bottom-up sweep forms the residual (weighted stress sums and the
// traction mismatch N^T (c2 s1 - c1 s2) of every laminate) and, in the same
// pass, eliminates the jumps: with the children's condensed tangents K1, K2
// and condensed stresses, X = (c2 K1 - c1 K2) N, M = N^T (c2^2 K1 + c1^2 K2) N,
// G = -M^-1 X^T, d0 = -M^-1 N^T (c2 s1' - c1 s2'), and the parent gets
// K = K1 + K2 + X G (the symmetric Schur complement) and s' = s1' + s2' + X d0.
// The top-down sweep turns a root strain change into the jumps' Newton steps
// da = d0 + G deps. The converged root tangent is the effective algorithmic
// tangent d<sigma>/dE.
// ---------------------------------------------------------------------------
namespace {

constexpr int ON_MAX_K = 8;
constexpr int ON_LANES = 64;  // one wave per point
constexpr int ON_WAVES = 1;   // of a SIMD, with all of its registers
constexpr int ON_SHUF = 6;    // levels combined across the lanes (2^6 = 64)
// per point: sigma 6, coupling, dissipation, dsde 36, dsdt 6, dDde 6, dDdt,
// residual, iterations, status
constexpr int ON_OUT = 64;
constexpr int O_DSDT = 44, O_DDDE = 50, O_DDDT = 56, O_RES = 57, O_IT = 58, O_ST = 59;
constexpr int ON_SCR = 24;  // per internal node: G (18), d0 (3), last Newton step (3)
constexpr int ON_NODE = 5;  // per heap node: unit direction (3), c1, subtree weight
constexpr int ON_LP = 16;   // per leaf: d sigma / d theta (6), d D / d eps (6), d D / d theta

// A node's or leaf's place in the arrays over them, laid out [group][field][stride]:
// the 64 lanes of a wave, each at the same node of its own subtree, touch
// consecutive doubles, and the fields of one group lie at constant distances. Nodes
// above depth S are group 0 in heap order; node k of the level r below depth S is
// group 2^r + k, leaf k of a lane's subtree group k, the index the lane.
struct Slot {
  int grp, idx;
};
// A node above depth S: its scratch, jump and table entry are in LDS while the
// kernel runs, [field][ON_LANES].
struct Top {
  int idx;
};
constexpr int TOP_JUMP = ON_SCR, TOP_TABLE = ON_SCR + 3, TOP_FIELDS = TOP_TABLE + ON_NODE;

struct OnArgs {
  int K, nleaf, S;
  const double* node;     // [group][ON_NODE][stride] of the network, then the leaf weights
  const ProbInc* inc;     // [distinct (theta, dt) of the call]
  const ProbInc* inc_pm;  // [distinct][2]: theta + h_theta, theta - h_theta (all four tangents)
  const int* inc_ix;      // [point] index into inc
  int what;               // 1: also the temperature and coupling tangents
  int trial;              // 1: never commit
  int pa_phase;           // phase (0: even leaves, 1: odd leaves) with the PA66 law, -1 if none
  double* state;          // [point][nstate][nleaf / 2]
  int nstate;
  double* hist;           // [point][HIST_SLOTS][nleaf / 2]
  double* epsn;           // [point][group][6][stride]
  double* a;              // [point][group][3][stride] jumps
  double* scr;            // [point][group][ON_SCR][stride]
  double* lp;             // [point][group][ON_LP][stride] leaf partials (what = 1)
  // predictor (pred = 1): jump change of the last committed increment, the
  // jumps at the start of this call and whether the point's last call
  // committed; the last committed macro strain and its change (kept with the
  // predictor off too)
  int pred;
  double* dah;            // [point][group][3][stride]
  double* a0;             // [point][group][3][stride]
  double* Ep;             // [point][12]: E of the last commit (6), its change (6)
  int* committed;         // [point]
  const double* E;        // [point][6] Mandel
  double* out;            // [point][ON_OUT]
  double tol, gamma;
  int maxit, maxbt;
};

// The arguments with the sizes known where there are register levels (then
// K = ON_SHUF + R).
template <int R_>
struct OnView : OnArgs {
  static constexpr int R = R_;
  double* top;  // LDS, [TOP_FIELDS][ON_LANES]
  __device__ int levels() const { return R > 0 ? ON_SHUF : S; }
  __device__ int leaves() const { return R > 0 ? ON_LANES << R : nleaf; }
  __device__ int stride() const { return R > 0 ? ON_LANES : nleaf; }
  // An offset worked out where it is used: kept over the sweeps, the addresses
  // of every node's fields fill the registers.
  static __device__ unsigned here(unsigned off) {
    asm volatile("" : "+v"(off));
    return off;
  }
  // first field of a slot of point pt; the next lie stride() apart
  __device__ double* at(double* base, int fields, int pt, Slot s) const {
    return base + (long long)pt * leaves() * fields + here(s.grp * fields * stride() + s.idx);
  }
  __device__ const double* table(Slot s) const { return node + here(s.grp * ON_NODE * stride() + s.idx); }
  __device__ double leaf_weight(Slot l) const { return node[(unsigned)(ON_NODE * leaves() + l.grp * stride() + l.idx)]; }
  // scratch, jump and table entry of a node, and the distance of their fields
  __device__ double* scratch(int pt, Slot s) const { return at(scr, ON_SCR, pt, s); }
  __device__ double* scratch(int, Top t) const { return top + t.idx; }
  __device__ double* jump(int pt, Slot s) const { return at(a, 3, pt, s); }
  __device__ double* jump(int, Top t) const { return top + TOP_JUMP * ON_LANES + t.idx; }
  __device__ const double* table(Top t) const { return top + TOP_TABLE * ON_LANES + t.idx; }
  __device__ int stride(Slot) const { return stride(); }
  __device__ static constexpr int stride(Top) { return ON_LANES; }
  // the same node in the arrays
  static __device__ Slot slot(Slot s) { return s; }
  static __device__ Slot slot(Top t) { return Slot{0, t.idx}; }
  // index of a leaf among those of its phase
  __device__ unsigned phase_index(Slot l) const { return here(R > 0 ? (l.grp >> 1) * ON_LANES + l.idx : l.idx >> 1); }
};

// node table of a network: unit directions, c1 and subtree weights
__global__ void k_dmn_node_table(const double* p, int nleaf, int S, double* node) {
  if (blockIdx.x != 0 || threadIdx.x != 0) return;
  const double* v = p + 3 * (nleaf - 1);
  const int stride = nleaf < ON_LANES ? nleaf : ON_LANES;
  const auto weight = [&](int h) {  // place of a heap node's weight
    const int d = 31 - __builtin_clz(h), r = d - S, j = h - (1 << d);
    const int in = r < 0 ? 0 : j & ((1 << r) - 1), lane = r < 0 ? h : j >> r;
    if (h >= nleaf) return ON_NODE * nleaf + in * stride + lane;
    return ((r < 0 ? 0 : (1 << r) + in) * ON_NODE + 4) * stride + lane;
  };
  for (int l = 0; l < nleaf; ++l) node[weight(nleaf + l)] = fmax(v[l], 0.0);
  for (int h = nleaf - 1; h >= 1; --h) {
    const double wl = node[weight(2 * h)], wr = node[weight(2 * h + 1)], sw = wl + wr;
    double nh[3], len;
    unit(p + 3 * param_of(h, nleaf), nh, len);
    double* f = node + weight(h);
    for (int k = 0; k < 3; ++k) f[(k - 4) * stride] = nh[k];
    f[-stride] = sw > 0.0 ? wl / sw : 0.5;
    f[0] = sw;
  }
}

// packed index of the symmetric 6 x 6 entry (i, j)
__host__ __device__ constexpr int sx(int i, int j) {
  return i <= j ? i * 6 - (i * (i - 1)) / 2 + (j - i) : j * 6 - (j * (j - 1)) / 2 + (i - j);
}

// a leaf: weight, compressed tangent 3K P1 + ca P2 + cb N N, weighted stress (or source)
struct LeafV {
  double w, K3, ca, cb, nd[6];
  double s[6];
};
// a condensed subtree: tangent (packed symmetric, in the lane's LDS slot:
// entry e at K[e * ON_LANES]), plain and condensed stress sums
struct NodeV {
  double* K;
  double s[6], sp[6];
};

__device__ __forceinline__ double kent(const LeafV& a, int i, int q) {
  return a.w * ((i == q ? a.ca : 0.0) + (i < 3 && q < 3 ? (a.K3 - a.ca) * (1.0 / 3.0) : 0.0) + a.cb * a.nd[i] * a.nd[q]);
}
__device__ __forceinline__ double kent(const NodeV& a, int i, int q) { return a.K[sx(i, q) * ON_LANES]; }
__device__ __forceinline__ const double* plain(const LeafV& a) { return a.s; }
__device__ __forceinline__ const double* plain(const NodeV& a) { return a.s; }
__device__ __forceinline__ const double* cond(const LeafV& a) { return a.s; }
__device__ __forceinline__ const double* cond(const NodeV& a) { return a.sp; }

__device__ __forceinline__ void to_node(const LeafV& L, NodeV& v) {
#pragma unroll
  for (int i = 0; i < 6; ++i)
#pragma unroll
    for (int q = i; q < 6; ++q) v.K[sx(i, q) * ON_LANES] = kent(L, i, q);
#pragma unroll
  for (int c = 0; c < 6; ++c) v.s[c] = v.sp[c] = L.s[c];
}

// N a = sym(a (x) n) (Mandel) for the unit direction n
__device__ __forceinline__ void n_apply(const double* n, const double* a, double* v) {
  v[0] = n[0] * a[0];
  v[1] = n[1] * a[1];
  v[2] = n[2] * a[2];
  v[3] = SQ2H * (n[2] * a[1] + n[1] * a[2]);
  v[4] = SQ2H * (n[2] * a[0] + n[0] * a[2]);
  v[5] = SQ2H * (n[1] * a[0] + n[0] * a[1]);
}
// N^T v
__device__ __forceinline__ void nt_apply(const double* n, const double* v, double* r) {
  r[0] = n[0] * v[0] + SQ2H * (n[2] * v[4] + n[1] * v[5]);
  r[1] = n[1] * v[1] + SQ2H * (n[2] * v[3] + n[0] * v[5]);
  r[2] = n[2] * v[2] + SQ2H * (n[1] * v[3] + n[0] * v[4]);
}
// Laminate h from its children A (phase 1 side) and B: residual contribution
// (PLAIN: from the plain sums), elimination factors into the node's scratch,
// condensed tangent and stresses into P. P may be A itself: every entry of P
// is written after the last read of the same entry of A.
template <bool PLAIN, class G, class H, class CA, class CB>
__device__ __forceinline__ void combine(const G& g, int pt, H h, const CA& A, const CB& B, NodeV& P,
                                        double& gg) {
  const int st = g.stride(h);
  const double* nt = g.table(h);
  const double n[3] = {nt[0], nt[st], nt[2 * st]};
  const double c1 = nt[3 * st], c2 = 1.0 - c1, wsub = nt[4 * st];
  const double s0 = SQ2H * n[0], s1 = SQ2H * n[1], s2 = SQ2H * n[2];
  // X = (c2 K1 - c1 K2) N and M = N^T (c2^2 K1 + c1^2 K2) N, column by column
  double X[6][3], M[3][3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    double hc[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      double a1, a2;
      if (k == 0) {
        a1 = kent(A, i, 0) * n[0] + kent(A, i, 4) * s2 + kent(A, i, 5) * s1;
        a2 = kent(B, i, 0) * n[0] + kent(B, i, 4) * s2 + kent(B, i, 5) * s1;
      } else if (k == 1) {
        a1 = kent(A, i, 1) * n[1] + kent(A, i, 3) * s2 + kent(A, i, 5) * s0;
        a2 = kent(B, i, 1) * n[1] + kent(B, i, 3) * s2 + kent(B, i, 5) * s0;
      } else {
        a1 = kent(A, i, 2) * n[2] + kent(A, i, 3) * s1 + kent(A, i, 4) * s0;
        a2 = kent(B, i, 2) * n[2] + kent(B, i, 3) * s1 + kent(B, i, 4) * s0;
      }
      X[i][k] = c2 * a1 - c1 * a2;
      hc[i] = c2 * c2 * a1 + c1 * c1 * a2;
    }
    double mc[3];
    nt_apply(n, hc, mc);
#pragma unroll
    for (int q = 0; q < 3; ++q) M[q][k] = mc[q];
  }
  const double* p1 = cond(A);
  const double* p2 = cond(B);
  double dv[6], r[3];
#pragma unroll
  for (int c = 0; c < 6; ++c) dv[c] = c2 * p1[c] - c1 * p2[c];
  nt_apply(n, dv, r);
  if constexpr (PLAIN) {
    const double* q1 = plain(A);
    const double* q2 = plain(B);
    double pv[6], rp[3];
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      pv[c] = c2 * q1[c] - c1 * q2[c];
      P.s[c] = q1[c] + q2[c];
    }
    nt_apply(n, pv, rp);
    gg += rp[0] * rp[0] + rp[1] * rp[1] + rp[2] * rp[2];
  }
  // a subtree without weight on one side has no say in its jump: it stays
  double Mi[3][3];
  const bool ok = (c1 * c2 * wsub > 0.0) && inv3(M, Mi);
  double* sc = g.scratch(pt, h);
  double d0[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    d0[k] = ok ? -(Mi[k][0] * r[0] + Mi[k][1] * r[1] + Mi[k][2] * r[2]) : 0.0;
    sc[(18 + k) * st] = d0[k];
  }
#pragma unroll
  for (int i = 0; i < 6; ++i) P.sp[i] = p1[i] + p2[i] + X[i][0] * d0[0] + X[i][1] * d0[1] + X[i][2] * d0[2];
  // G = -M^-1 X^T one column at a time; K = K1 + K2 + X G
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    double gq[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      gq[k] = ok ? -(Mi[k][0] * X[q][0] + Mi[k][1] * X[q][1] + Mi[k][2] * X[q][2]) : 0.0;
      sc[(6 * k + q) * st] = gq[k];
    }
#pragma unroll
    for (int i = 0; i <= q; ++i)
      P.K[sx(i, q) * ON_LANES] =
          kent(A, i, q) + kent(B, i, q) + X[i][0] * gq[0] + X[i][1] * gq[1] + X[i][2] * gq[2];
  }
}

// children strains of laminate h: eps1 = eps + c2 N a, eps2 = eps - c1 N a
template <class G, class H>
__device__ __forceinline__ void split(const G& g, H h, const double* jump, const double* e, double* el, double* er) {
  const int st = g.stride(h);
  const double* nt = g.table(h);
  const double n[3] = {nt[0], nt[st], nt[2 * st]};
  const double c1 = nt[3 * st], c2 = 1.0 - c1;
  double jn[6];
  n_apply(n, jump, jn);
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    el[c] = e[c] + c2 * jn[c];
    er[c] = e[c] - c1 * jn[c];
  }
}

// ... at the node's current jump
template <class G, class H>
__device__ __forceinline__ void split_jump(const G& g, int pt, H h, const double* e, double* el, double* er) {
  const int st = g.stride(h);
  const double* ah = g.jump(pt, h);
  const double jump[3] = {ah[0], ah[st], ah[2 * st]};
  split(g, h, jump, e, el, er);
}

// Newton step of node h from the strain change of the node: da = d0 + G deps
// (kept in the scratch; added to the jump if `update`), and the children's
// strain changes
struct StepData {
  double G[18], d0[3];
};
template <class G, class H>
__device__ __forceinline__ void load_step(const G& g, int pt, H h, StepData& d) {
  const double* sc = g.scratch(pt, h);
  const int st = g.stride(h);
#pragma unroll
  for (int k = 0; k < 18; ++k) d.G[k] = sc[k * st];
#pragma unroll
  for (int k = 0; k < 3; ++k) d.d0[k] = sc[(18 + k) * st];
}
template <class G, class H>
__device__ __forceinline__ void node_step(const G& g, int pt, H h, const StepData& d, const double* de, bool update,
                                          double* dl, double* dr) {
  double* sc = g.scratch(pt, h);
  const int st = g.stride(h);
  double da[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    double x = d.d0[k];
#pragma unroll
    for (int i = 0; i < 6; ++i) x += d.G[6 * k + i] * de[i];
    da[k] = x;
    sc[(21 + k) * st] = x;
  }
  if (update) {
    double* ah = g.jump(pt, h);
#pragma unroll
    for (int k = 0; k < 3; ++k) ah[k * st] += da[k];
  }
  split(g, h, da, de, dl, dr);
}

// phase of a leaf, known where it is reached: 0 at even leaves, 1 at odd ones
template <int P>
using PhaseOf = std::integral_constant<int, P>;

// the register levels of a lane: the subtree of LV levels below its node n of
// the level R - LV. The halves of a subtree run through the same code, one
// after the other: unrolled, four copies of the leaf law and their live values
// took 560 registers a lane.
template <int LV, class G>
struct RegTree {
  static constexpr int LEVEL = G::R - LV;
  using Half = RegTree<LV - 1, G>;
  static __device__ __forceinline__ Slot node(int n, int lane) { return Slot{(1 << LEVEL) + n, lane}; }
  // strains from the jumps, leaves by leaf(phase, slot, eps, LeafV&), combination upwards
  template <bool PLAIN, class LeafFn>
  static __device__ __forceinline__ void up(const G& g, int pt, int n, int lane, const double* e, NodeV& out,
                                            double& gg, LeafFn& leaf) {
    double el[6], er[6];
    split_jump(g, pt, node(n, lane), e, el, er);
    if constexpr (LV == 1) {
      LeafV A, B;
      leaf(PhaseOf<0>{}, Slot{2 * n, lane}, el, A);
      leaf(PhaseOf<1>{}, Slot{2 * n + 1, lane}, er, B);
      combine<PLAIN>(g, pt, node(n, lane), A, B, out, gg);
    } else {
      NodeV B;
#pragma unroll 1
      for (int k = 0; k < 2; ++k) {
        if (k == 1) {
#pragma unroll
          for (int c = 0; c < 6; ++c) {
            el[c] = er[c];
            out.s[c] = B.s[c];
            out.sp[c] = B.sp[c];
          }
        }
        B.K = out.K + k * 21 * ON_LANES;  // the second half's tangent in the next slot
        Half::template up<PLAIN>(g, pt, 2 * n + k, lane, el, B, gg, leaf);
      }
      combine<PLAIN>(g, pt, node(n, lane), out, B, out, gg);
    }
  }
  // leaf strains from the jumps: fn(phase, slot, eps)
  template <class Fn>
  static __device__ __forceinline__ void down(const G& g, int pt, int n, int lane, const double* e, Fn& fn) {
    double el[6], er[6];
    split_jump(g, pt, node(n, lane), e, el, er);
    if constexpr (LV == 1) {
      fn(PhaseOf<0>{}, Slot{2 * n, lane}, el);
      fn(PhaseOf<1>{}, Slot{2 * n + 1, lane}, er);
    } else {
#pragma unroll 1
      for (int k = 0; k < 2; ++k) {
        if (k == 1)
#pragma unroll
          for (int c = 0; c < 6; ++c) el[c] = er[c];
        Half::down(g, pt, 2 * n + k, lane, el, fn);
      }
    }
  }
  // Newton steps from the node's strain change; leaf strain changes: fn(slot, deps)
  template <class Fn>
  static __device__ __forceinline__ void expand(const G& g, int pt, int n, int lane, const StepData* d,
                                                const double* de, bool update, Fn& fn) {
    double dl[6], dr[6];
    node_step(g, pt, node(n, lane), d[(1 << LEVEL) + n - 1], de, update, dl, dr);
    if constexpr (LV == 1) {
      fn(Slot{2 * n, lane}, dl);
      fn(Slot{2 * n + 1, lane}, dr);
    } else {
      Half::expand(g, pt, 2 * n, lane, d, dl, update, fn);
      Half::expand(g, pt, 2 * n + 1, lane, d, dr, update, fn);
    }
  }
};

__device__ __forceinline__ double shdown(double v, int d) { return __shfl_down(v, d, ON_LANES); }
__device__ __forceinline__ double shup(double v, int d) { return __shfl_up(v, d, ON_LANES); }

// sum over the wave, the same value on every lane
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = ON_LANES / 2; off >= 1; off >>= 1) v += __shfl_xor(v, off, ON_LANES);
  return __shfl(v, 0, ON_LANES);
}

// root strain (E, or 0 for a change) to the lane's depth-S node: shuffle levels,
// each owner splits its node with `jump(h, jn)`
template <class G, class JumpFn>
__device__ __forceinline__ void shuffle_down(const G& g, int lane, double* e, JumpFn& jump) {
  const int S = g.levels();
  const bool act = lane < (1 << S);
  for (int d = 0; d < S; ++d) {
    const int sh = S - d, half = 1 << (sh - 1);
    const int pos = lane & ((1 << sh) - 1);
    double er[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (act && pos == 0) jump(Top{(1 << d) + (lane >> sh)}, e, er);
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      const double t = shup(er[c], half);
      if (act && pos == half) e[c] = t;
    }
  }
}

// the lane's depth-S node value up to the root (lane 0), combining at every
// shuffle level: stress sums by shuffles, tangents read from the right
// child's LDS slot
template <bool PLAIN, class G>
__device__ __forceinline__ void shuffle_up(const G& g, int pt, int lane, NodeV& cur, double& gg) {
  const int S = g.levels();
  const bool act = lane < (1 << S);
  for (int d = S - 1; d >= 0; --d) {
    const int sh = S - d, half = 1 << (sh - 1);
    __syncthreads();  // the children's tangents are in their lanes' slots
    NodeV rb;
    rb.K = cur.K + half;
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      rb.s[c] = PLAIN ? shdown(cur.s[c], half) : 0.0;
      rb.sp[c] = shdown(cur.sp[c], half);
    }
    if (act && (lane & ((1 << sh) - 1)) == 0) combine<PLAIN>(g, pt, Top{(1 << d) + (lane >> sh)}, cur, rb, cur, gg);
  }
}

// Strains of every leaf at the current jumps (leaves by `leaf`), residual
// and elimination of the whole tree; root values on lane 0. root.K names the
// lane's first LDS slot.
template <bool PLAIN, class G, class LeafFn>
__device__ __forceinline__ void eval_pass(const G& g, int pt, int lane, LeafFn& leaf, NodeV& root, double& gg) {
  __syncthreads();  // the slots of the previous sweep have been read
  double e[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) e[c] = lane == 0 ? g.E[6 * pt + c] : 0.0;
  auto jump = [&](Top h, double* ev, double* er) {
    double el[6];
    split_jump(g, pt, h, ev, el, er);
#pragma unroll
    for (int c = 0; c < 6; ++c) ev[c] = el[c];
  };
  shuffle_down(g, lane, e, jump);
  if constexpr (G::R == 0) {
    LeafV L{};
    if (lane < g.leaves()) {
      if (lane & 1)
        leaf(PhaseOf<1>{}, Slot{0, lane}, e, L);
      else
        leaf(PhaseOf<0>{}, Slot{0, lane}, e, L);
    }
    to_node(L, root);
  } else {
    RegTree<G::R, G>::template up<PLAIN>(g, pt, 0, lane, e, root, gg, leaf);
  }
  shuffle_up<PLAIN>(g, pt, lane, root, gg);
}

// leaf strains at the current jumps: fn(phase, slot, eps)
template <class G, class Fn>
__device__ __forceinline__ void strains_pass(const G& g, int pt, int lane, Fn& fn) {
  double e[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) e[c] = lane == 0 ? g.E[6 * pt + c] : 0.0;
  auto jump = [&](Top h, double* ev, double* er) {
    double el[6];
    split_jump(g, pt, h, ev, el, er);
#pragma unroll
    for (int c = 0; c < 6; ++c) ev[c] = el[c];
  };
  shuffle_down(g, lane, e, jump);
  if constexpr (G::R == 0) {
    if (lane < g.leaves()) {
      if (lane & 1)
        fn(PhaseOf<1>{}, Slot{0, lane}, e);
      else
        fn(PhaseOf<0>{}, Slot{0, lane}, e);
    }
  } else {
    RegTree<G::R, G>::down(g, pt, 0, lane, e, fn);
  }
}

// Newton steps of all jumps for a zero root strain change (after eval_pass);
// the leaf strain changes: fn(slot, deps)
template <class G, class Fn>
__device__ __forceinline__ void expand_pass(const G& g, int pt, int lane, bool update, Fn& fn) {
  double de[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  // the lane's own nodes from memory, on their way during the levels above
  StepData own[1 << G::R];
#pragma unroll
  for (int n = 1; n < (1 << G::R); ++n) load_step(g, pt, Slot{n, lane}, own[n - 1]);
  auto step = [&](Top h, double* dv, double* dr) {
    double dl[6];
    StepData d;
    load_step(g, pt, h, d);
    node_step(g, pt, h, d, dv, update, dl, dr);
#pragma unroll
    for (int c = 0; c < 6; ++c) dv[c] = dl[c];
  };
  shuffle_down(g, lane, de, step);
  if constexpr (G::R == 0) {
    if (lane < g.leaves()) fn(Slot{0, lane}, de);
  } else {
    RegTree<G::R, G>::expand(g, pt, 0, lane, own, de, update, fn);
  }
}

// every internal node the lane owns: fn(slot)
template <class G, class Fn>
__device__ __forceinline__ void for_owned(const G& g, int lane, Fn& fn) {
  const int S = g.levels();
  if (lane >= (1 << S)) return;
  for (int d = 0; d < S; ++d) {
    const int sh = S - d;
    if ((lane & ((1 << sh) - 1)) == 0) fn(Top{(1 << d) + (lane >> sh)});
  }
#pragma unroll
  for (int n = 1; n < (1 << G::R); ++n) fn(Slot{n, lane});
}

// effective stress and the full 6 x 6 tangent of the root
__device__ __forceinline__ void put_root(double* o, const NodeV& root) {
#pragma unroll
  for (int c = 0; c < 6; ++c) o[c] = root.s[c];
#pragma unroll
  for (int i = 0; i < 6; ++i)
#pragma unroll
    for (int j = 0; j < 6; ++j) o[8 + 6 * i + j] = root.K[sx(i, j) * ON_LANES];
}

// |A^T W sigma| / ((2^K - 1) |sigma_bar|) from the lanes' sums and the root on lane 0
__device__ __forceinline__ double residual_norm(const OnArgs& g, int lane, const NodeV& root, double gg) {
  gg = wave_sum(gg);
  double sb = 0.0;
#pragma unroll
  for (int c = 0; c < 6; ++c) sb += root.s[c] * root.s[c];
  const double r = sqrt(gg) / ((double)(g.nleaf - 1) * fmax(sqrt(sb), 1e-300));
  return __shfl(r, 0, ON_LANES);
}

// State of step n, history sums and last plastic increment of a lane's PA66
// leaves, in registers for all sweeps of the call.
template <int N>
struct PaLeaves {
  double st[N][7], hs[N][7], dp[N];
};

// leaf law: stress and compressed tangent 3K P1 + ca P2 + cb N N
template <int PA, int PHASE, int N>
__device__ __forceinline__ void leaf_eval(const ProbInc& in, PaLeaves<N>& pl, Slot l, const double* e, double* sg,
                                          double& K3, double& ca, double& cb, double* nd) {
  const PhaseInc& pi = in.ph[PHASE];
  if constexpr (PHASE == PA) {
    const bool second = N > 1 && l.grp >> 1;
    double st[7], hs[7], dp = second ? pl.dp[N - 1] : pl.dp[0];
#pragma unroll
    for (int c = 0; c < 7; ++c) {
      st[c] = second ? pl.st[N - 1][c] : pl.st[0][c];
      hs[c] = second ? pl.hs[N - 1][c] : pl.hs[0][c];
    }
    PaOut o;
    pa66_point(in, e, st, 1, nullptr, nullptr, o, nullptr, nullptr, hs, &dp);
    if (second)
      pl.dp[N - 1] = dp;
    else
      pl.dp[0] = dp;
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      sg[c] = o.sig[c];
      nd[c] = o.nd[c];
    }
    K3 = pi.K3;
    ca = o.a;
    cb = o.b;
  } else {
    const double tr3 = (e[0] + e[1] + e[2]) * (1.0 / 3.0);
    const double sph = pi.K3 * (tr3 - pi.alpha_dth) - pi.G2 * tr3;
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      sg[c] = pi.G2 * e[c] + (c < 3 ? sph : 0.0);
      nd[c] = 0.0;
    }
    K3 = pi.K3;
    ca = pi.G2;
    cb = 0.0;
  }
}

// point partials of leaf l at its converged strain e, from state n:
// d sigma / d theta, d D / d eps, d D / d theta (closed form for the
// thermoelastic phase, central differences of the PA66 update)
template <int PA, int PHASE, class G>
__device__ __forceinline__ void leaf_partials(const G& g, const ProbInc& in, int pt, Slot l, const double* e,
                                              double* st_, double* gd, double& hd) {
  const double* enp = g.at(g.epsn, 6, pt, l);
  double en[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) en[c] = enp[c * g.stride()];
  if constexpr (PHASE == PA) {
    const long long ss = g.leaves() >> 1;
    const unsigned q = g.phase_index(l);
    const double* st = g.state + (long long)pt * g.nstate * ss + q;
    const double* hs = g.hist + (long long)pt * HIST_SLOTS * ss + q;
    double sp[6], Dp = 0.0;
    for (int k = 0; k < 14; ++k) {
      const bool th = k < 2;
      const ProbInc& ik = th ? g.inc_pm[2 * g.inc_ix[pt] + k] : in;
      double ek[6];
#pragma unroll
      for (int c = 0; c < 6; ++c) ek[c] = e[c];
      const int dir = (k - 2) >> 1;
      if (!th) ek[dir] += (k & 1) ? -FD_H_EPS : FD_H_EPS;
      PaOut po;
      double dis, cpl;
      pa66_point(ik, ek, st, ss, nullptr, en, po, &dis, &cpl, th ? nullptr : hs, nullptr);
      if (!(k & 1)) {
#pragma unroll
        for (int c = 0; c < 6; ++c) sp[c] = po.sig[c];
        Dp = cpl;
      } else if (th) {
#pragma unroll
        for (int c = 0; c < 6; ++c) st_[c] = (sp[c] - po.sig[c]) * (0.5 / FD_H_THETA);
        hd = (Dp - cpl) * (0.5 / FD_H_THETA);
      } else {
        gd[dir] = (Dp - cpl) * (0.5 / FD_H_EPS);
      }
    }
  } else {
    const PhaseInc& pi = in.ph[PHASE];
    const double ca = pi.K3 * pi.alpha0;
    const double trd = (e[0] - en[0]) + (e[1] - en[1]) + (e[2] - en[2]);
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      st_[c] = c < 3 ? -ca : 0.0;
      gd[c] = c < 3 ? -in.theta * ca / in.dt : 0.0;
    }
    hd = -ca * trd / in.dt;
  }
}

// R register levels, PA the phase with the PA66 law (-1: none), T: all four tangents
template <int R, int PA, bool T>
__global__ void __launch_bounds__(ON_LANES, ON_WAVES) k_dmn_online(OnView<R> g) {
  // condensed tangents: one slot per register level (at least one), lane-interleaved
  __shared__ double kslot[(R > 0 ? R : 1) * 21 * ON_LANES];
  __shared__ double top[TOP_FIELDS * ON_LANES];
  g.top = top;
  const int pt = blockIdx.x;
  const int lane = threadIdx.x;
  const int st = g.stride();
  if (lane >= 1 && lane < g.leaves()) {  // node `lane` of those above depth S
    const double* nt = g.table(Slot{0, lane});
    const double* ah = g.jump(pt, Slot{0, lane});
#pragma unroll
    for (int f = 0; f < ON_NODE; ++f) top[(TOP_TABLE + f) * ON_LANES + lane] = nt[f * st];
#pragma unroll
    for (int k = 0; k < 3; ++k) top[(TOP_JUMP + k) * ON_LANES + lane] = ah[k * st];
  }
  __syncthreads();
  constexpr int LPT = 1 << R;  // leaves per lane
  const int ix = g.inc_ix[pt];
  const ProbInc& in = g.inc[ix];
  const bool leaves = lane * LPT < g.leaves();
  // branch history sums of this lane's PA66 leaves for this increment
  constexpr int NPA = R > 0 ? LPT / 2 : 1;
  PaLeaves<NPA> pl;
  if (PA >= 0 && leaves && (R > 0 || (lane & 1) == PA)) {
    const long long ss = g.leaves() >> 1;
#pragma unroll
    for (int i = 0; i < NPA; ++i) {
      const unsigned q = g.phase_index(Slot{2 * i, lane});
      const double* state = g.state + (long long)pt * g.nstate * ss + q;
      pa66_history(in, state, ss, pl.hs[i], pl.hs[i][6]);
      double* h = g.hist + (long long)pt * HIST_SLOTS * ss + q;
#pragma unroll
      for (int c = 0; c < 7; ++c) {
        pl.st[i][c] = state[c * ss];
        h[c * ss] = pl.hs[i][c];
      }
      pl.dp[i] = -1.0;
    }
  }
  // predictor: start from the committed jumps plus s times their last change,
  // s = projection of this macro increment on the last committed one
  double pred_s = 0.0;
  if (g.pred) {
    const double* ep = g.Ep + 12 * pt;
    double ee = 0.0, pp = 0.0;
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      ee += (g.E[6 * pt + c] - ep[c]) * ep[6 + c];
      pp += ep[6 + c] * ep[6 + c];
    }
    if (g.committed[pt] && pp > 0.0 && isfinite(ee)) pred_s = fmin(2.0, fmax(0.0, ee / pp));
    auto start = [&](auto h) {
      double* ah = g.jump(pt, h);
      const int sh = g.stride(h);
      double* a0 = g.at(g.a0, 3, pt, g.slot(h));
      const double* dh = g.at(g.dah, 3, pt, g.slot(h));
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        a0[k * st] = ah[k * sh];
        ah[k * sh] += pred_s * dh[k * st];
      }
    };
    for_owned(g, lane, start);
  }
  auto law = [&](auto ph, Slot l, const double* e, LeafV& L) {
    double sg[6];
    leaf_eval<PA, decltype(ph)::value>(in, pl, l, e, sg, L.K3, L.ca, L.cb, L.nd);
    L.w = g.leaf_weight(l);
#pragma unroll
    for (int c = 0; c < 6; ++c) L.s[c] = L.w * sg[c];
  };
  NodeV root;
  root.K = kslot + lane;
  auto nothing = [](Slot, const double*) {};
  // sweeps: the start's, then after a Newton step (it counts them) and after
  // each cut back of a step that did not lower the residual (1, gamma, gamma^2, ..)
  int it = 0, cuts = 0;
  double res, res_old = 0.0;
  for (;;) {
    double gg = 0.0;
    eval_pass<true>(g, pt, lane, law, root, gg);
    res = residual_norm(g, lane, root, gg);
    if (it > 0) {
      if (!(res < res_old) && cuts < g.maxbt) {
        const double cut = pow(g.gamma, (double)cuts) * (1.0 - g.gamma);
        auto back = [&](auto h) {
          double* ah = g.jump(pt, h);
          const double* sc = g.scratch(pt, h);
          const int sh = g.stride(h);
#pragma unroll
          for (int k = 0; k < 3; ++k) ah[k * sh] -= cut * sc[(21 + k) * sh];
        };
        for_owned(g, lane, back);
        ++cuts;
        continue;
      }
      if (res < g.tol) break;
    }
    if (++it > g.maxit) break;
    expand_pass(g, pt, lane, true, nothing);
    res_old = res;
    cuts = 0;
  }
  const bool conv = res < g.tol;
  const bool commit = conv && !g.trial;
  if (it > g.maxit) it = g.maxit;
  // effective stress and tangent: the root of the last sweep
  double* o = g.out + (long long)pt * ON_OUT;
  if (lane == 0) put_root(o, root);
  if constexpr (T) {
    auto partials = [&](auto ph, Slot l, const double* e) {
      double st_[6], gd[6], hd;
      leaf_partials<PA, decltype(ph)::value>(g, in, pt, l, e, st_, gd, hd);
      double* lp = g.at(g.lp, ON_LP, pt, l);
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        lp[c * st] = st_[c];
        lp[(6 + c) * st] = gd[c];
      }
      lp[12 * st] = hd;
    };
    strains_pass(g, pt, lane, partials);
    // k = 0, d<sigma>/dtheta: the jumps equilibrate the leaf sources w dsigma/dtheta;
    // k = 1, d<D>/dE = sum_l w_l (d eps_l / dE)^T dD/deps_l: the condensed value of
    // the leaf sources w dD/deps (the localization is symmetric in this sense)
#pragma unroll 1
    for (int k = 0; k < 2; ++k) {
      auto source = [&](auto ph, Slot l, const double* e, LeafV& L) {
        const double* lp = g.at(g.lp, ON_LP, pt, l) + 6 * k * st;
        double sg[6];
        leaf_eval<PA, decltype(ph)::value>(in, pl, l, e, sg, L.K3, L.ca, L.cb, L.nd);
        L.w = g.leaf_weight(l);
#pragma unroll
        for (int c = 0; c < 6; ++c) L.s[c] = L.w * lp[c * st];
      };
      NodeV rt;
      rt.K = kslot + lane;
      double unused = 0.0;
      eval_pass<false>(g, pt, lane, source, rt, unused);
      if (lane == 0)
#pragma unroll
        for (int c = 0; c < 6; ++c) o[(k == 0 ? O_DSDT : O_DDDE) + c] = rt.sp[c];
      if (k == 1) break;
      // d<D>/dtheta = sum_l w_l (dD/dtheta_l + dD/deps_l . d eps_l / d theta)
      double dT = 0.0;
      auto heat = [&](Slot l, const double* de) {
        const double* lp = g.at(g.lp, ON_LP, pt, l);
        double x = lp[12 * st];
#pragma unroll
        for (int c = 0; c < 6; ++c) x += lp[(6 + c) * st] * de[c];
        dT += g.leaf_weight(l) * x;
      };
      expand_pass(g, pt, lane, false, heat);
      dT = wave_sum(dT);
      if (lane == 0) o[O_DDDT] = dT;
    }
  }
  __syncthreads();  // the jumps above depth S go back: the next call starts from them
  if (lane >= 1 && lane < g.leaves()) {
    double* ah = g.jump(pt, Slot{0, lane});
#pragma unroll
    for (int k = 0; k < 3; ++k) ah[k * st] = top[(TOP_JUMP + k) * ON_LANES + lane];
  }
  // coupling term and dissipation of every leaf; commit if converged
  double D = 0.0, Dd = 0.0;
  auto fin = [&](auto ph, Slot l, const double* e) {
    constexpr int PHASE = decltype(ph)::value;
    double* enp = g.at(g.epsn, 6, pt, l);
    double en[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) en[c] = enp[c * st];
    double Dl = 0.0, Ddl = 0.0;
    if constexpr (PHASE == PA) {
      const long long ss = g.leaves() >> 1;
      const unsigned q = g.phase_index(l);
      double* state = g.state + (long long)pt * g.nstate * ss + q;
      double* hs = g.hist + (long long)pt * HIST_SLOTS * ss + q;
      PaOut po;
      pa66_point(in, e, state, ss, commit ? state : nullptr, en, po, &Ddl, &Dl, hs, nullptr);
    } else {
      const PhaseInc& pi = in.ph[PHASE];
      const double trd = (e[0] - en[0]) + (e[1] - en[1]) + (e[2] - en[2]);
      Dl = -in.theta * pi.K3 * pi.alpha0 * trd / in.dt;
    }
    const double w = g.leaf_weight(l);
    D += w * Dl;
    Dd += w * Ddl;
    if (commit)
#pragma unroll
      for (int c = 0; c < 6; ++c) enp[c * st] = e[c];
  };
  strains_pass(g, pt, lane, fin);
  if (g.pred) {
    if (commit) {
      auto change = [&](auto h) {
        const double* ah = g.jump(pt, h);
        const int sh = g.stride(h);
        const double* a0 = g.at(g.a0, 3, pt, g.slot(h));
        double* dh = g.at(g.dah, 3, pt, g.slot(h));
#pragma unroll
        for (int k = 0; k < 3; ++k) dh[k * st] = ah[k * sh] - a0[k * st];
      };
      for_owned(g, lane, change);
    }
    if (lane == 0) g.committed[pt] = commit ? 1 : 0;
  }
  // the committed macro strain and its last change are kept with the
  // predictor off too, so that switching it on measures the next increment
  // from the right base
  if (lane == 0 && commit) {
    double* ep = g.Ep + 12 * pt;
    for (int c = 0; c < 6; ++c) {
      ep[6 + c] = g.E[6 * pt + c] - ep[c];
      ep[c] = g.E[6 * pt + c];
    }
  }
  D = wave_sum(D);
  Dd = wave_sum(Dd);
  if (lane == 0) {
    o[6] = D;
    o[7] = Dd;
    o[O_RES] = res;
    o[O_IT] = it;
    o[O_ST] = conv ? 1.0 : 0.0;
  }
}

}  // namespace

namespace {
template <int R, int PA>
void launch_online_tangents(const OnArgs& g, hipStream_t s, int n) {
  OnView<R> v;
  static_cast<OnArgs&>(v) = g;
  v.top = nullptr;
  if (g.what)
    hipLaunchKernelGGL((k_dmn_online<R, PA, true>), dim3(n), dim3(ON_LANES), 0, s, v);
  else
    hipLaunchKernelGGL((k_dmn_online<R, PA, false>), dim3(n), dim3(ON_LANES), 0, s, v);
}
template <int R>
void launch_online_phase(const OnArgs& g, hipStream_t s, int n) {
  if (g.pa_phase == 0)
    launch_online_tangents<R, 0>(g, s, n);
  else if (g.pa_phase == 1)
    launch_online_tangents<R, 1>(g, s, n);
  else
    launch_online_tangents<R, -1>(g, s, n);
}
void launch_online_levels(const OnArgs& g, hipStream_t s, int n) {
  static_assert(ON_MAX_K - ON_SHUF <= 2, "at most two register levels per lane");
  switch (g.K - g.S) {  // register levels below the shuffle levels
    case 0:
      return launch_online_phase<0>(g, s, n);
    case 1:
      return launch_online_phase<1>(g, s, n);
    default:
      return launch_online_phase<2>(g, s, n);
  }
}
}  // namespace

struct PairHash {
  size_t operator()(const std::pair<uint64_t, uint64_t>& k) const {
    return std::hash<uint64_t>()(k.first * 0x9E3779B97F4A7C15ull ^ k.second);
  }
};

struct DmnOnline {
  int K, nleaf, npoints, nstate = 0, pa_phase = -1;
  double tol;
  int maxit;
  std::vector<hom_law> laws;
  std::vector<void*> allocs;
  double *p = nullptr, *node = nullptr, *state = nullptr, *hist = nullptr, *epsn = nullptr, *a = nullptr;
  double *scr = nullptr, *lp = nullptr, *E = nullptr, *out = nullptr;
  double *dah = nullptr, *a0 = nullptr, *Ep = nullptr;
  int* committed = nullptr;
  int pred = 0;
  ProbInc *inc = nullptr, *inc_pm = nullptr;
  int* inc_ix = nullptr;
  std::vector<ProbInc> inc_h, inc_pm_h;
  // pinned staging of the per-point inputs and outputs
  double *E_h = nullptr, *out_h = nullptr;
  int* ix_h = nullptr;
  ~DmnOnline() {
    for (void* ptr : allocs) (void)hipFree(ptr);
    for (void* ptr : {(void*)E_h, (void*)out_h, (void*)ix_h})
      if (ptr) (void)hipHostFree(ptr);
  }
};

DmnOnline* dmn_online_create(const Dmn& net, const hom_law* laws, int npoints, double tol, int maxit) {
  if (net.K > ON_MAX_K) fail(HOM_E_UNSUPPORTED, "online evaluation supports depths up to 8");
  if (npoints < 1) fail(HOM_E_ARG, "need at least one point");
  if (!(tol > 0.0) || maxit < 1) fail(HOM_E_ARG, "need tol > 0 and maxit >= 1");
  if (!laws) fail(HOM_E_ARG, "null laws");
  validate_laws(laws, 2);
  auto o = std::make_unique<DmnOnline>();
  o->K = net.K;
  o->nleaf = net.nleaf;
  o->npoints = npoints;
  o->tol = tol;
  o->maxit = maxit;
  o->laws.assign(laws, laws + 2);
  for (int i = 0; i < 2; ++i)
    if (laws[i].kind == HOM_LAW_PA66) {
      o->pa_phase = i;
      int nm = 0;
      for (int j = 0; j < laws[i].n_maxwell; ++j) nm += laws[i].E_i[j] > 0.0 ? 1 : 0;
      o->nstate = 7 + 6 * nm;
    }
  const size_t half = (size_t)o->nleaf / 2;
  o->p = dalloc_into<double>(o->allocs, net.nparam);
  hip_check(hipMemcpy(o->p, net.p, net.nparam * sizeof(double), hipMemcpyDeviceToDevice), "hipMemcpy");
  o->node = dalloc_into<double>(o->allocs, (size_t)o->nleaf * (ON_NODE + 1));
  hipLaunchKernelGGL(k_dmn_node_table, dim3(1), dim3(1), 0, nullptr, o->p, o->nleaf, std::min(o->K, ON_SHUF),
                     o->node);
  hip_check(hipGetLastError(), "k_dmn_node_table");
  if (o->nstate) {
    o->state = dalloc_into<double>(o->allocs, (size_t)npoints * o->nstate * half);
    o->hist = dalloc_into<double>(o->allocs, (size_t)npoints * HIST_SLOTS * half);
  }
  o->epsn = dalloc_into<double>(o->allocs, (size_t)npoints * o->nleaf * 6);
  o->a = dalloc_into<double>(o->allocs, (size_t)npoints * o->nleaf * 3);
  o->scr = dalloc_into<double>(o->allocs, (size_t)npoints * o->nleaf * ON_SCR);
  o->lp = dalloc_into<double>(o->allocs, (size_t)npoints * o->nleaf * ON_LP);
  o->dah = dalloc_into<double>(o->allocs, (size_t)npoints * o->nleaf * 3);
  o->a0 = dalloc_into<double>(o->allocs, (size_t)npoints * o->nleaf * 3);
  o->Ep = dalloc_into<double>(o->allocs, (size_t)npoints * 12);
  o->committed = dalloc_into<int>(o->allocs, npoints);
  o->E = dalloc_into<double>(o->allocs, (size_t)npoints * 6);
  o->out = dalloc_into<double>(o->allocs, (size_t)npoints * ON_OUT);
  o->inc = dalloc_into<ProbInc>(o->allocs, npoints);
  o->inc_pm = dalloc_into<ProbInc>(o->allocs, 2 * (size_t)npoints);
  o->inc_ix = dalloc_into<int>(o->allocs, npoints);
  o->inc_h.reserve(npoints);
  o->inc_pm_h.reserve(2 * (size_t)npoints);
  hip_check(hipHostMalloc((void**)&o->E_h, (size_t)npoints * 6 * sizeof(double)), "hipHostMalloc");
  hip_check(hipHostMalloc((void**)&o->out_h, (size_t)npoints * ON_OUT * sizeof(double)), "hipHostMalloc");
  hip_check(hipHostMalloc((void**)&o->ix_h, (size_t)npoints * sizeof(int)), "hipHostMalloc");
  return o.release();
}

void dmn_online_destroy(DmnOnline* o) { delete o; }

void dmn_online_set_predictor(DmnOnline* o, int on) {
  if (on != 0 && on != 1) fail(HOM_E_ARG, "predictor must be 0 or 1");
  // jump changes are recorded only while the predictor is on: switching it
  // on forgets what an earlier on-period left, so the first call starts from
  // the current jumps
  if (on && !o->pred)
    hip_check(hipMemset(o->committed, 0, (size_t)o->npoints * sizeof(int)), "hipMemset");
  o->pred = on;
}

void dmn_online_step(DmnOnline* o, const double* strain, const double* theta, const double* dt, int what,
                     int trial, hom_dmn_result* res) {
  if (what != 0 && what != 1) fail(HOM_E_ARG, "what must be 0 (d sigma / dE) or 1 (all four tangents)");
  if (trial != 0 && trial != 1) fail(HOM_E_ARG, "trial must be 0 or 1");
  const int n = o->npoints;
  const double sq2 = std::sqrt(2.0);
  const double w[6] = {1, 1, 1, sq2, sq2, sq2};
  // one increment record per distinct (theta, dt): points of one macroscopic
  // step usually share both
  o->inc_h.clear();
  o->inc_pm_h.clear();
  std::unordered_map<std::pair<uint64_t, uint64_t>, int, PairHash> seen;
  double last_t = NAN, last_d = NAN;
  int last_ix = -1;
  for (int i = 0; i < n; ++i) {
    if (!(dt[i] > 0.0) || !std::isfinite(dt[i])) fail(HOM_E_ARG, "dt must be positive and finite");
    if (!(theta[i] > 0.0) || !std::isfinite(theta[i])) fail(HOM_E_ARG, "theta must be positive");
    for (int c = 0; c < 6; ++c) {
      if (!std::isfinite(strain[6 * i + c])) fail(HOM_E_ARG, "macro strain must be finite");
      o->E_h[6 * i + c] = w[c] * strain[6 * i + c];
    }
    if (theta[i] != last_t || dt[i] != last_d) {
      uint64_t kt, kd;
      std::memcpy(&kt, &theta[i], 8);
      std::memcpy(&kd, &dt[i], 8);
      auto it = seen.find({kt, kd});
      if (it != seen.end()) {
        last_ix = it->second;
      } else {
        last_ix = (int)o->inc_h.size();
        seen.emplace(std::make_pair(kt, kd), last_ix);
        o->inc_h.emplace_back();
        fill_inc(o->inc_h.back(), o->laws, theta[i], dt[i]);
        if (what) {
          o->inc_pm_h.emplace_back();
          fill_inc(o->inc_pm_h.back(), o->laws, theta[i] + FD_H_THETA, dt[i]);
          o->inc_pm_h.emplace_back();
          fill_inc(o->inc_pm_h.back(), o->laws, theta[i] - FD_H_THETA, dt[i]);
        }
      }
      last_t = theta[i];
      last_d = dt[i];
    }
    o->ix_h[i] = last_ix;
  }
  const size_t nu = o->inc_h.size();
  if (what)
    hip_check(hipMemcpy(o->inc_pm, o->inc_pm_h.data(), 2 * nu * sizeof(ProbInc), hipMemcpyHostToDevice),
              "hipMemcpy");
  hip_check(hipMemcpy(o->inc, o->inc_h.data(), nu * sizeof(ProbInc), hipMemcpyHostToDevice), "hipMemcpy");
  hip_check(hipMemcpy(o->inc_ix, o->ix_h, n * sizeof(int), hipMemcpyHostToDevice), "hipMemcpy");
  hip_check(hipMemcpy(o->E, o->E_h, 6 * n * sizeof(double), hipMemcpyHostToDevice), "hipMemcpy");
  OnArgs g{};
  g.K = o->K;
  g.nleaf = o->nleaf;
  g.S = std::min(o->K, ON_SHUF);
  g.node = o->node;
  g.inc = o->inc;
  g.inc_pm = o->inc_pm;
  g.inc_ix = o->inc_ix;
  g.what = what;
  g.trial = trial;
  g.pa_phase = o->pa_phase;
  g.state = o->state;
  g.nstate = o->nstate;
  g.hist = o->hist;
  g.epsn = o->epsn;
  g.a = o->a;
  g.scr = o->scr;
  g.lp = o->lp;
  g.pred = o->pred;
  g.dah = o->dah;
  g.a0 = o->a0;
  g.Ep = o->Ep;
  g.committed = o->committed;
  g.E = o->E;
  g.out = o->out;
  g.tol = o->tol;
  g.gamma = 0.5;
  g.maxit = o->maxit;
  g.maxbt = 8;
  launch_online_levels(g, nullptr, n);
  hip_check(hipGetLastError(), "k_dmn_online");
  hip_check(hipMemcpy(o->out_h, o->out, (size_t)ON_OUT * n * sizeof(double), hipMemcpyDeviceToHost), "hipMemcpy");
  for (int i = 0; i < n; ++i) {
    const double* r = o->out_h + (size_t)ON_OUT * i;
    hom_dmn_result& t = res[i];
    std::memset(&t, 0, sizeof(t));
    for (int c = 0; c < 6; ++c) t.stress[c] = r[c] / w[c];
    t.coupling = r[6];
    t.dissipation = r[7];
    for (int I = 0; I < 6; ++I)
      for (int J = 0; J < 6; ++J) t.dsde[6 * I + J] = r[8 + 6 * I + J] * w[J] / w[I];
    for (int c = 0; c < 6; ++c) {
      t.dsdt[c] = what ? r[O_DSDT + c] / w[c] : NAN;
      t.dDde[c] = what ? r[O_DDDE + c] * w[c] : NAN;
    }
    t.dDdt = what ? r[O_DDDT] : NAN;
    t.residual = r[O_RES];
    t.newton_iters = (int)r[O_IT];
    t.status = r[O_ST] == 1.0 ? HOM_OK : HOM_E_NOT_CONVERGED;
  }
}

}  // namespace hom
