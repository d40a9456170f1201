// Surrogate network: n_in (<= 32) -> 4 x 256 (GELU) -> n_out (<= 16).
//
// Forward: one work-group of 8 waves per 64 rows (each wave all 64 rows x
// 32 output columns); every layer is a [64 x K] x [K x 256] product on the
// bf16 matrix cores (v_mfma_f32_16x16x32_bf16, FP32 accumulation). Weights are bf16; the
// activations are kept in LDS split into bf16 hi + lo parts (two MFMAs per
// tile), so the product sees the activations to ~16 significant bits. In "precise" mode the
// weights are split as well (three MFMAs: a_hi w_hi + a_lo w_hi + a_hi w_lo),
// which reproduces FP32 weights for gradient checks. Bias and GELU are fused
// into the epilogue; the layer output stays in LDS for the next layer.
//
// Training: FP32 backward on the FP32 matrix cores, one launch a layer (dW = dZ^T A
// in splits of the batch, db, and dA = dZ W with gelu'), weighted MSE on normalized outputs,
// and one launch that sums the splits, applies Adam to the FP32 master weights and refreshes
// their bf16 copies: eight launches a step.
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>
#include <cstring>
#include <future>
#include <mutex>
#include <random>
#include <type_traits>
#include <vector>

#include "mlp.h"
#include "runtime.h"

// Per-network outputs of the allocation-free ensemble inference. One copy per
// GPU, at that GPU's own address: host code never passes this name to a
// kernel, only the address hipGetSymbolAddress returns for the current device.
static __device__ __align__(256) float scratch[HOM_STATIC_SCRATCH_FLOATS];

namespace hom {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));

constexpr int FWD_WAVES = 8;          // waves per forward work-group
// Work-groups of 16 rows (over all networks) up to which a forward launch takes
// them, so that more CUs have one; beyond, 64 rows each. The line lies where a
// CU would get one more round of small ones: three a CU fit beside each other
// (12288 rows 20.4 us with 16 rows and 22.9 with 64, 13312 rows 25.7 and 22.9;
// of eight networks 38.6 and 42.1, 43.8 and 42.8), in precise mode two (8192
// rows 20.2 and 27.1, 10240 rows 27.0 and 27.1, 12288 rows 28.6 and 27.2). Rows
// for another round of large ones make no second line: 20480 rows 31.9 and 36.2,
// but 24576 37.5 and 37.1. A row's result does not depend on the choice.
constexpr long long few_groups(bool precise) { return precise ? 640 : 768; }
constexpr int NCB = MLP_W / (16 * FWD_WAVES);  // 16-column tiles per wave
constexpr int AST = 264;              // LDS row stride of the bf16 activation tiles (16-byte aligned rows)

// erf by Abramowitz and Stegun's rational approximation 7.1.26 (Handbook of
// Mathematical Functions, 1964): erf(x) = 1 - t (a1 + t (a2 + ... + t a5))
// exp(-x^2), t = 1 / (1 + p x) for x >= 0, odd extension; absolute error
// below 1.5e-7 (2e-7 with the hardware reciprocal), about a third of the
// instructions of the library erf. The network's forward and backward passes
// both use it, so training sees one consistent activation function.
__device__ __forceinline__ float erf_as(float x) {
  const float ax = fabsf(x);
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, ax, 1.0f));  // v_rcp_f32, 1 ulp
  float p = fmaf(1.061405429f, t, -1.453152027f);
  p = fmaf(p, t, 1.421413741f);
  p = fmaf(p, t, -0.284496736f);
  p = fmaf(p, t, 0.254829592f);
  const float e = __expf(-ax * ax);
  return copysignf(fmaf(-p * t, e, 1.0f), x);
}
__device__ __forceinline__ float gelu_prime_f(float z) {
  return 0.5f * (1.0f + erf_as(z * 0.70710678118654752f)) + z * __expf(-0.5f * z * z) * 0.39894228040143268f;
}

// The same approximation arranged for the forward pass: with x = z / sqrt 2,
// Phi(z) = 1 - q / 2 for z >= 0 and q / 2 below, q = p(t) t exp(-x^2), so
// GELU(z) = z Phi(z) = max(z, 0) - |z| q / 2 (no cancellation for negative z);
// the 1 / sqrt 2 and the 1 / 2 are folded into the constants.
__device__ __forceinline__ float gelu_fwd(float z) {
  const float az = fabsf(z);
  const float t = __builtin_amdgcn_rcpf(fmaf(0.2316418883f, az, 1.0f));
  float p = fmaf(0.5307027145f, t, -0.7265760135f);
  p = fmaf(p, t, 0.7107068705f);
  p = fmaf(p, t, -0.142248368f);
  p = fmaf(p, t, 0.127414796f);
  const float e = __builtin_amdgcn_exp2f(z * z * -0.7213475204f);  // exp(-z^2 / 2)
  return fmaf(-az, p * t * e, fmaxf(z, 0.0f));
}

// bf16 weight copies in fragment order: the 16 x 32 block of output rows
// 16 cb .. 16 cb + 15 and inputs 32 s .. 32 s + 31 is one contiguous 1 KiB
// fragment, lane-major (lane = 16 (k / 8 mod 4) + output mod 16, then 8
// consecutive inputs), so a wave's B operand of one k-step is a single
// coalesced 1 KiB load. Offset of the lane's 8 values in a layer with inner
// dimension K:
__host__ __device__ __forceinline__ long long frag_offset(int cb, int s, int K, int lane) {
  return (((long long)cb * (K / 32) + s) * 64 + lane) * 8;
}

// One network of a forward launch (blockIdx.y): its parameter arrays, whose
// layer offsets are the same for every network.
struct NetRef {
  const __bf16* hi;
  const __bf16* lo;
  const float* w;     // FP32 parameters (the biases)
  const float* scal;  // xmean[32] xinv[32] ymean[16] ystd[16]
  const float* skip;  // G [16][MLP_GATES][32], c [16], then G's bf16 hi and lo parts
  int g0, g1, g2;     // gate input indices
};

struct FwdArgs {
  const float* x;
  const int* idx;  // row r of the launch is row idx[r] of x, or null (row r)
  long long n;
  int n_in, n_out;
  int woff[MLP_LAYERS], boff[MLP_LAYERS];
  NetRef net[HOM_ENSEMBLE_MAX_NETS];
  float* y;      // [networks][n][n_out] outputs in physical units (optional)
  float* yhat;   // [n][16] normalized outputs (optional)
  float* xs;     // [n][32] normalized inputs (optional, training)
  float* zs[MLP_LAYERS - 1];  // [n][256] pre-activations (optional)
  float* as[MLP_LAYERS - 1];  // [n][256] activations (optional)
};

// SAVE: keep the normalized inputs, pre-activations, activations and
// normalized outputs for the backward pass (training); inference writes y only
// MROWS: rows per work-group, 64 where that fills the chip (the weights are
// read once a work-group), 16 for fewer rows, whose launches are bound by the
// latency of a work-group's layers. A row's arithmetic is the same in both.
template <int PRECISE, bool SAVE, int MROWS>
__global__ void __launch_bounds__(FWD_WAVES * 64) __attribute__((amdgpu_waves_per_eu(4))) k_mlp_fwd(FwdArgs a) {
  constexpr int NRB = MROWS / 16;  // 16-row tiles per wave (every wave spans all rows)
  // The tile's activations live in LDS already split into bf16 hi + lo: each
  // value is split once, by the lane that produced it, and every wave reads
  // its MFMA fragments directly.
  __shared__ __attribute__((aligned(16))) __bf16 ahi[MROWS * AST];
  __shared__ __attribute__((aligned(16))) __bf16 alo[MROWS * AST];
  __shared__ float xin[MROWS * (MLP_IN + 1)];  // normalized inputs, kept for the skip
  const int tid = threadIdx.x;
  const int wave = tid >> 6;
  const int lane = tid & 63;
  const long long row0 = (long long)blockIdx.x * MROWS;
  const NetRef& net = a.net[blockIdx.y];
  const float *xmean = net.scal, *xinv = net.scal + MLP_IN;
  const float *ymean = net.scal + 2 * MLP_IN, *ystd = ymean + MLP_OUT;
  const __bf16* skip_hi = reinterpret_cast<const __bf16*>(net.skip + MLP_OUT * MLP_GATES * MLP_IN + MLP_OUT);
  const __bf16* skip_lo = skip_hi + MLP_OUT * MLP_GATES * MLP_IN;
  float* y = a.y ? a.y + (long long)blockIdx.y * a.n * a.n_out : nullptr;
  for (int i = tid; i < MROWS * MLP_IN; i += FWD_WAVES * 64) {
    const int r = i / MLP_IN, k = i % MLP_IN;
    const long long gr = row0 + r;
    float v = 0.0f;
    if (gr < a.n && k < a.n_in) v = (a.x[(a.idx ? a.idx[gr] : gr) * a.n_in + k] - xmean[k]) * xinv[k];
    const __bf16 h = (__bf16)v;
    ahi[r * AST + k] = h;
    alo[r * AST + k] = (__bf16)(v - (float)h);
    xin[r * (MLP_IN + 1) + k] = v;
    if (SAVE && gr < a.n) a.xs[gr * MLP_IN + k] = v;
  }
  __syncthreads();
  const int lrow = lane & 15;
  const int kq = (lane >> 4) * 8;
#pragma unroll 1
  for (int l = 0; l < MLP_LAYERS - 1; ++l) {
    const int K = l == 0 ? MLP_IN : MLP_W;
    const __bf16* whi = net.hi + a.woff[l];
    const __bf16* wlo = net.lo + a.woff[l];
    const float* bias = net.w + a.boff[l];
    // lane: row m = rb 16 + lrow, outputs nn0 .. nn0 + 3 of tile cb; the
    // bias enters as the first product's accumulator input
    floatx4_t bv[NCB];
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
      bv[cb] = *reinterpret_cast<const floatx4_t*>(bias + wave * (16 * NCB) + cb * 16 + (lane >> 4) * 4);
    floatx4_t acc[NRB][NCB];
    bf16x8_t bh[NCB], bl[NCB];
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      const long long f = frag_offset(wave * NCB + cb, 0, K, lane);
      bh[cb] = *reinterpret_cast<const bf16x8_t*>(whi + f);
      if constexpr (PRECISE) bl[cb] = *reinterpret_cast<const bf16x8_t*>(wlo + f);
    }
    const auto step = [&](int k0, auto first) {
      constexpr bool FIRST = decltype(first)::value;
      bf16x8_t xh[NRB], xl[NRB];
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb) {
        const int o = (rb * 16 + lrow) * AST + k0 + kq;
        xh[rb] = *reinterpret_cast<const bf16x8_t*>(ahi + o);
        xl[rb] = *reinterpret_cast<const bf16x8_t*>(alo + o);
      }
      // weights of the next k-step in flight during this step's products
      const int k1 = k0 + 32 < K ? k0 + 32 : k0;
      bf16x8_t nh[NCB], nl[NCB];
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        const long long f = frag_offset(wave * NCB + cb, k1 / 32, K, lane);
        nh[cb] = *reinterpret_cast<const bf16x8_t*>(whi + f);
        if constexpr (PRECISE) nl[cb] = *reinterpret_cast<const bf16x8_t*>(wlo + f);
      }
      // the transposed tile Z^T = W A^T (weights as the first operand): each
      // lane's four accumulator values are four consecutive outputs of one
      // row, stored as one 8-byte LDS write per part in the epilogue. hi and
      // lo passes over all of the wave's tiles: no product waits on the
      // previous one into the same accumulator
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
          if constexpr (FIRST)
            acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bh[cb], xh[rb], bv[cb], 0, 0, 0);
          else
            acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bh[cb], xh[rb], acc[rb][cb], 0, 0, 0);
        }
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
          acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bh[cb], xl[rb], acc[rb][cb], 0, 0, 0);
      if constexpr (PRECISE) {
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb)
            acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bl[cb], xh[rb], acc[rb][cb], 0, 0, 0);
      }
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        bh[cb] = nh[cb];
        if constexpr (PRECISE) bl[cb] = nl[cb];
      }
    };
    step(0, std::true_type{});
    for (int k0 = 32; k0 < K; k0 += 32) step(k0, std::false_type{});
    __syncthreads();  // all waves done reading this layer's input
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        const int m = rb * 16 + lrow;
        const int nn0 = wave * (16 * NCB) + cb * 16 + (lane >> 4) * 4;
        floatx4_t z, g;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          z[i] = acc[rb][cb][i];
          g[i] = gelu_fwd(z[i]);
        }
        unsigned hp[2], lp[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const bf16x2_t hh = {(__bf16)g[2 * j], (__bf16)g[2 * j + 1]};
          hp[j] = __builtin_bit_cast(unsigned, hh);
          const float h0 = __builtin_bit_cast(float, hp[j] << 16);
          const float h1 = __builtin_bit_cast(float, hp[j] & 0xffff0000u);
          const bf16x2_t ll = {(__bf16)(g[2 * j] - h0), (__bf16)(g[2 * j + 1] - h1)};
          lp[j] = __builtin_bit_cast(unsigned, ll);
        }
        *reinterpret_cast<uint2*>(ahi + m * AST + nn0) = make_uint2(hp[0], hp[1]);
        *reinterpret_cast<uint2*>(alo + m * AST + nn0) = make_uint2(lp[0], lp[1]);
        if constexpr (SAVE) {
          const long long gr = row0 + m;
          if (gr < a.n) {
            *reinterpret_cast<floatx4_t*>(a.zs[l] + gr * MLP_W + nn0) = z;
            *reinterpret_cast<floatx4_t*>(a.as[l] + gr * MLP_W + nn0) = g;
          }
        }
      }
    __syncthreads();
  }
  // output layer: each wave 16 rows x 16 outputs
  if (wave < MROWS / 16) {
    const int l = MLP_LAYERS - 1;
    const __bf16* whi = net.hi + a.woff[l];
    const __bf16* wlo = net.lo + a.woff[l];
    const float* bias = net.w + a.boff[l];
    floatx4_t acc = floatx4_t{0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < MLP_W; k0 += 32) {
      const int o = (wave * 16 + lrow) * AST + k0 + kq;
      const bf16x8_t xh = *reinterpret_cast<const bf16x8_t*>(ahi + o);
      const bf16x8_t xl = *reinterpret_cast<const bf16x8_t*>(alo + o);
      const bf16x8_t bh = *reinterpret_cast<const bf16x8_t*>(whi + frag_offset(0, k0 / 32, MLP_W, lane));
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xh, bh, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xl, bh, acc, 0, 0, 0);
      if constexpr (PRECISE) {
        const bf16x8_t bl = *reinterpret_cast<const bf16x8_t*>(wlo + frag_offset(0, k0 / 32, MLP_W, lane));
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xh, bl, acc, 0, 0, 0);
      }
    }
    // gated cubic skip, sk = c + sum_g s_g(x) (G_g . x), on the matrix cores:
    // for every gate polynomial s_g the 16 rows x 16 outputs of G_g . x in one
    // tile whose layout matches acc (x and G split into bf16 hi + lo parts,
    // three products: about 16 significant bits)
    floatx4_t sk = floatx4_t{0.f, 0.f, 0.f, 0.f};
    if (y) {  // uniform over the work-group
      bf16x8_t xh, xl;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float v = xin[(wave * 16 + lrow) * (MLP_IN + 1) + kq + j];
        xh[j] = (__bf16)v;
        xl[j] = (__bf16)(v - (float)xh[j]);
      }
      float sg[4][MLP_GATES];  // the gate polynomials of this lane's four rows
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float* xr = xin + (wave * 16 + (lane >> 4) * 4 + i) * (MLP_IN + 1);
        const float va = xr[net.g0], vb = xr[net.g1], vc = xr[net.g2];
        const float s[MLP_GATES] = {1.f, va, va * va, va * va * va, vb, vb * vb, vb * vb * vb,
                                    vc, vc * vc, vc * vc * vc};
#pragma unroll
        for (int gi = 0; gi < MLP_GATES; ++gi) sg[i][gi] = s[gi];
      }
      const size_t gb = (size_t)lrow * MLP_GATES * MLP_IN + kq;  // output lrow, inputs kq ..
#pragma unroll
      for (int gi = 0; gi < MLP_GATES; ++gi) {
        const bf16x8_t gh = *reinterpret_cast<const bf16x8_t*>(skip_hi + gb + gi * MLP_IN);
        const bf16x8_t gl = *reinterpret_cast<const bf16x8_t*>(skip_lo + gb + gi * MLP_IN);
        floatx4_t t = floatx4_t{0.f, 0.f, 0.f, 0.f};
        t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xh, gh, t, 0, 0, 0);
        t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xl, gh, t, 0, 0, 0);
        t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xh, gl, t, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) sk[i] += sg[i][gi] * t[i];
      }
      const float c = net.skip[MLP_OUT * MLP_GATES * MLP_IN + lrow];
#pragma unroll
      for (int i = 0; i < 4; ++i) sk[i] += c;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = wave * 16 + (lane >> 4) * 4 + i;
      const long long gr = row0 + m;
      if (gr >= a.n) continue;
      const float z = acc[i] + bias[lrow];
      if (SAVE) a.yhat[gr * MLP_OUT + lrow] = z;
      if (y && lrow < a.n_out) y[gr * a.n_out + lrow] = z * ystd[lrow] + ymean[lrow] + sk[i];
    }
  }
}

// ---------------------------------------------------------------------------
// backward of one layer: both products, the bias gradient and gelu' in one launch
// ---------------------------------------------------------------------------
// Work-groups of two kinds, 64 x 64 tiles each, on the FP32 matrix cores
// (v_mfma_f32_16x16x4_f32: exact products, FP32 accumulation):
//   dW[N][K] = dZ^T A over a split of the batch rows (partials, summed in a
//   fixed order by the update), and the split's FP64 column sums of dZ (db);
//   dZ_prev (B x K) = (dZ W) gelu'(Z_prev), if there is a layer before.
// The inner dimension advances in slabs of 64, the next slab's loads in flight
// during the products. With slabs of 16 loaded and used in turn a product was a
// chain of sixteen memory latencies; the accumulation order of every output is
// the same. A batch of 4096: 21 us a 256 x 256 layer (1.1 GFLOP, 50 TFLOP/s; bound by
// the LDS reads that feed the products) where the two products, the column sums and
// gelu' took 40 + 30 + 17 + 6 us in launches of their own; a training step takes
// 120 us of GPU time instead of 530.
constexpr int BK_TILE = 64, BK_SLAB = 64;
// LDS row pitches: a wave's four k rows lie on different banks; the odd one also
// spreads the transposing stores of an operand whose rows run along x
constexpr int BK_PITCH = 80, BK_PITCH_X = 81;
constexpr int BK_VEC = BK_SLAB * BK_TILE / 4 / 256;        // 16-byte loads of a thread per slab and operand

struct BackArgs {
  int B, N, K;          // batch rows, outputs and inputs of the layer
  const float* dZ;      // [B][N]
  const float* A;       // [B][K] inputs of the layer
  const float* W;       // [N][K]
  const float* Zp;      // [B][K] pre-activations of the layer before
  float* dZp;           // [B][K], or null
  float* Pw;            // [splits][N][K]
  double* Pb;           // [splits][N]
  int kc, splits;       // batch rows of a split
  int tn, tk, tb;       // tiles over N, K and B
};

// A slab of an operand whose rows run along the inner dimension (element
// (k, x) at src[k ld + x], x < X, k < K; X a multiple of 4): registers, then LDS.
__device__ __forceinline__ void slab_load_k(const float* src, int ld, int k0, int K, int x0, int X, floatx4_t (&r)[BK_VEC]) {
#pragma unroll
  for (int i = 0; i < BK_VEC; ++i) {
    const int e = threadIdx.x + i * 256;
    const int k = k0 + (e >> 4), x = x0 + (e & 15) * 4;
    r[i] = k < K && x < X ? *reinterpret_cast<const floatx4_t*>(src + (long long)k * ld + x)
                          : floatx4_t{0.f, 0.f, 0.f, 0.f};
  }
}
__device__ __forceinline__ void slab_store_k(float* S, const floatx4_t (&r)[BK_VEC]) {
#pragma unroll
  for (int i = 0; i < BK_VEC; ++i) {
    const int e = threadIdx.x + i * 256;
    *reinterpret_cast<floatx4_t*>(S + (e >> 4) * BK_PITCH + (e & 15) * 4) = r[i];
  }
}
// ... and of one whose rows run along x (element (k, x) at src[x ld + k]; K a
// multiple of 4)
__device__ __forceinline__ void slab_load_x(const float* src, int ld, int k0, int K, int x0, int X, floatx4_t (&r)[BK_VEC]) {
#pragma unroll
  for (int i = 0; i < BK_VEC; ++i) {
    const int e = threadIdx.x + i * 256;
    const int x = x0 + (e >> 4), k = k0 + (e & 15) * 4;
    r[i] = k < K && x < X ? *reinterpret_cast<const floatx4_t*>(src + (long long)x * ld + k)
                          : floatx4_t{0.f, 0.f, 0.f, 0.f};
  }
}
__device__ __forceinline__ void slab_store_x(float* S, const floatx4_t (&r)[BK_VEC]) {
#pragma unroll
  for (int i = 0; i < BK_VEC; ++i) {
    const int e = threadIdx.x + i * 256;
#pragma unroll
    for (int j = 0; j < 4; ++j) S[((e & 15) * 4 + j) * BK_PITCH_X + (e >> 4)] = r[i][j];
  }
}

__global__ void __launch_bounds__(256) k_layer_back(BackArgs a) {
  __shared__ __attribute__((aligned(16))) float As[BK_SLAB * BK_PITCH_X];
  __shared__ __attribute__((aligned(16))) float Bs[BK_SLAB * BK_PITCH];
  __shared__ double red[4][BK_TILE];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;  // the wave's 32 x 32 quarter of the tile
  const int nw = a.tn * a.tk * a.splits;
  const bool dw = (int)blockIdx.x < nw;  // which of the two products
  int m0, n0, k0, k1, split = 0;
  if (dw) {
    const int t = blockIdx.x % (a.tn * a.tk);
    split = blockIdx.x / (a.tn * a.tk);
    m0 = (t / a.tk) * BK_TILE;
    n0 = (t % a.tk) * BK_TILE;
    k0 = split * a.kc;
    k1 = min(a.B, k0 + a.kc);
  } else {
    const int t = blockIdx.x - nw;
    m0 = (t / a.tk) * BK_TILE;
    n0 = (t % a.tk) * BK_TILE;
    k0 = 0;
    k1 = a.N;
  }
  floatx4_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  const int pa = dw ? BK_PITCH : BK_PITCH_X;
  const bool bias = dw && n0 == 0;
  double bsum = 0.0;  // column m0 + lane of dZ, rows k0 + wave, k0 + wave + 4, ..
  floatx4_t ra[BK_VEC], rb[BK_VEC];
  const auto load = [&](int k) {
    if (dw) {
      slab_load_k(a.dZ, a.N, k, k1, m0, a.N, ra);
      slab_load_k(a.A, a.K, k, k1, n0, a.K, rb);
    } else {
      slab_load_x(a.dZ, a.N, k, k1, m0, a.B, ra);
      slab_load_k(a.W, a.K, k, k1, n0, a.K, rb);
    }
  };
  load(k0);
  for (int k = k0; k < k1; k += BK_SLAB) {
    if (dw)
      slab_store_k(As, ra);
    else
      slab_store_x(As, ra);
    slab_store_k(Bs, rb);
    __syncthreads();
    if (k + BK_SLAB < k1) load(k + BK_SLAB);
    // lane l feeds A[l % 16][l / 16] and B[l / 16][l % 16] of a 16 x 4 x 16 step
    // and holds C rows 4 (l / 16) .. + 3 of column l % 16
#pragma unroll
    for (int ks = 0; ks < BK_SLAB / 4; ++ks) {
      const int kk = ks * 4 + (lane >> 4);
      float av[2], bv[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        av[t] = As[kk * pa + wm + t * 16 + (lane & 15)];
        bv[t] = Bs[kk * BK_PITCH + wn + t * 16 + (lane & 15)];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i], bv[j], acc[i][j], 0, 0, 0);
    }
    if (bias) {
#pragma unroll
      for (int kk = 0; kk < BK_SLAB; kk += 4) bsum += As[(kk + wave) * pa + lane];
    }
    __syncthreads();
  }
  if (bias) {  // uniform over the work-group
    red[wave][lane] = bsum;
    __syncthreads();
    if (wave == 0 && m0 + lane < a.N)
      a.Pb[(long long)split * a.N + m0 + lane] = red[0][lane] + red[1][lane] + red[2][lane] + red[3][lane];
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int gm = m0 + wm + i * 16 + (lane >> 4) * 4 + r, gn = n0 + wn + j * 16 + (lane & 15);
        if (gn >= a.K) continue;
        if (dw) {
          if (gm < a.N) a.Pw[((long long)split * a.N + gm) * a.K + gn] = acc[i][j][r];
        } else if (gm < a.B) {
          const long long o = (long long)gm * a.K + gn;
          a.dZp[o] = acc[i][j][r] * gelu_prime_f(a.Zp[o]);
        }
      }
}

// weighted MSE on normalized outputs: dyhat = 2 w (yhat - t) / B and loss partials;
// output weights w [16], row weights rw [B] (or null)
__global__ void k_loss(const float* yhat, const float* t, const float* w, const float* rw, const int* idx, long long B,
                       int n_out, float* dy, double* part) {
  __shared__ double red[256];
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  double l = 0.0;
  if (i < B * MLP_OUT) {
    const int j = (int)(i % MLP_OUT);
    float g = 0.f;
    if (j < n_out) {
      const long long r = i / MLP_OUT, s = idx ? idx[r] : r;  // row of t and rw
      const float d = yhat[i] - t[s * MLP_OUT + j];
      const float wj = w[j] * (rw ? rw[s] : 1.0f);
      g = 2.0f * wj * d / (float)B;
      l = (double)wj * (double)d * (double)d / (double)B;
    }
    dy[i] = g;
  }
  red[threadIdx.x] = l;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// Layer spans of the parameter array and of the backward pass's partials.
struct LayerSpans {
  long long off[MLP_LAYERS];   // weights; the biases follow
  int n[MLP_LAYERS], k[MLP_LAYERS];
  long long pw[MLP_LAYERS], pb[MLP_LAYERS];  // offsets of the layer's weight and bias partials
  int splits;
};

// Gradient of parameter i: its partials over the splits in a fixed order.
__device__ __forceinline__ float sum_splits(const LayerSpans& ls, const float* Pw, const double* Pb, long long i) {
#pragma unroll
  for (int L = 0; L < MLP_LAYERS; ++L) {
    const long long r = i - ls.off[L], nk = (long long)ls.n[L] * ls.k[L];
    if (r >= 0 && r < nk) {
      const float* p = Pw + ls.pw[L] + r;
      float v = 0.f;
#pragma unroll 8
      for (int s = 0; s < ls.splits; ++s) v += p[s * nk];
      return v;
    }
    if (r >= nk && r < nk + ls.n[L]) {
      const double* p = Pb + ls.pb[L] + (r - nk);
      double v = 0.0;
#pragma unroll 8
      for (int s = 0; s < ls.splits; ++s) v += p[(long long)s * ls.n[L]];
      return (float)v;
    }
  }
  return 0.f;
}

__global__ void __launch_bounds__(256) k_sum_splits(LayerSpans ls, const float* Pw, const double* Pb, float* g,
                                                    long long count) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i < count) g[i] = sum_splits(ls, Pw, Pb, i);
}

// master FP32 weight -> bf16 hi / lo copies (weight matrices in fragment
// order) and the effective FP32 weights the forward pass uses (hi, or hi + lo
// in precise mode)
__device__ __forceinline__ void split_weight(const LayerSpans& ls, float v, long long i, __bf16* hi, __bf16* lo,
                                             float* eff_bf, float* eff_pr) {
  const __bf16 h = (__bf16)v;
  const __bf16 l = (__bf16)(v - (float)h);
  long long d = i;  // biases and padding keep their place
#pragma unroll
  for (int L = 0; L < MLP_LAYERS; ++L) {
    const long long r = i - ls.off[L];
    if (r >= 0 && r < (long long)ls.n[L] * ls.k[L]) {
      const int nn = (int)(r / ls.k[L]), k = (int)(r % ls.k[L]);
      d = ls.off[L] + frag_offset(nn >> 4, k >> 5, ls.k[L], ((k & 31) >> 3) * 16 + (nn & 15)) + (k & 7);
    }
  }
  hi[d] = h;
  lo[d] = l;
  eff_bf[i] = (float)h;
  eff_pr[i] = (float)h + (float)l;
}

__global__ void k_split(const float* w, __bf16* hi, __bf16* lo, float* eff_bf, float* eff_pr, long long count,
                        LayerSpans ls) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) split_weight(ls, w[i], i, hi, lo, eff_bf, eff_pr);
}

// Targets as the loss sees them, (t - mean) / std in FP64 (networks with a
// skip subtract it on the host).
struct TargetScale {
  double mean[MLP_OUT], std[MLP_OUT];
};
__global__ void k_normalize_targets(const float* t, long long n, int n_out, TargetScale ts, float* out) {
  // a launch has fewer than 2^32 threads, a training set may have more values
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n * MLP_OUT;
       i += (long long)gridDim.x * blockDim.x) {
    const long long r = i / MLP_OUT;
    const int j = (int)(i % MLP_OUT);
    out[i] = j < n_out ? (float)(((double)t[r * n_out + j] - ts.mean[j]) / ts.std[j]) : 0.f;
  }
}

// One training step's end: gradient from the partials, Adam, the weight
// copies, and (the last work-group) the step's loss added to the epoch's.
struct UpdateArgs {
  LayerSpans ls;
  const float* Pw;
  const double* Pb;
  float *w, *m, *v;
  __bf16 *hi, *lo;
  float *eff_bf, *eff_pr;
  long long count;
  float lr, b1, b2, c1, c2, eps;
  const double* lpart;  // loss partials of the step
  int nl;
  double* loss;
};
__global__ void __launch_bounds__(256) k_update(UpdateArgs a) {
  if (blockIdx.x == gridDim.x - 1) {  // fixed-order sum of the loss partials
    __shared__ double red[256];
    double v = 0.0;
    for (int i = threadIdx.x; i < a.nl; i += 256) v += a.lpart[i];
    red[threadIdx.x] = v;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
      if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
      __syncthreads();
    }
    if (threadIdx.x == 0) *a.loss += red[0];
    return;
  }
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= a.count) return;
  const float gi = sum_splits(a.ls, a.Pw, a.Pb, i);
  const float mi = a.b1 * a.m[i] + (1.f - a.b1) * gi;
  const float vi = a.b2 * a.v[i] + (1.f - a.b2) * gi * gi;
  a.m[i] = mi;
  a.v[i] = vi;
  const float wi = a.w[i] - a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
  a.w[i] = wi;
  split_weight(a.ls, wi, i, a.hi, a.lo, a.eff_bf, a.eff_pr);
}

// M networks: y = mean, spread = RMS pairwise distance of the stress outputs
// (sqrt(2 / (M - 1) sum_m |s_m - s_mean|^2), |s_a - s_b| for two networks)
// over max(|s_mean|, floor_scale)
__global__ void k_accept_n(const float* ys /* [M][n][n_out] */, int M, long long n, int n_out, float* y,
                           float* spread, uint8_t* accept, float thr, float floor_scale) {
  const long long r = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  const float inv = 1.f / (float)M;
  float d2 = 0.f, m2 = 0.f;
  for (int j = 0; j < n_out; ++j) {
    float mean = 0.f;
    for (int m = 0; m < M; ++m) mean += ys[((long long)m * n + r) * n_out + j];
    mean *= inv;
    y[r * n_out + j] = mean;
    if (j < 6) {
      for (int m = 0; m < M; ++m) {
        const float d = ys[((long long)m * n + r) * n_out + j] - mean;
        d2 += d * d;
      }
      m2 += mean * mean;
    }
  }
  const float s = sqrtf(2.f * d2 / (float)(M - 1)) / fmaxf(sqrtf(m2), floor_scale);
  spread[r] = s;
  accept[r] = s <= thr ? 1 : 0;
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
static int lay_k(int l) { return l == 0 ? MLP_IN : MLP_W; }
static int lay_n(int l) { return l == MLP_LAYERS - 1 ? MLP_OUT : MLP_W; }

Mlp::Mlp(int n_in_, int n_out_, uint64_t seed) : n_in(n_in_), n_out(n_out_) {
  if (n_in < 1 || n_in > MLP_IN || n_out < 1 || n_out > MLP_OUT) fail(HOM_E_ARG, "network size out of range");
  size_t off = 0;
  for (int l = 0; l < MLP_LAYERS; ++l) {
    woff[l] = off;
    off += (size_t)lay_n(l) * lay_k(l);
    boff[l] = off;
    off += lay_n(l);
  }
  npad = off;
  auto alloc = [&](void** p, size_t b) {
    HIPCHK(hipMalloc(p, b));
    HIPCHK(hipMemset(*p, 0, b));
    allocs.push_back(*p);
  };
  alloc((void**)&w, npad * 4);
  alloc((void**)&g, npad * 4);
  alloc((void**)&m, npad * 4);
  alloc((void**)&v, npad * 4);
  alloc((void**)&eff_bf, npad * 4);
  alloc((void**)&eff_pr, npad * 4);
  alloc((void**)&hi, npad * 2);
  alloc((void**)&lo, npad * 2);
  alloc((void**)&scal, 5 * MLP_OUT * 4 + 2 * MLP_IN * 4);
  // G and c in FP32, then G's bf16 hi and lo parts
  alloc((void**)&skip, (MLP_OUT * MLP_GATES * MLP_IN + MLP_OUT) * 4 + 2 * MLP_OUT * MLP_GATES * MLP_IN * 2);
  // He initialization (normal, std sqrt(2 / fan_in)), seeded; biases zero
  std::vector<float> hw(npad, 0.f);
  std::mt19937_64 gen(seed);
  for (int l = 0; l < MLP_LAYERS; ++l) {
    const int K = lay_k(l), N = lay_n(l);
    const int kin = l == 0 ? n_in : K;
    const int nout = l == MLP_LAYERS - 1 ? n_out : N;
    std::normal_distribution<double> nd(0.0, std::sqrt((l == MLP_LAYERS - 1 ? 1.0 : 2.0) / kin));
    for (int i = 0; i < nout; ++i)
      for (int k = 0; k < kin; ++k) hw[woff[l] + (size_t)i * K + k] = (float)nd(gen);
  }
  HIPCHK(hipMemcpy(w, hw.data(), npad * 4, hipMemcpyHostToDevice));
  std::vector<float> s(5 * MLP_OUT + 2 * MLP_IN, 0.f);
  for (int j = 0; j < MLP_IN; ++j) s[MLP_IN + j] = 1.f;            // xinv
  for (int j = 0; j < MLP_OUT; ++j) s[2 * MLP_IN + MLP_OUT + j] = 1.f;  // ystd
  for (int j = 0; j < MLP_OUT; ++j) s[2 * MLP_IN + 2 * MLP_OUT + j] = 1.f;  // loss weights
  HIPCHK(hipMemcpy(scal, s.data(), s.size() * 4, hipMemcpyHostToDevice));
  hx_mean.assign(n_in, 0.f);
  hx_inv.assign(n_in, 1.f);
  hy_mean.assign(n_out, 0.f);
  hy_std.assign(n_out, 1.f);
  refresh(nullptr);
  HIPCHK(hipDeviceSynchronize());
}

Mlp::~Mlp() {
  free_work();
  for (void* p : allocs) (void)hipFree(p);
  if (splitk) (void)hipFree(splitk);
  if (csum) (void)hipFree(csum);
}

void Mlp::free_work() {
  for (void* p : work) (void)hipFree(p);
  work.clear();
  work_rows = 0;
}

static LayerSpans layer_spans(const Mlp& net, int splits) {
  LayerSpans ls;
  long long pw = 0, pb = 0;
  for (int l = 0; l < MLP_LAYERS; ++l) {
    ls.off[l] = (long long)net.woff[l];
    ls.n[l] = lay_n(l);
    ls.k[l] = lay_k(l);
    ls.pw[l] = pw;
    ls.pb[l] = pb;
    pw += (long long)splits * ls.n[l] * ls.k[l];
    pb += (long long)splits * ls.n[l];
  }
  ls.splits = splits;
  return ls;
}

void Mlp::refresh(hipStream_t s) {
  const long long n = (long long)npad;
  hipLaunchKernelGGL(k_split, dim3((n + 255) / 256), dim3(256), 0, s, w, hi, lo, eff_bf, eff_pr, n,
                     layer_spans(*this, 1));
}

void Mlp::set_scaling(const float* xmean, const float* xstd, const float* ymean, const float* ystd,
                      const float* lw) {
  std::vector<float> s(5 * MLP_OUT + 2 * MLP_IN, 0.f);
  for (int j = 0; j < MLP_IN; ++j) {
    s[j] = j < n_in ? xmean[j] : 0.f;
    s[MLP_IN + j] = j < n_in ? 1.f / xstd[j] : 1.f;
    if (j < n_in && !(xstd[j] > 0.f)) fail(HOM_E_ARG, "input scale must be positive");
  }
  for (int j = 0; j < MLP_OUT; ++j) {
    s[2 * MLP_IN + j] = j < n_out ? ymean[j] : 0.f;
    s[2 * MLP_IN + MLP_OUT + j] = j < n_out ? ystd[j] : 1.f;
    s[2 * MLP_IN + 2 * MLP_OUT + j] = j < n_out ? (lw ? lw[j] : 1.f) : 0.f;
    if (j < n_out && !(ystd[j] > 0.f)) fail(HOM_E_ARG, "output scale must be positive");
  }
  HIPCHK(hipMemcpy(scal, s.data(), s.size() * 4, hipMemcpyHostToDevice));
  for (int j = 0; j < n_in; ++j) {
    hx_mean[j] = xmean[j];
    hx_inv[j] = 1.f / xstd[j];
  }
  for (int j = 0; j < n_out; ++j) {
    hy_mean[j] = ymean[j];
    hy_std[j] = ystd[j];
  }
}

void Mlp::normalized_targets(const float* X, const float* T, long long n, float* out) const {
  std::vector<double> xn(n_in);
  for (long long r = 0; r < n; ++r) {
    if (!hskip.empty()) normalize_row(X + r * n_in, xn.data());
    for (int j = 0; j < MLP_OUT; ++j) {
      float v = 0.f;
      if (j < n_out) {
        const double sk = hskip.empty() ? 0.0 : skip_value(xn.data(), j);
        v = (float)((T[r * n_out + j] - sk - hy_mean[j]) / hy_std[j]);
      }
      out[r * MLP_OUT + j] = v;
    }
  }
}

void Mlp::set_skip(const int* gates, const float* G, const float* c) {
  for (int i = 0; i < 3; ++i) {
    if (gates[i] < 0 || gates[i] >= n_in) fail(HOM_E_ARG, "gate index out of range");
    gate[i] = gates[i];
  }
  std::vector<float> f(MLP_OUT * MLP_GATES * MLP_IN + MLP_OUT, 0.f);
  hskip.assign((size_t)n_out * MLP_GATES * n_in + n_out, 0.0);
  for (int j = 0; j < n_out; ++j) {
    for (int g = 0; g < MLP_GATES; ++g)
      for (int k = 0; k < n_in; ++k) {
        const float v = G[((size_t)j * MLP_GATES + g) * n_in + k];
        f[((size_t)j * MLP_GATES + g) * MLP_IN + k] = v;
        hskip[((size_t)j * MLP_GATES + g) * n_in + k] = v;
      }
    f[MLP_OUT * MLP_GATES * MLP_IN + j] = c[j];
    hskip[(size_t)n_out * MLP_GATES * n_in + j] = c[j];
  }
  HIPCHK(hipMemcpy(skip, f.data(), f.size() * 4, hipMemcpyHostToDevice));
  // bf16 hi + lo parts of G (round to nearest even; G is finite)
  const auto bf16_bits = [](float x) {
    uint32_t u;
    std::memcpy(&u, &x, 4);
    return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
  };
  constexpr size_t NG = (size_t)MLP_OUT * MLP_GATES * MLP_IN;
  std::vector<uint16_t> parts(2 * NG);
  for (size_t i = 0; i < NG; ++i) {
    parts[i] = bf16_bits(f[i]);
    const uint32_t hu = (uint32_t)parts[i] << 16;
    float h;
    std::memcpy(&h, &hu, 4);
    parts[NG + i] = bf16_bits(f[i] - h);
  }
  HIPCHK(hipMemcpy(skip + f.size(), parts.data(), parts.size() * 2, hipMemcpyHostToDevice));
}

void Mlp::normalize_row(const float* x, double* xn) const {
  for (int k = 0; k < n_in; ++k) xn[k] = ((double)x[k] - hx_mean[k]) * hx_inv[k];
}

double Mlp::skip_value(const double* xn, int j) const {
  if (hskip.empty()) return 0.0;
  const double va = xn[gate[0]], vb = xn[gate[1]], vc = xn[gate[2]];
  const double s[MLP_GATES] = {1, va, va * va, va * va * va, vb, vb * vb, vb * vb * vb, vc, vc * vc, vc * vc * vc};
  double y = hskip[(size_t)n_out * MLP_GATES * n_in + j];
  for (int g = 0; g < MLP_GATES; ++g) {
    double t = 0.0;
    for (int k = 0; k < n_in; ++k) t += hskip[((size_t)j * MLP_GATES + g) * n_in + k] * xn[k];
    y += s[g] * t;
  }
  return y;
}

// Host-side least squares in FP64: normal equations of the design
// [1, xhat * s_g(xhat)] with a tiny ridge, solved by Cholesky.
void Mlp::fit_skip(const float* X, const float* Y, long long n, const int* gates, const float* lw,
                   const float* rw) {
  if (n < 2) fail(HOM_E_ARG, "need rows to fit");
  for (int i = 0; i < 3; ++i)
    if (gates[i] < 0 || gates[i] >= n_in) fail(HOM_E_ARG, "gate index out of range");
  // input scaling from the rows
  std::vector<double> xm(n_in, 0.0), xv(n_in, 0.0);
  for (long long r = 0; r < n; ++r)
    for (int k = 0; k < n_in; ++k) xm[k] += X[r * n_in + k];
  for (int k = 0; k < n_in; ++k) xm[k] /= (double)n;
  for (long long r = 0; r < n; ++r)
    for (int k = 0; k < n_in; ++k) {
      const double d = X[r * n_in + k] - xm[k];
      xv[k] += d * d;
    }
  std::vector<float> xmf(n_in), xsf(n_in);
  for (int k = 0; k < n_in; ++k) {
    const double sd = std::sqrt(xv[k] / (double)n);
    xmf[k] = (float)xm[k];
    xsf[k] = sd > 1e-12 ? (float)sd : 1.f;
  }
  hx_mean.assign(xmf.begin(), xmf.end());
  hx_inv.resize(n_in);
  for (int k = 0; k < n_in; ++k) hx_inv[k] = 1.f / xsf[k];
  const int P = 1 + MLP_GATES * n_in;
  std::vector<double> AtA((size_t)P * P, 0.0), AtY((size_t)P * n_out, 0.0), phi(P), xn(n_in);
  for (long long r = 0; r < n; ++r) {
    normalize_row(X + r * n_in, xn.data());
    const double va = xn[gates[0]], vb = xn[gates[1]], vc = xn[gates[2]];
    const double s[MLP_GATES] = {1, va, va * va, va * va * va, vb, vb * vb, vb * vb * vb, vc, vc * vc, vc * vc * vc};
    phi[0] = 1.0;
    for (int g = 0; g < MLP_GATES; ++g)
      for (int k = 0; k < n_in; ++k) phi[1 + g * n_in + k] = s[g] * xn[k];
    const double wr = rw ? (double)rw[r] : 1.0;  // weighted least squares
    for (int a = 0; a < P; ++a) {
      const double pa = wr * phi[a];
      double* row = &AtA[(size_t)a * P];
      for (int b = 0; b <= a; ++b) row[b] += pa * phi[b];
      for (int j = 0; j < n_out; ++j) AtY[(size_t)a * n_out + j] += pa * Y[r * n_out + j];
    }
  }
  double tr = 0.0;
  for (int a = 0; a < P; ++a) tr += AtA[(size_t)a * P + a];
  // Cholesky (lower, in place) with a small ridge; the cubic gate features
  // make the normal equations ill-conditioned, so the ridge grows until the
  // factorization succeeds in FP64
  const std::vector<double> A0(AtA);
  bool ok = false;
  for (double ridge : {1e-12, 1e-10, 1e-8, 1e-6}) {
    AtA = A0;
    for (int a = 0; a < P; ++a) AtA[(size_t)a * P + a] += ridge * tr / P;
    ok = true;
    for (int j = 0; j < P && ok; ++j) {
      double d = AtA[(size_t)j * P + j];
      for (int k = 0; k < j; ++k) d -= AtA[(size_t)j * P + k] * AtA[(size_t)j * P + k];
      if (!(d > 0.0)) {
        ok = false;
        break;
      }
      d = std::sqrt(d);
      AtA[(size_t)j * P + j] = d;
      for (int i = j + 1; i < P; ++i) {
        double v = AtA[(size_t)i * P + j];
        for (int k = 0; k < j; ++k) v -= AtA[(size_t)i * P + k] * AtA[(size_t)j * P + k];
        AtA[(size_t)i * P + j] = v / d;
      }
    }
    if (ok) break;
  }
  if (!ok) fail(HOM_E_NAN, "skip fit: normal equations not positive definite");
  std::vector<float> G((size_t)n_out * MLP_GATES * n_in), c(n_out);
  std::vector<double> z(P);
  for (int j = 0; j < n_out; ++j) {
    for (int i = 0; i < P; ++i) {
      double v = AtY[(size_t)i * n_out + j];
      for (int k = 0; k < i; ++k) v -= AtA[(size_t)i * P + k] * z[k];
      z[i] = v / AtA[(size_t)i * P + i];
    }
    for (int i = P - 1; i >= 0; --i) {
      double v = z[i];
      for (int k = i + 1; k < P; ++k) v -= AtA[(size_t)k * P + i] * z[k];
      z[i] = v / AtA[(size_t)i * P + i];
    }
    c[j] = (float)z[0];
    for (int g = 0; g < MLP_GATES; ++g)
      for (int k = 0; k < n_in; ++k) G[((size_t)j * MLP_GATES + g) * n_in + k] = (float)z[1 + g * n_in + k];
  }
  set_skip(gates, G.data(), c.data());
  // residual scaling
  std::vector<double> rm(n_out, 0.0), rv(n_out, 0.0);
  std::vector<double> res((size_t)n * n_out);
  for (long long r = 0; r < n; ++r) {
    normalize_row(X + r * n_in, xn.data());
    for (int j = 0; j < n_out; ++j) {
      const double v = Y[r * n_out + j] - skip_value(xn.data(), j);
      res[r * n_out + j] = v;
      rm[j] += v;
    }
  }
  for (int j = 0; j < n_out; ++j) rm[j] /= (double)n;
  for (long long r = 0; r < n; ++r)
    for (int j = 0; j < n_out; ++j) rv[j] += (res[r * n_out + j] - rm[j]) * (res[r * n_out + j] - rm[j]);
  std::vector<float> rmf(n_out), rsf(n_out);
  for (int j = 0; j < n_out; ++j) {
    const double sd = std::sqrt(rv[j] / (double)n);
    rmf[j] = (float)rm[j];
    rsf[j] = sd > 1e-12 ? (float)sd : 1.f;
  }
  set_scaling(xmf.data(), xsf.data(), rmf.data(), rsf.data(), lw);
}

void Mlp::ensure_work(long long rows) {
  if (rows <= work_rows) return;
  free_work();
  auto alloc = [&](float** p, size_t count) {
    HIPCHK(hipMalloc((void**)p, count * 4));
    work.push_back(*p);
  };
  alloc(&xs, rows * MLP_IN);
  for (int l = 0; l < MLP_LAYERS - 1; ++l) {
    alloc(&zs[l], rows * MLP_W);
    alloc(&as[l], rows * MLP_W);
  }
  alloc(&yhat, rows * MLP_OUT);
  alloc(&dy, rows * MLP_OUT);
  alloc(&dz[0], rows * MLP_W);
  alloc(&dz[1], rows * MLP_W);
  alloc(&lpart, (rows * MLP_OUT + 255) / 256 * 2);
  work_rows = rows;
}

template <int PRECISE, bool SAVE>
static void launch_fwd(const FwdArgs& a, int nets, hipStream_t s) {
  const long long few = (a.n + 15) / 16;
  if (few * nets <= few_groups(PRECISE))
    hipLaunchKernelGGL((k_mlp_fwd<PRECISE, SAVE, 16>), dim3((unsigned)few, nets), dim3(FWD_WAVES * 64), 0, s, a);
  else
    hipLaunchKernelGGL((k_mlp_fwd<PRECISE, SAVE, 64>), dim3((unsigned)((a.n + 63) / 64), nets), dim3(FWD_WAVES * 64), 0,
                       s, a);
}

static FwdArgs forward_args(const Mlp* const* nets, int M, const float* x, float* y, long long n) {
  FwdArgs a;
  std::memset(&a, 0, sizeof(a));
  a.x = x;
  a.n = n;
  a.n_in = nets[0]->n_in;
  a.n_out = nets[0]->n_out;
  a.y = y;
  for (int l = 0; l < MLP_LAYERS; ++l) {
    a.woff[l] = (int)nets[0]->woff[l];
    a.boff[l] = (int)nets[0]->boff[l];
  }
  for (int m = 0; m < M; ++m) {
    const Mlp& net = *nets[m];
    a.net[m] = NetRef{net.hi, net.lo, net.w, net.scal, net.skip, net.gate[0], net.gate[1], net.gate[2]};
  }
  return a;
}

void Mlp::forward(const float* x, float* y, long long n, bool precise, bool save, hipStream_t s, const int* idx) {
  const Mlp* self = this;
  FwdArgs a = forward_args(&self, 1, x, y, n);
  a.idx = idx;
  if (save) {
    a.yhat = yhat;
    a.xs = xs;
    for (int l = 0; l < MLP_LAYERS - 1; ++l) {
      a.zs[l] = zs[l];
      a.as[l] = as[l];
    }
    precise ? launch_fwd<1, true>(a, 1, s) : launch_fwd<0, true>(a, 1, s);
  } else {
    precise ? launch_fwd<1, false>(a, 1, s) : launch_fwd<0, false>(a, 1, s);
  }
}

// Batch rows of a split of the weight gradients: 256 each, at most 64 splits
// (fewer than 1024 rows: one)
static int back_splits(long long B, int& kc) {
  const int splits = B >= 1024 ? (int)std::min<long long>(64, B / 256) : 1;
  kc = (int)((B + splits - 1) / splits);
  return (int)((B + kc - 1) / kc);  // every split has at least one row
}

// loss and gradient of the rows (x raw [B][n_in], t normalized [B][16], or
// their rows idx)
double Mlp::loss_grad(const float* x, const float* tnorm, long long B, bool precise, hipStream_t s,
                      const float* rw) {
  const int lb = grad_partials(x, tnorm, B, precise, s, rw, nullptr);
  const long long np = (long long)npad;
  int kc;
  hipLaunchKernelGGL(k_sum_splits, dim3((unsigned)((np + 255) / 256)), dim3(256), 0, s,
                     layer_spans(*this, back_splits(B, kc)), splitk, csum, g, np);
  std::vector<double> lp(lb);
  HIPCHK(hipMemcpyAsync(lp.data(), lpart, lb * sizeof(double), hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  double L = 0.0;
  for (double v : lp) L += v;
  return L;
}

int Mlp::grad_partials(const float* x, const float* tnorm, long long B, bool precise, hipStream_t s, const float* rw,
                       const int* idx) {
  ensure_work(B);
  int kc;
  const int splits = back_splits(B, kc);
  const LayerSpans ls = layer_spans(*this, splits);
  const size_t needw = (size_t)ls.pw[MLP_LAYERS - 1] + (size_t)splits * MLP_OUT * MLP_W;
  const size_t needb = (size_t)ls.pb[MLP_LAYERS - 1] + (size_t)splits * MLP_OUT;
  if (needw > splitk_n) {
    if (splitk) HIPCHK(hipFree(splitk));
    splitk = nullptr;
    splitk_n = 0;
    HIPCHK(hipMalloc((void**)&splitk, needw * sizeof(float)));
    splitk_n = needw;
  }
  if (needb > csum_n) {
    if (csum) HIPCHK(hipFree(csum));
    csum = nullptr;
    csum_n = 0;
    HIPCHK(hipMalloc((void**)&csum, needb * sizeof(double)));
    csum_n = needb;
  }
  forward(x, nullptr, B, precise, true, s, idx);
  const long long cnt = B * MLP_OUT;
  const int lb = (int)((cnt + 255) / 256);
  hipLaunchKernelGGL(k_loss, dim3(lb), dim3(256), 0, s, yhat, tnorm, scal + 2 * MLP_IN + 2 * MLP_OUT, rw, idx, B,
                     n_out, dy, reinterpret_cast<double*>(lpart));
  const float* eff = precise ? eff_pr : eff_bf;
  const float* dcur = dy;
  for (int l = MLP_LAYERS - 1; l >= 0; --l) {
    BackArgs a;
    a.B = (int)B;
    a.N = lay_n(l);
    a.K = lay_k(l);
    a.dZ = dcur;
    a.A = l == 0 ? xs : as[l - 1];
    a.W = eff + woff[l];
    a.Zp = l > 0 ? zs[l - 1] : nullptr;
    a.dZp = l > 0 ? dz[l & 1] : nullptr;  // not the buffer that this layer reads
    a.Pw = splitk + ls.pw[l];
    a.Pb = csum + ls.pb[l];
    a.kc = kc;
    a.splits = splits;
    a.tn = (a.N + BK_TILE - 1) / BK_TILE;
    a.tk = (a.K + BK_TILE - 1) / BK_TILE;
    a.tb = (int)((B + BK_TILE - 1) / BK_TILE);
    const unsigned groups = (unsigned)(a.tn * a.tk * splits + (l > 0 ? a.tb * a.tk : 0));
    hipLaunchKernelGGL(k_layer_back, dim3(groups), dim3(256), 0, s, a);
    dcur = a.dZp;
  }
  return lb;
}

void Mlp::get_params(float* out) const {
  std::vector<float> hw(npad);
  HIPCHK(hipMemcpy(hw.data(), w, npad * 4, hipMemcpyDeviceToHost));
  size_t o = 0;
  for (int l = 0; l < MLP_LAYERS; ++l) {
    const int K = lay_k(l);
    const int kin = l == 0 ? n_in : K;
    const int nout = l == MLP_LAYERS - 1 ? n_out : lay_n(l);
    for (int i = 0; i < nout; ++i)
      for (int k = 0; k < kin; ++k) out[o++] = hw[woff[l] + (size_t)i * K + k];
    for (int i = 0; i < nout; ++i) out[o++] = hw[boff[l] + i];
  }
}

void Mlp::get_grads(float* out) const {
  std::vector<float> hg(npad);
  HIPCHK(hipMemcpy(hg.data(), g, npad * 4, hipMemcpyDeviceToHost));
  size_t o = 0;
  for (int l = 0; l < MLP_LAYERS; ++l) {
    const int K = lay_k(l);
    const int kin = l == 0 ? n_in : K;
    const int nout = l == MLP_LAYERS - 1 ? n_out : lay_n(l);
    for (int i = 0; i < nout; ++i)
      for (int k = 0; k < kin; ++k) out[o++] = hg[woff[l] + (size_t)i * K + k];
    for (int i = 0; i < nout; ++i) out[o++] = hg[boff[l] + i];
  }
}

void Mlp::set_params(const float* in) {
  std::vector<float> hw(npad, 0.f);
  size_t o = 0;
  for (int l = 0; l < MLP_LAYERS; ++l) {
    const int K = lay_k(l);
    const int kin = l == 0 ? n_in : K;
    const int nout = l == MLP_LAYERS - 1 ? n_out : lay_n(l);
    for (int i = 0; i < nout; ++i)
      for (int k = 0; k < kin; ++k) hw[woff[l] + (size_t)i * K + k] = in[o++];
    for (int i = 0; i < nout; ++i) hw[boff[l] + i] = in[o++];
  }
  HIPCHK(hipMemcpy(w, hw.data(), npad * 4, hipMemcpyHostToDevice));
  refresh(nullptr);
  HIPCHK(hipDeviceSynchronize());
}

size_t Mlp::param_count() const {
  size_t c = 0;
  for (int l = 0; l < MLP_LAYERS; ++l) {
    const int kin = l == 0 ? n_in : lay_k(l);
    const int nout = l == MLP_LAYERS - 1 ? n_out : lay_n(l);
    c += (size_t)nout * kin + nout;
  }
  return c;
}

void Mlp::train(const float* X, const float* T, long long n, int epochs, int batch, double lr0, uint64_t seed,
                const float* row_weight, float* loss_out) {
  if (n < batch || batch < 1) fail(HOM_E_ARG, "need at least one full batch");
  // a stream of this call (default priority): networks trained from several
  // host threads overlap on the device
  hipStream_t s = nullptr;
  HIPCHK(hipStreamCreateWithFlags(&s, hipStreamNonBlocking));
  struct StreamGuard {
    hipStream_t s;
    ~StreamGuard() { (void)hipStreamDestroy(s); }
  } sguard{s};
  // The first epoch's order is drawn while the rows are copied, the targets are
  // normalized on the device and the arrays are one allocation: 16384 rows in two
  // epochs of 4096 a batch 1.55 -> 1.38 ms (1 ms of it the steps' kernels).
  std::mt19937_64 gen(seed);
  std::vector<int> order[2];  // of even and odd epochs: one is drawn while the other may still be copied
  for (auto& o : order) o.resize(n);
  const auto draw_order = [&](int e) {
    std::vector<int>& o = order[e & 1];
    for (long long i = 0; i < n; ++i) o[i] = (int)i;
    std::shuffle(o.begin(), o.end(), gen);
  };
  std::future<void> first_order;
  if (epochs > 0) first_order = std::async(std::launch::async, draw_order, 0);
  // one allocation for the call's arrays: each one's bytes rounded up to 256
  const auto bytes = [](long long b) { return (b + 255) / 256 * 256; };
  const long long bx = bytes(n * n_in * 4), bt = bytes(n * MLP_OUT * 4), bi_ = bytes(n * 4),
                  bw = row_weight ? bytes(n * 4) : 0, bl = bytes(std::max(epochs, 1) * (long long)sizeof(double));
  const bool raw = hskip.empty();  // targets normalized on the device
  const long long br = raw ? bytes(n * n_out * 4) : 0;
  char* base = nullptr;
  HIPCHK(hipMalloc((void**)&base, bx + bt + bi_ + bw + bl + br));
  struct Guard {  // destroyed before sguard: waits for the stream, then frees
    hipStream_t s;
    void* p;
    ~Guard() {
      (void)hipStreamSynchronize(s);
      (void)hipFree(p);
    }
  } guard{s, base};
  float* dX = reinterpret_cast<float*>(base);
  float* dT = reinterpret_cast<float*>(base + bx);
  int* didx = reinterpret_cast<int*>(base + bx + bt);
  float* dW = row_weight ? reinterpret_cast<float*>(base + bx + bt + bi_) : nullptr;
  double* dloss = reinterpret_cast<double*>(base + bx + bt + bi_ + bw);  // per-epoch loss sums
  HIPCHK(hipMemcpy(dX, X, n * n_in * 4, hipMemcpyHostToDevice));
  float* draw = reinterpret_cast<float*>(base + bx + bt + bi_ + bw + bl);  // raw targets
  if (raw) {
    HIPCHK(hipMemcpy(draw, T, n * n_out * 4, hipMemcpyHostToDevice));
  } else {
    std::vector<float> tn((size_t)n * MLP_OUT);
    normalized_targets(X, T, n, tn.data());
    HIPCHK(hipMemcpy(dT, tn.data(), tn.size() * 4, hipMemcpyHostToDevice));
  }
  if (row_weight) {  // scaled to mean 1, so the learning rate keeps its meaning
    double sum = 0.0;
    for (long long r = 0; r < n; ++r) sum += row_weight[r];
    if (!(sum > 0.0)) fail(HOM_E_ARG, "row weights sum to zero");
    std::vector<float> rw(row_weight, row_weight + n);
    for (float& x : rw) x = (float)(x * (double)n / sum);
    HIPCHK(hipMemcpy(dW, rw.data(), n * 4, hipMemcpyHostToDevice));
  }
  ensure_work(batch);
  const long long steps_per_epoch = n / batch;
  HIPCHK(hipMemsetAsync(dloss, 0, std::max(epochs, 1) * sizeof(double), s));
  // the copies went over the null stream, which this non-blocking stream does
  // not wait for
  HIPCHK(hipStreamSynchronize(nullptr));
  if (raw) {
    TargetScale ts;
    for (int j = 0; j < MLP_OUT; ++j) {
      ts.mean[j] = j < n_out ? hy_mean[j] : 0.0;
      ts.std[j] = j < n_out ? hy_std[j] : 1.0;
    }
    const unsigned blocks = (unsigned)std::min<long long>((n * MLP_OUT + 255) / 256, 1 << 16);
    hipLaunchKernelGGL(k_normalize_targets, dim3(blocks), dim3(256), 0, s, draw, n, n_out, ts, dT);
    HIPCHK(hipGetLastError());
  }
  const long long total = steps_per_epoch * epochs;
  long long step = 0;
  const float b1 = 0.9f, b2 = 0.999f;
  for (int e = 0; e < epochs; ++e) {
    if (e == 0)
      first_order.get();
    else
      draw_order(e);
    HIPCHK(hipStreamSynchronize(s));  // the last epoch's order has been copied, and read
    HIPCHK(hipMemcpyAsync(didx, order[e & 1].data(), n * 4, hipMemcpyHostToDevice, s));
    for (long long sidx = 0; sidx < steps_per_epoch; ++sidx) {
      const int* bi = didx + sidx * batch;
      const int lb = grad_partials(dX, dT, batch, false, s, dW, bi);
      ++step;
      // cosine decay to 1 % with a short warm-up
      const double prog = (double)step / (double)total;
      double lr = lr0 * (0.01 + 0.99 * 0.5 * (1.0 + std::cos(3.14159265358979 * prog)));
      if (step < 200) lr *= (double)step / 200.0;
      const float c1 = 1.f - std::pow(b1, (float)step), c2 = 1.f - std::pow(b2, (float)step);
      UpdateArgs u;
      int kc;
      u.ls = layer_spans(*this, back_splits(batch, kc));
      u.Pw = splitk;
      u.Pb = csum;
      u.w = w;
      u.m = m;
      u.v = v;
      u.hi = hi;
      u.lo = lo;
      u.eff_bf = eff_bf;
      u.eff_pr = eff_pr;
      u.count = (long long)npad;
      u.lr = (float)lr;
      u.b1 = b1;
      u.b2 = b2;
      u.c1 = c1;
      u.c2 = c2;
      u.eps = 1e-8f;
      u.lpart = reinterpret_cast<const double*>(lpart);
      u.nl = lb;
      u.loss = dloss + e;
      hipLaunchKernelGGL(k_update, dim3((unsigned)((u.count + 255) / 256 + 1)), dim3(256), 0, s, u);
    }
  }
  HIPCHK(hipStreamSynchronize(s));
  if (loss_out && epochs > 0) {
    std::vector<double> hl(epochs);
    HIPCHK(hipMemcpy(hl.data(), dloss, epochs * sizeof(double), hipMemcpyDeviceToHost));
    for (int e = 0; e < epochs; ++e) loss_out[e] = (float)(hl[e] / steps_per_epoch);
  }
}

void Mlp::reset_optimizer() {
  HIPCHK(hipMemset(m, 0, npad * 4));
  HIPCHK(hipMemset(v, 0, npad * 4));
  HIPCHK(hipDeviceSynchronize());
}

void ensemble_accept(const Mlp* const* nets, int M, const float* x, float* y, float* ys, float* spread,
                        uint8_t* accept, long long n, float thr, float floor_scale, hipStream_t s) {
  const int n_out = nets[0]->n_out;
  // every network in one launch: a few rows are bound by the latency of a
  // work-group's layers
  launch_fwd<0, false>(forward_args(nets, M, x, ys, n), M, s);
  hipLaunchKernelGGL(k_accept_n, dim3((n + 255) / 256), dim3(256), 0, s, ys, M, n, n_out, y, spread, accept, thr,
                     floor_scale);
}

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float* g_scratch_ptr[kMaxDevices] = {};  // device address of `scratch`, per device
}  // namespace

// address of the static array on the current device, looked up once per device
static float* static_scratch() {
  int dev = 0;
  HIPCHK(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) fail(HOM_E_DEVICE, "device index beyond the static scratch table");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    HIPCHK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    g_scratch_ptr[dev] = static_cast<float*>(p);
  }
  return g_scratch_ptr[dev];
}

void ensemble_accept_static(const Mlp* const* nets, int M, const float* x, float* y, float* spread, uint8_t* accept,
                            long long n, float thr, float floor_scale, hipStream_t s) {
  const unsigned long long need = (unsigned long long)n * (unsigned long long)M * (unsigned long long)nets[0]->n_out;
  if (need > (unsigned long long)HOM_STATIC_SCRATCH_FLOATS)
    fail(HOM_E_ARG, "rows x networks x outputs = " + std::to_string(need) + " exceeds the static scratch of " +
                        std::to_string(HOM_STATIC_SCRATCH_FLOATS) + " floats");
  ensemble_accept(nets, M, x, y, static_scratch(), spread, accept, n, thr, floor_scale, s);
}

}  // namespace hom
