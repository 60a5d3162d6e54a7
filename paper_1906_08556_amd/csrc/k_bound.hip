// Candidate selection by an upper bound (large batches, C >= 512).
//
// The dense kernel (k_frame.hip) forms all C expanded-feature scores of a
// frame in FP32 on the matrix cores: 2 K C FLOP per frame (K = 1891 at D = 60),
// 235 ms for 4M frames, although all but one or two components lie hundreds of
// nats below the frame's best.  Here a bound that is never below a component's
// score is formed for all of them first, and only the few that the bound
// cannot exclude are scored:
//
//   ||L_c^-1 (x - mu_c)||^2 >= ||W_c (x - mu_c)||^2  for any W_c with
//   W_c^T W_c <= P_c = Sigma_c^-1.  W_c (32 x D, two blocks of 16 rows) is the
//   Nystroem minorant of P_c on its dominant subspace (k_bound_dirs): the
//   smallest eigenvalues of Sigma_c carry most of the distance.
//
// W_c x' (x' = x - shift) runs on v_mfma_f32_32x32x16_f16; the rounding of
// both operands to FP16 is covered by a bound on its norm (see below), so a
// component is dropped only when its score is certainly more than the margin
// below the frame's best.  The steps, per batch:
//
//   k_sample_sums / k_sample_count
//                   the bound of a sample of the frames: whether it excludes
//                   enough of their components to be worth the sweeps; if not,
//                   the steps below get no frames and the dense kernel all
//   k_bound_best    sweep 1 over all components finds the frame's best bound
//                   (16 rows) and keeps the sums of all; the best component is
//                   scored exactly (FP32 L^-1): M, a lower limit of the frame's
//                   maximum
//   k_bound_list    sweep 2 lists the components whose bound (the kept 16 rows,
//                   then 32 where any lane of the wave needs them) reaches
//                   M - margin
//   k_bound_hist / scan / k_bound_scatter
//                   the listed pairs bucketed by component
//   k_bound_quad    FP32 score of every pair through L_c^-1, per-frame maximum
//   k_bound_replay  the pairs within the margin are scored again with the
//                   dense kernel's own arithmetic (the same FP32 products and
//                   fused additions in the same order, or the same BF16 MFMA
//                   sequence), so that the candidate lists are the dense ones
//                   (but for the dense kernel's overflows in mid sweep)
//   k_bound_final   lists sorted into the dense kernel's order, running
//                   maximum, overflow flag
//
// Frames that the bound cannot serve (a list longer than 32 per lane-half,
// non-finite features) go to the dense kernel, which reads their indices.
#include <algorithm>
#include <climits>
#include <cmath>

#include "ivx_internal.h"
#include "k_exact.h"

namespace ivx {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int BR = 32;            // bound rows per component (two blocks of 16)
constexpr int BK = 64;            // features: D, mean (high, low), zero padding
constexpr int BW = 8;             // waves per workgroup of k_bound
constexpr int CH = 4;             // row blocks (component pairs) per LDS stage, sweep 1
constexpr int CL = 8;             // and sweep 2
constexpr int SL = 32;            // listed components per lane-half and frame
constexpr int kReplay = 1 << 16;    // flag bits above the candidate count
constexpr int kFallback = 1 << 20;
constexpr int kListed = 14;       // listed pairs per frame that the entry array holds
constexpr float kRelErr = 4e-6f;    // relative part of the allowance for FP32 scores
constexpr float kFlush = 6.103515625e-5f;  // 2^-14, smallest normal FP16

// ------------------------------------------------------------- preparation
// Directions of the bound, one workgroup per component: W_c [32][64] FP32 with
// W_c^T W_c <= P_c.  S = orthonormal basis from three steps of simultaneous
// iteration with P_c (started on the 32 largest diagonal entries; columns end
// up ordered by dominance, so the first 16 rows are a good bound alone);
// B = P S, G = S^T B = L_G L_G^T, W = L_G^-1 B^T.  For any S, W^T W =
// B G^-1 B^T <= P.  On the workload's covariances the 16-row bound lists 20
// components per frame (19 with exact eigenvectors, 75 with 16 rows of
// L_c^-1), the 32-row one 4.8.
__global__ void __launch_bounds__(256)
k_bound_dirs(const double* __restrict__ linv, const double* __restrict__ cst, int D,
             float* __restrict__ Wd) {
  extern __shared__ double smd[];
  double* P = smd;            // [D][D]
  double* S = P + D * D;      // [D][32]
  double* B = S + D * BR;     // [D][32]
  double* G = B + D * BR;     // [32][32]
  double* rs = G + BR * BR;   // [32]
  double* Lt = S;             // L^-1 packed by columns while P is formed: D (D + 1) / 2 <= 64 D
  const int c = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int Dp = D * (D + 1) / 2;
  if (!isfinite(cst[c])) {  // covariance rejected: the component is never listed
    for (int e = tid; e < BR * 64; e += 256) Wd[(size_t)c * BR * 64 + e] = 0.0f;
    return;
  }
  for (int e = tid; e < Dp; e += 256) Lt[e] = linv[(size_t)c * Dp + e];
  __syncthreads();
  for (int e = tid; e < D * D; e += 256) {
    const int i = e / D, j = e - i * D;
    const int lo = i > j ? i : j;
    const double* ci = Lt + i * D - i * (i - 1) / 2 - i;  // column i: row m at ci[m]
    const double* cj = Lt + j * D - j * (j - 1) / 2 - j;
    double s = 0.0;
    for (int m = lo; m < D; ++m) s += ci[m] * cj[m];
    P[e] = s;
  }
  __syncthreads();
  // B = columns of P with the largest diagonal entries
  if (tid < D) {
    const double v = P[tid * D + tid];
    int r = 0;
    for (int j = 0; j < D; ++j) r += (P[j * D + j] > v) || (P[j * D + j] == v && j < tid);
    if (r < BR)
      for (int i = 0; i < D; ++i) B[i * BR + r] = P[i * D + tid];
  }
  __syncthreads();
  // G = A^T B' (32 x 32, lower part used) = L L^T, kept as L L^T's unscaled
  // columns (pivots on the diagonal): one barrier per column
  auto gram_factor = [&](const double* A, const double* Bm) {
    for (int e = tid; e < BR * BR; e += 256) {
      const int i = e >> 5, j = e & 31;
      double s = 0.0;
      for (int k = 0; k < D; ++k) s += A[k * BR + i] * Bm[k * BR + j];
      G[e] = s;
      if (i == j) rs[i] = s;  // diagonal before the elimination
    }
    __syncthreads();
    for (int j = 0; j < BR; ++j) {
      const double p = G[j * BR + j];
      const bool ok = p > 1e-13 * rs[j];  // lost to rounding: a zero column
      const double inv = ok ? 1.0 / p : 0.0;
      for (int e = tid; e < BR * BR; e += 256) {
        const int i = e >> 5, k = e & 31;
        if (k > j && i >= k) G[e] -= G[i * BR + j] * inv * G[k * BR + j];
      }
      __syncthreads();
      if (tid == 0) rs[j] = ok ? 1.0 / sqrt(p) : 0.0;  // 1 / L_jj
    }
    __syncthreads();
  };
  // out(i) = row i of L^-1 applied to the row `tid` of Bm
  auto solve_row = [&](const double* Bm, double (&w)[BR]) {
    double t[BR];
#pragma unroll
    for (int i = 0; i < BR; ++i) {
      double s = Bm[tid * BR + i];
#pragma unroll
      for (int k = 0; k < i; ++k) s -= G[i * BR + k] * t[k];
      w[i] = s * rs[i];
      t[i] = w[i] * rs[i];
    }
  };
  for (int it = 0; it < 4; ++it) {
    gram_factor(B, B);
    if (tid < D) {  // S = B L^-T: orthonormal columns
      double w[BR];
      solve_row(B, w);
#pragma unroll
      for (int i = 0; i < BR; ++i) S[tid * BR + i] = w[i];
    }
    __syncthreads();
    for (int e = tid; e < D * BR; e += 256) {
      const int i = e >> 5, r = e & 31;
      double s = 0.0;
      for (int k = 0; k < D; ++k) s += P[i * D + k] * S[k * BR + r];
      B[e] = s;
    }
    __syncthreads();
  }
  gram_factor(S, B);
  if (tid < 64) {  // W[:, tid] = L^-1 B[tid, :]^T
    double w[BR];
#pragma unroll
    for (int i = 0; i < BR; ++i) w[i] = 0.0;
    if (tid < D) solve_row(B, w);
#pragma unroll
    for (int i = 0; i < BR; ++i) Wd[(size_t)c * BR * 64 + i * 64 + tid] = (float)w[i];
  }
}

// (w_c, w_c (tr Sigma_c + ||mu'_c||^2) / D), mu' = mu - shift: one wave per component
__global__ void __launch_bounds__(256)
k_bound_spread(const double* __restrict__ w, const double* __restrict__ mu,
               const double* __restrict__ cov, const double* __restrict__ cst,
               const float* __restrict__ shift, int C, int D, double2* __restrict__ spread) {
  const int lane = threadIdx.x & 63, c = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (c >= C) return;
  double v = 0.0;
  if (lane < D) {
    const double m = mu[(size_t)c * D + lane] - (double)shift[lane];
    v = cov[((size_t)c * D + lane) * D + lane] + m * m;
  }
  v = wave_sum(v);
  if (lane == 0) {
    const bool ok = isfinite(cst[c]) && isfinite(v);
    spread[c] = ok ? make_double2(w[c], w[c] * v / D) : make_double2(0.0, 0.0);
  }
}

// The bound works in units of 2^-a of the features, 2^a bringing their root mean
// square per dimension under the model to [2, 4), so that neither the FP16
// range nor the least rounding term of a frame (k_bound_frames) depends on the
// features' scale.  With the features as they come, 131,072 frames at C = 2048, D =
// 60 took 1.50 ms at the workload's scale (a = 0) and 9.5 ms at a hundredth of it.
// W_c mu'_c, Frobenius norms in these units, the largest magnitude of all (bits
// of a non-negative float order as integers), 2^a: one wave per component.
__global__ void __launch_bounds__(256)
k_bound_scale(const float* __restrict__ Wd, const double* __restrict__ mu,
              const double* __restrict__ cst, const float* __restrict__ shift,
              const double2* __restrict__ spread, int C, int D, float* __restrict__ wmu,
              float2* __restrict__ norms, int* __restrict__ maxbits, float* __restrict__ unit) {
  const int lane = threadIdx.x & 63, c = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (c >= C) return;
  double sw = 0.0, sv = 0.0;  // every wave for itself, in the same order
  for (int i = lane; i < C; i += 64) {
    sw += spread[i].x;
    sv += spread[i].y;
  }
  const double rms = sqrt(wave_sum(sv) / wave_sum(sw));
  const int a = rms > 0.0 && isfinite(rms) ? max(-60, min(60, 1 - ilogb(rms))) : 0;
  if (c == 0 && lane == 0) unit[0] = ldexpf(1.0f, a);
  const float iu = ldexpf(1.0f, -a);
  const double m = lane < D ? mu[(size_t)c * D + lane] - (double)shift[lane] : 0.0;
  double fro = 0.0, bm = 0.0;
  float mx = 0.0f;
  for (int i = 0; i < BR; ++i) {
    const float w = lane < D ? Wd[((size_t)c * BR + i) * 64 + lane] : 0.0f;
    const double s = wave_sum((double)w * m), wu = (double)w * iu;
    fro += wu * wu;
    bm += s * s;
    mx = fmaxf(mx, fmaxf(fabsf((float)wu), fabsf((float)s)));
    if (lane == 0) wmu[(size_t)c * BR + i] = (float)s;
  }
  fro = wave_sum(fro);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
  if (lane == 0) {
    norms[c] = make_float2((float)sqrt(fro), (float)sqrt(bm));
    if (isfinite(cst[c]) && isfinite(mx)) atomicMax(maxbits, __float_as_int(mx));
  }
}

// Power of two S that brings the largest magnitude to [2^13, 2^14).
__device__ inline float bound_scale(const int* maxbits) {
  const float m = __int_as_float(maxbits[0]);
  const int ex = m > 0.0f ? ilogbf(m) : 0;
  return ldexpf(1.0f, max(-60, min(60, 13 - ex)));
}

__device__ inline _Float16 to_half(float v) {
  return fabsf(v) < kFlush ? (_Float16)0.0f : (_Float16)v;
}

// FP16 operand in MFMA fragment order, [component pair][block of 16 rows]
// [k step of 16][lane][8]: lane l holds row l % 32, features 16 ks + 8 (l / 32)
// + e.  Rows with bit 2 clear belong to the pair's first component, the others
// to the second, so that a lane of the result holds the 16 rows of one
// component (the first for lanes < 32).  Columns: S W_c, then -S W_c mu'_c
// split into high and low parts (feature value 1), zeros.
// cb[c] = (2 S^2 cst_c, e_c^2): e_c times the frame's rounding term bounds the
// norm of the error of the scaled W_c (x' - mu'_c).
__global__ void __launch_bounds__(256)
k_bound_pack(const float* __restrict__ Wd, const float* __restrict__ wmu,
             const float2* __restrict__ norms, const double* __restrict__ cst, int C, int Cpad,
             int D, const int* __restrict__ maxbits, const float* __restrict__ unit,
             _Float16* __restrict__ Wf, float2* __restrict__ cb) {
  const float S = bound_scale(maxbits), iu = 1.0f / unit[0];
  const int rb = blockIdx.x;  // component pair
  for (int e = threadIdx.x; e < 2 * 4 * 64; e += 256) {
    const int blk = e >> 8, ks = (e >> 6) & 3, l = e & 63;
    const int row = l & 31, c = 2 * rb + ((row >> 2) & 1), i = 16 * blk + (row & 3) + 4 * (row >> 3);
    const bool ok = c < C && isfinite(cst[c]);
    half8 v;
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      const int k = 16 * ks + 8 * (l >> 5) + x;
      float w = 0.0f;
      if (ok) {
        if (k < D) {
          w = S * (iu * Wd[((size_t)c * BR + i) * 64 + k]);
        } else if (k <= D + 1) {
          const float m = -S * wmu[(size_t)c * BR + i];
          const float hi = (float)to_half(m);
          w = k == D ? hi : m - hi;
        }
      }
      v[x] = to_half(w);
    }
    *reinterpret_cast<half8*>(Wf + ((size_t)rb * 512 + e) * 8) = v;
  }
  if (threadIdx.x < 2) {
    const int c = 2 * rb + threadIdx.x;
    // rejected and padding components: never the best, never listed
    float2 o = make_float2(-INFINITY, 0.0f);
    if (c < C && isfinite(cst[c])) {
      const float e = S * (1.001f * norms[c].x + 0.0009765625f * norms[c].y) + 8.0f;
      o = make_float2((float)(2.0 * (double)S * (double)S * cst[c]), e * e);
    }
    cb[c] = o;
  }
}

// L_c^-1 in FP32, [C][16][64][4]: element (row, 4 g + x) at ((c 16 + g) 64 + row) 4 + x
__global__ void k_linv_quads(const double* __restrict__ linv, int C, int D,
                             float* __restrict__ lquad) {
  const int Dp = D * (D + 1) / 2;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < (int64_t)C * 4096;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int c = (int)(e >> 12), g = (int)((e >> 8) & 15), i = (int)((e >> 2) & 63);
    const int j = 4 * g + (int)(e & 3);
    lquad[e] = (i < D && j <= i) ? (float)linv[(size_t)c * Dp + j * D - j * (j - 1) / 2 + (i - j)]
                                 : 0.0f;
  }
}

// ------------------------------------------------------------------ the bound
// Scaled quantities (S: bound_scale; t: the frame's power of two; x', mu' and W in
// the units of k_bound_scale): x^ = fp16(t x'), y^ = S t W (x' - mu') + d with ||d|| <= e_c g, g = ||t x' - x^|| +
// 2^-11 ||x^|| (rounding of the frame, of W_c; the FP32 sums and the split
// mean are inside the rounded-up constants).  A component can reach the
// threshold thr only if
//   ||y^||^2 <= (1 + eta) S^2 t^2 2 (cst_c - thr) + (1 + 1 / eta) e_c^2 g^2
// for any eta > 0 (taken from the frame's best component).

// x^ [F][64] FP16 (columns D and D + 1 hold t, the rest zero) and (t^2, g) of
// every frame; t^2 = -1 marks frames outside the FP16 range (or not finite).
// 16 lanes per frame, four columns each.
__global__ void __launch_bounds__(256)
k_bound_frames(const float* __restrict__ X, int64_t F, int D, const float* __restrict__ shift,
               const float* __restrict__ unit, const int* __restrict__ Fdev,
               _Float16* __restrict__ xh, float2* __restrict__ tg) {
  if (Fdev && (int64_t)Fdev[0] < F) F = Fdev[0];
  const int l16 = threadIdx.x & 15;
  const int64_t g = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
  if (g >= F) return;  // uniform over the frame's 16 lanes
  float v[4], mx = 1.0f;
  const float u0 = unit[0];
  bool fin = true;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int k = 4 * l16 + e;
    v[e] = k < D ? u0 * (X[g * D + k] - shift[k]) : 0.0f;
    fin = fin && isfinite(v[e]);
    mx = fmaxf(mx, fabsf(v[e]));
  }
#pragma unroll
  for (int o = 8; o >= 1; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 16));
  const uint64_t allf = __ballot(fin);
  const bool ok = ((allf >> (threadIdx.x & 48)) & 0xffffull) == 0xffffull && mx < 8388608.0f;
  const float t = ok ? ldexpf(1.0f, 9 - ilogbf(mx)) : 1.0f;  // |x^| < 2^10
  float rho = 0.0f, nx = 0.0f;
  _Float16 q[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int k = 4 * l16 + e;
    const float u = ok ? t * v[e] : 0.0f;
    q[e] = to_half(u);
    const float r = u - (float)q[e];
    rho = fmaf(r, r, rho);
    nx = fmaf((float)q[e], (float)q[e], nx);
    if (k == D || k == D + 1) q[e] = (_Float16)t;
  }
#pragma unroll
  for (int o = 8; o >= 1; o >>= 1) {
    rho += __shfl_xor(rho, o, 16);
    nx += __shfl_xor(nx, o, 16);
  }
  typedef _Float16 half4 __attribute__((ext_vector_type(4)));
  *reinterpret_cast<half4*>(xh + g * BK + 4 * l16) = half4{q[0], q[1], q[2], q[3]};
  if (l16 == 0)
    tg[g] = make_float2(ok ? t * t : -1.0f,
                        fmaxf(1.01f * sqrtf(rho) + 0.000512f * sqrtf(nx), 0.015625f * t));
}

// The test of a frame, in nats: a component can reach thr = M - margin only if
// v <= k1 u + k2 e - k3 with (u, e) its constants in cb and v its sum times rn.
struct BoundTest {
  float k1, k2, k3, rn;
  bool good;  // false: outside the bound's range, nothing passes
};
__device__ inline BoundTest bound_test(float2 q, float S, float M, float margin, bool ok,
                                       const float2* __restrict__ cb, int bc) {
  BoundTest b;
  const float S2x2 = 2.0f * S * S;
  // 3 nats for the FP32 errors of M, of the dense scores and of the test
  const float thr = M - margin - 3.0f - kRelErr * fabsf(M);
  b.good = ok && bc >= 0 && q.x > 0.0f && isfinite(M);
  float eta = 1.0f;
  if (b.good) {
    const float2 cv = cb[bc];
    const float T = q.x * (cv.x - S2x2 * thr);
    eta = fminf(fmaxf(sqrtf(cv.y / T) * q.y, 0.0009765625f), 8.0f);
    if (!(eta > 0.0f)) eta = 1.0f;
  }
  b.rn = 1.0f / (S2x2 * q.x);
  b.k1 = (1.0f + eta) / S2x2;
  b.k2 = (1.0f + 1.0f / eta) * q.y * q.y * b.rn;
  b.k3 = (1.0f + eta) * thr;
  b.good = b.good && isfinite(b.k1) && isfinite(b.k2) && isfinite(b.k3) && isfinite(b.rn);
  if (!b.good) {
    b.k1 = b.k2 = 0.0f;
    b.k3 = INFINITY;
  }
  return b;
}
__device__ inline float bound_limit(const BoundTest& b, float2 cv) {
  return fmaf(b.k1, cv.x, fmaf(b.k2, cv.y, -b.k3));
}

// ------------------------------------------------------------------ the sample
// How many components the bound leaves depends on the model's covariances and on
// the frames: with 32 rows it sees little of a well-conditioned covariance (600
// degrees of freedom instead of the workload's D + 5: 1800 of 2048 components
// pass, every list overflows).  So 32 to 128 frames spread over the batch take
// the test with all 32 rows first (19 us at C = 2048; where the bound
// fails, the sweeps would waste 1.5 ms per 131,072 frames).
constexpr int kSample = 128;
constexpr int SP = 2;  // component pairs per workgroup of k_sample_sums
// Costs by that of one dense tile of 128 frames per CU (2.3 ms in FP32 and 1.0 in
// BF16 at C = 2048, D = 60, proportional to K): the bound's sweeps over F frames b0 +
// b1 F, dearer by 0.4 of the share that it hands on; further dense rounds of two
// tiles per CU h2; a frame by the split scores 1 / 20000.  (C = 2048, D = 60, FP32 /
// BF16: bound 0.67 / 0.70 ms for 36,000 frames, 2.0 / 1.95 for 262,144; dense 2.5 /
// 1.0 ms for 32,768, 4.2 / 1.4 for 65,536.)
struct SampleRule {
  float b0, b1, h2;
  int round, fs;  // frames of a tile per CU, frames of the score buffer
};
__device__ inline bool bound_pays(const SampleRule& r, float F, float p) {
  auto dense = [&](float n) { return n <= r.round ? 1.0f : r.h2 * ceilf(n / (2.0f * r.round)); };
  const float n = p * F;
  return (r.b0 + r.b1 * F) * (1.0f + 0.4f * p) + (n <= r.fs ? n * 5e-5f : dense(n)) < dense(F);
}
__device__ inline int64_t sample_frame(int64_t F, int i, int n) { return F * i / n; }

// sv [ns][Cpad]: the sums over 16 and over 32 rows in nats; a wave per 32 frames
__global__ void __launch_bounds__(256)
k_sample_sums(const _Float16* __restrict__ xh, const float2* __restrict__ tg, int64_t F,
              const _Float16* __restrict__ Wf, const int* __restrict__ maxbits, int Cpad, int ns,
              float2* __restrict__ sv, int* __restrict__ dec, const int* __restrict__ Fdev) {
  if (Fdev && (int64_t)Fdev[0] < F) F = Fdev[0];
  if (blockIdx.x == 0 && threadIdx.x < 5) dec[threadIdx.x] = 0;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, h = lane >> 5, l32 = lane & 31;
  if (F <= 0 || 32 * wave >= ns) return;
  const int64_t g = sample_frame(F, 32 * wave + l32, ns);
  const float S = bound_scale(maxbits);
  const float rn = 1.0f / (2.0f * S * S * tg[g].x);
  half8 xf[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
    xf[ks] = *reinterpret_cast<const half8*>(xh + g * BK + 16 * ks + 8 * h);
  const half8* W8 = reinterpret_cast<const half8*>(Wf) + (size_t)blockIdx.x * SP * 512 + lane;
  float2* out = sv + (size_t)(32 * wave + l32) * Cpad + (size_t)blockIdx.x * SP * 2 + h;
#pragma unroll
  for (int i = 0; i < SP; ++i) {
    float sq[2] = {0.0f, 0.0f};
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
      floatx16 ac = floatx16{0};
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        ac = __builtin_amdgcn_mfma_f32_32x32x16_f16(W8[i * 512 + blk * 256 + ks * 64], xf[ks], ac,
                                                    0, 0, 0);
#pragma unroll
      for (int r = 0; r < 16; ++r) sq[blk] = fmaf(ac[r], ac[r], sq[blk]);
    }
    out[2 * i] = make_float2(sq[0] * rn, (sq[0] + sq[1]) * rn);
  }
}

// One workgroup per sampled frame: its best component (on 16 rows, as in sweep 1),
// that one's exact score, the components that pass.  The last one decides: dec[0]
// frames for the bound, dec[1] for the dense kernel (all or none); dec[2..4]
// counters.
__global__ void __launch_bounds__(256)
k_sample_count(const float* __restrict__ X, int64_t F, int D, const float2* __restrict__ tg,
               const float2* __restrict__ cb, const int* __restrict__ maxbits, int Cpad,
               float margin, const double* __restrict__ mu, const float* __restrict__ lquad,
               const double* __restrict__ cst, const float2* __restrict__ sv, SampleRule rule,
               int* __restrict__ dec, const int* __restrict__ Fdev) {
  __shared__ float ds[64], wv[4], yp[4][64];
  __shared__ int wc[4], odd[4], even[4];
  if (Fdev && (int64_t)Fdev[0] < F) F = Fdev[0];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, ns = gridDim.x;
  const float S = bound_scale(maxbits), r2 = 0.5f / (S * S);
  bool bad = false;
  int cnt = 0;
  if (F > 0) {  // uniform
    const int64_t g = sample_frame(F, blockIdx.x, ns);
    const float2* v = sv + (size_t)blockIdx.x * Cpad;
    float bv = INFINITY;
    int bc = -1;
#pragma unroll 8
    for (int c = tid; c < Cpad; c += 256) {
      const float k = v[c].x - cb[c].x * r2;
      bc = k < bv ? c : bc;
      bv = fminf(k, bv);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      const float ov = __shfl_xor(bv, o);
      const int oc = __shfl_xor(bc, o);
      if (ov < bv || (ov == bv && oc < bc)) bc = oc;
      bv = fminf(bv, ov);
    }
    if (lane == 0) {
      wv[w] = bv;
      wc[w] = bc;
    }
    __syncthreads();
    bv = INFINITY;
    bc = -1;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (wv[i] < bv || (wv[i] == bv && wc[i] < bc)) {
        bv = wv[i];
        bc = wc[i];
      }
    float M = -INFINITY;
    if (bc >= 0) {  // uniform; a quarter of the columns per wave
      if (tid < 64)
        ds[lane] = lane < D ? (float)((double)X[g * D + lane] - mu[(size_t)bc * D + lane]) : 0.0f;
      const float4* Lq = reinterpret_cast<const float4*>(lquad) + (size_t)bc * 1024 + lane;
      float4 l[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) l[q] = Lq[(4 * w + q) * 64];
      __syncthreads();
      float y = 0.0f;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float* d = ds + 16 * w + 4 * q;
        y = fmaf(l[q].x, d[0], y);
        y = fmaf(l[q].y, d[1], y);
        y = fmaf(l[q].z, d[2], y);
        y = fmaf(l[q].w, d[3], y);
      }
      yp[w][lane] = y;
      __syncthreads();
      y = (yp[0][lane] + yp[1][lane]) + (yp[2][lane] + yp[3][lane]);
      float q = y * y;
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) q += __shfl_xor(q, o);
      M = (float)cst[bc] - 0.5f * q;
    }
    const BoundTest b = bound_test(tg[g], S, M, margin, true, cb, bc);
    // c = tid + 256 i: the parity of the thread is the component's
#pragma unroll 8
    for (int c = tid; c < Cpad; c += 256) cnt += v[c].y <= bound_limit(b, cb[c]) ? 1 : 0;
#pragma unroll
    for (int o = 32; o >= 2; o >>= 1) cnt += __shfl_xor(cnt, o);
    if (lane == 0) even[w] = cnt;
    if (lane == 1) odd[w] = cnt;
    __syncthreads();
    const int n0 = even[0] + even[1] + even[2] + even[3], n1 = odd[0] + odd[1] + odd[2] + odd[3];
    bad = !b.good || n0 > SL || n1 > SL;
    cnt = n0 + n1;
  }
  if (tid != 0) return;
  if (bad)
    atomicAdd(dec + 2, 1);
  else
    atomicAdd(dec + 3, cnt);
  __threadfence();
  if (atomicAdd(dec + 4, 1) != ns - 1) return;
  __threadfence();
  const int nbad = atomicAdd(dec + 2, 0), sum = atomicAdd(dec + 3, 0);
  // Pairs beyond kListed per frame do not fit the entry array; a frame with one of
  // them is handed on: of a excess pairs per frame a share of min(1, a), about
  // (14.4 pairs at C = 16384 on the workload's kind of model).
  const float over = fmaxf(0.0f, (float)sum / ns - kListed);
  const bool use = bound_pays(rule, (float)F, fminf(1.0f, (float)nbad / ns + over));
  dec[0] = use ? (int)F : 0;
  dec[1] = use ? 0 : (int)F;
}

// Both sweeps: one persistent workgroup of 8 waves per 256 FB frames, FB blocks
// of 32 frames per wave (lane l: frame l % 32 of each block, component parity
// l / 32).  Sweep 1 is bound by the matrix cores (per 32 x 32 block 4 MFMAs, 128
// cycles, and 21 vector instructions, 84 cycles, which overlap between the four
// waves of a SIMD) and by power: 4 M frames at C = 2048 take 15.1 ms at 1.74 GHz,
// 61 % of the cycles in MFMAs.  The FP16 operand of a pair of components (4 KB
// per 16 rows) is staged through LDS in fragment order and serves the FB frame
// blocks of all waves; at one block per wave the LDS reads alone would take as
// long as the MFMAs.  Sweep 2 reads the sums (16 GB) and forms the second 16
// rows of 43 % of the blocks: 11.1 ms with 8 pairs per stage, 12.7 with 4 (its
// stages are short, the loads of the next must be complete at their end), 22 ms
// when it forms the first 16 rows again (no room for the sums).

// 16 bytes per lane from device memory straight into LDS: lane l's at dst + 16 l
// (dst wave-uniform).  Complete after dma_wait() and a barrier.
__device__ inline void dma16(const uint4* src, uint4* dst) {
  __builtin_amdgcn_global_load_lds(
      (const __attribute__((address_space(1))) void*)src,
      (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}
__device__ inline void dma_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Between the sweeps the 16-row sums of all pairs are kept, so that sweep 2 need
// not form them again: in nats, as FP16 cut towards zero (below 65504), which
// only lowers them: the bound stays a bound.  A lane's values of the CH pairs
// of a stage are 8 bytes, [tile][stage][block][thread].  (8 bits would not do:
// thresholds of 2000 nats are usual, and the cut must stay at a few nats.)
static_assert(CH == 4, "four values per 8 bytes");
typedef __fp16 cut2 __attribute__((ext_vector_type(2)));
typedef uint32_t uint2v __attribute__((ext_vector_type(2)));
__device__ inline uint32_t cut_pair(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(a, b));
}
__device__ inline float cut_value(uint32_t w, int half) {
  return (float)__builtin_bit_cast(cut2, w)[half];
}

// Sweep 1: the component with the largest bound (16 rows) of every frame; KEEP:
// the sums are kept for sweep 2.
template <int FB, bool KEEP>
__global__ void __launch_bounds__(64 * BW, 4)
k_bound_best(const _Float16* __restrict__ xh, const float2* __restrict__ tg, int64_t f0, int64_t F,
             const _Float16* __restrict__ Wf, const float2* __restrict__ cb,
             const int* __restrict__ maxbits, int npair, int* __restrict__ best,
             uint2v* __restrict__ sums, const int* __restrict__ Fdev) {
  __shared__ __attribute__((aligned(16))) uint4 st[2][CH * 256];
  __shared__ float sc[2][2 * CH];
  if (Fdev && (int64_t)Fdev[0] < F) F = Fdev[0];
  constexpr int FT = 32 * BW * FB;
  const int64_t ntile = (F - f0 + FT - 1) / FT;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5, l32 = lane & 31;
  const uint4* W4 = reinterpret_cast<const uint4*>(Wf) + (size_t)(tid >> 8) * 512 + (tid & 255);
  const int nch = npair / CH;
  const float S = bound_scale(maxbits);
  for (int64_t tile = blockIdx.x; tile < ntile; tile += gridDim.x) {
    const int64_t fw = f0 + tile * FT + wave * 32 * FB;
    half8 xf[FB][4];
    float t2[FB], rn[FB], bv[FB];
    int bc[FB];
    float v[FB][CH];
#pragma unroll
    for (int fb = 0; fb < FB; ++fb) {
      const int64_t g = min(fw + 32 * fb + l32, F - 1);
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        xf[fb][ks] = *reinterpret_cast<const half8*>(xh + g * BK + 16 * ks + 8 * h);
      t2[fb] = tg[g].x;
      rn[fb] = 0.5f / (S * S * t2[fb]);
      bv[fb] = INFINITY;
      bc[fb] = -1;
    }
    // stage ch in buffer b: the first 16 rows of CH pairs and their constants
    auto stage = [&](int ch, int b) {
      dma16(W4 + (size_t)ch * CH * 512, &st[b][wave * 64]);
      dma16(W4 + (size_t)ch * CH * 512 + 1024, &st[b][512 + wave * 64]);
      if (tid < 2 * CH) sc[b][tid] = cb[2 * CH * ch + tid].x;
    };
    uint2v* ct = sums + (size_t)tile * nch * FB * (64 * BW) + tid;
    uint2v w[FB];
    auto put = [&](int ch) {
#pragma unroll
      for (int fb = 0; fb < FB; ++fb)
        __builtin_nontemporal_store(w[fb], ct + (size_t)(ch * FB + fb) * (64 * BW));
    };
    __syncthreads();  // the previous tile's stage is consumed
    stage(0, 0);
    dma_wait();
    __syncthreads();
#pragma unroll 1
    for (int ch = 0; ch < nch; ++ch) {
      const int b = ch & 1;
      if (ch + 1 < nch) stage(ch + 1, b ^ 1);  // last read before the previous barrier
      if (KEEP && ch > 0) put(ch - 1);         // complete by the wait below
#pragma unroll
      for (int i = 0; i < CH; ++i) {
        half8 a[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
          a[ks] = *reinterpret_cast<const half8*>(&st[b][i * 256 + ks * 64 + lane]);
        const float u = sc[b][2 * i + h];
        floatx16 acc[FB];
#pragma unroll
        for (int fb = 0; fb < FB; ++fb)
          acc[fb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0], xf[fb][0], floatx16{0}, 0, 0, 0);
#pragma unroll
        for (int ks = 1; ks < 4; ++ks)
#pragma unroll
          for (int fb = 0; fb < FB; ++fb)
            acc[fb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[ks], xf[fb][ks], acc[fb], 0, 0, 0);
        const int c = 2 * (ch * CH + i) + h;
#pragma unroll
        for (int fb = 0; fb < FB; ++fb) {
          float sq = acc[fb][0] * acc[fb][0];
#pragma unroll
          for (int r = 1; r < 16; ++r) sq = fmaf(acc[fb][r], acc[fb][r], sq);
          const float q = fmaf(-u, t2[fb], sq);
          bc[fb] = q < bv[fb] ? c : bc[fb];
          bv[fb] = fminf(q, bv[fb]);
          v[fb][i] = sq * rn[fb];
        }
      }
#pragma unroll
      for (int fb = 0; fb < FB; ++fb)
        w[fb] = uint2v{cut_pair(v[fb][0], v[fb][1]), cut_pair(v[fb][2], v[fb][3])};
      dma_wait();
      __syncthreads();
    }
    if (KEEP) put(nch - 1);
#pragma unroll
    for (int fb = 0; fb < FB; ++fb) {
      const float ov = __shfl_xor(bv[fb], 32);
      const int oc = __shfl_xor(bc[fb], 32);
      if (ov < bv[fb] || (ov == bv[fb] && oc < bc[fb])) bc[fb] = oc;
      const int64_t g = fw + 32 * fb + l32;
      if (h == 0 && g < F) best[g] = t2[fb] > 0.0f ? bc[fb] : -1;
    }
  }
}

// Sweep 2: the components whose bound reaches the threshold M - margin, M the
// exact score of the component of sweep 1 (in cM, best in flag).  The first 16
// rows come from sweep 1 (KEPT: the same tiles) or are formed again; the second
// 16 rows are formed where any lane of the wave passes on the first 16.
// Lists: surv [F][2][32] component ids, counts (or -1) over flag.
template <int FB, bool KEPT>
__global__ void __launch_bounds__(64 * BW, 4)
k_bound_list(const _Float16* __restrict__ xh, const float2* __restrict__ tg, int64_t f0, int64_t F,
             const _Float16* __restrict__ Wf, const float2* __restrict__ cb,
             const int* __restrict__ maxbits, int npair, float margin,
             const float* __restrict__ Mf, const uint2v* __restrict__ sums,
             uint16_t* __restrict__ surv, int* __restrict__ flag, const int* __restrict__ Fdev) {
  constexpr int NP = KEPT ? CL : CL / 2;  // pairs per stage
  constexpr int PW = KEPT ? 256 : 512;    // staged operand of a pair: the second block, or both
  __shared__ __attribute__((aligned(16))) uint4 st[2][NP * PW];
  __shared__ float2 sc[2][2 * NP];
  if (Fdev && (int64_t)Fdev[0] < F) F = Fdev[0];
  constexpr int FT = 32 * BW * FB;
  const int64_t ntile = (F - f0 + FT - 1) / FT;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5, l32 = lane & 31;
  const uint4* W4 = reinterpret_cast<const uint4*>(Wf) +
                    (KEPT ? (size_t)(tid >> 8) * 512 + 256 + (tid & 255) : tid);
  const int nch = npair / NP;  // Cpad is a multiple of 256
  for (int64_t tile = blockIdx.x; tile < ntile; tile += gridDim.x) {
    const int64_t fw = f0 + tile * FT + wave * 32 * FB;
    half8 xf[FB][4];
    BoundTest bt[FB];
    int cnt[FB];
#pragma unroll
    for (int fb = 0; fb < FB; ++fb) {
      const int64_t g = min(fw + 32 * fb + l32, F - 1);
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        xf[fb][ks] = *reinterpret_cast<const half8*>(xh + g * BK + 16 * ks + 8 * h);
      bt[fb] = bound_test(tg[g], bound_scale(maxbits), Mf[g], margin, fw + 32 * fb + l32 < F, cb,
                          flag[g]);
      cnt[fb] = bt[fb].good ? 0 : SL + 1;
    }
    // stage ch in buffer b: the operands of NP pairs (512 entries per copy: two
    // pairs' second blocks, or one pair) and their constants
    auto stage = [&](int ch, int b) {
#pragma unroll
      for (int j = 0; j < NP * PW / 512; ++j)
        dma16(W4 + (size_t)ch * NP * 512 + (KEPT ? 1024 : 512) * j, &st[b][512 * j + wave * 64]);
      if (tid < 2 * NP) sc[b][tid] = cb[2 * NP * ch + tid];
    };
    const uint2v* ct = sums + (KEPT ? (size_t)tile * nch * 2 * FB * (64 * BW) + tid : 0);
    // half a stage's sums, loaded half a stage ahead
    uint2v w[2][FB];
    auto get = [&](int ch, int j) {
      if (!KEPT) return;
#pragma unroll
      for (int fb = 0; fb < FB; ++fb)
        w[j][fb] = __builtin_nontemporal_load(ct + (size_t)((2 * ch + j) * FB + fb) * (64 * BW));
    };
    static_assert(CL == 2 * CH, "two halves");
    __syncthreads();  // the previous tile's stage is consumed
    stage(0, 0);
    get(0, 0);
    dma_wait();
    __syncthreads();
#pragma unroll 1
    for (int ch = 0; ch < nch; ++ch) {
      const int b = ch & 1;
      if (ch + 1 < nch) stage(ch + 1, b ^ 1);  // last read before the previous barrier
      get(ch, 1);
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        if (i == CH) get(min(ch + 1, nch - 1), 0);
        half8 a[4];
        if (!KEPT) {
#pragma unroll
          for (int ks = 0; ks < 4; ++ks)
            a[ks] = *reinterpret_cast<const half8*>(&st[b][i * PW + ks * 64 + lane]);
        }
        const float2 cv = sc[b][2 * i + h];
        float t[FB], v[FB];
        bool pass[FB], any = false;
#pragma unroll
        for (int fb = 0; fb < FB; ++fb) {
          t[fb] = bound_limit(bt[fb], cv);
          if constexpr (KEPT) {
            v[fb] = cut_value(w[i / CH][fb][i % CH >> 1], i & 1);
          } else {
            floatx16 ac = floatx16{0};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
              ac = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[ks], xf[fb][ks], ac, 0, 0, 0);
            float sq = ac[0] * ac[0];
#pragma unroll
            for (int r = 1; r < 16; ++r) sq = fmaf(ac[r], ac[r], sq);
            v[fb] = sq * bt[fb].rn;
          }
          pass[fb] = v[fb] <= t[fb];
          any = any || pass[fb];
        }
        if (__ballot(any) == 0) continue;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
          a[ks] = *reinterpret_cast<const half8*>(&st[b][i * PW + (PW - 256) + ks * 64 + lane]);
#pragma unroll
        for (int fb = 0; fb < FB; ++fb) {
          if (__ballot(pass[fb]) == 0) continue;
          floatx16 ac = floatx16{0};
#pragma unroll
          for (int ks = 0; ks < 4; ++ks)
            ac = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[ks], xf[fb][ks], ac, 0, 0, 0);
          float sq = ac[0] * ac[0];
#pragma unroll
          for (int r = 1; r < 16; ++r) sq = fmaf(ac[r], ac[r], sq);
          if (pass[fb] && fmaf(sq, bt[fb].rn, v[fb]) <= t[fb]) {
            const int64_t g = fw + 32 * fb + l32;
            if (cnt[fb] < SL) surv[g * 64 + h * SL + cnt[fb]] = (uint16_t)(2 * (ch * NP + i) + h);
            ++cnt[fb];
          }
        }
      }
      dma_wait();
      __syncthreads();
    }
#pragma unroll
    for (int fb = 0; fb < FB; ++fb) {
      const int64_t g = fw + 32 * fb + l32;
      const int oc = __shfl_xor(cnt[fb], 32);
      if (h == 0 && g < F) flag[g] = (cnt[fb] <= SL && oc <= SL) ? (cnt[fb] | (oc << 8)) : -1;
    }
  }
}

// --------------------------------------------------------- pairs by component
// Sweep 1: one pair (frame, best) per frame.
__global__ void __launch_bounds__(256)
k_best_hist(int64_t f0, int64_t F, int fpb, int C, const int* __restrict__ best, const int* __restrict__ Fdev,
            int* __restrict__ hist) {
  extern __shared__ int hl[];
  if (Fdev && (int64_t)Fdev[0] < F) F = Fdev[0];
  for (int c = threadIdx.x; c < C; c += 256) hl[c] = 0;
  __syncthreads();
  const int64_t g0 = f0 + (int64_t)blockIdx.x * fpb, g1 = min(F, g0 + fpb);
  for (int64_t g = g0 + threadIdx.x; g < g1; g += 256) {
    const int c = best[g];
    if (c >= 0) atomicAdd(&hl[c], 1);
  }
  __syncthreads();
  for (int c = threadIdx.x; c < C; c += 256) hist[(size_t)blockIdx.x * C + c] = hl[c];
}

__global__ void __launch_bounds__(256)
k_best_scatter(int64_t f0, int64_t F, int fpb, int C, const int* __restrict__ best,
               const int* __restrict__ Fdev, const int* __restrict__ base,
               const int* __restrict__ coff, int2* __restrict__ ent) {
  extern __shared__ int cur[];
  if (Fdev && (int64_t)Fdev[0] < F) F = Fdev[0];
  for (int c = threadIdx.x; c < C; c += 256) cur[c] = coff[c] + base[(size_t)blockIdx.x * C + c];
  __syncthreads();
  const int64_t g0 = f0 + (int64_t)blockIdx.x * fpb, g1 = min(F, g0 + fpb);
  for (int64_t g = g0 + threadIdx.x; g < g1; g += 256) {
    const int c = best[g];
    if (c >= 0) ent[atomicAdd(&cur[c], 1)] = make_int2((int)g, c);
  }
}

// 16 lanes per frame, 4 list slots (8 bytes) each.
__device__ inline void list_of(int l16, int sc, int& lo, int& n) {
  const int s = 4 * l16;  // first slot of the lane
  const int cnt = s < SL ? (sc & 0xff) : (sc >> 8);
  lo = s < SL ? s : s - SL;
  n = sc < 0 ? 0 : max(0, min(4, cnt - lo));
}

__global__ void __launch_bounds__(256)
k_bound_hist(int64_t F, int fpb, int C, const uint16_t* __restrict__ surv,
             const int* __restrict__ scount, const int* __restrict__ Fdev, int* __restrict__ hist,
             int* __restrict__ cnts) {
  extern __shared__ int hl[];
  if (Fdev && (int64_t)Fdev[0] < F) F = Fdev[0];
  if (blockIdx.x == 0 && threadIdx.x < 2) cnts[threadIdx.x] = 0;
  for (int c = threadIdx.x; c < C; c += 256) hl[c] = 0;
  __syncthreads();
  const int64_t g0 = (int64_t)blockIdx.x * fpb, g1 = min(F, g0 + fpb);
  const int l16 = threadIdx.x & 15;
  for (int64_t g = g0 + (threadIdx.x >> 4); g < g1; g += 16) {
    int lo, n;
    list_of(l16, scount[g], lo, n);
    const uint16_t* p = surv + g * 64 + 4 * l16;
    for (int e = 0; e < n; ++e) atomicAdd(&hl[p[e]], 1);
  }
  __syncthreads();
  for (int c = threadIdx.x; c < C; c += 256) hist[(size_t)blockIdx.x * C + c] = hl[c];
}

// ent[pos] = (frame, component), sorted by component; the frame's candidate
// slots, running maximum (as an ordered integer) and append count are reset.
// Lists that do not fit the entry array send their frame to the dense kernel.
__global__ void __launch_bounds__(256)
k_bound_scatter(int64_t F, int fpb, int C, int2* __restrict__ cand, int* __restrict__ flag,
                const int* __restrict__ Fdev, const int* __restrict__ base,
                const int* __restrict__ coff, int64_t cap,
                int2* __restrict__ ent, int* __restrict__ cMi) {
  extern __shared__ int cur[];
  if (Fdev && (int64_t)Fdev[0] < F) F = Fdev[0];
  for (int c = threadIdx.x; c < C; c += 256) cur[c] = coff[c] + base[(size_t)blockIdx.x * C + c];
  __syncthreads();
  const int64_t g0 = (int64_t)blockIdx.x * fpb, g1 = min(F, g0 + fpb);
  const int l16 = threadIdx.x & 15;
  for (int64_t g = g0 + (threadIdx.x >> 4); g < g1; g += 16) {
    const int sc = flag[g];
    int lo, n;
    list_of(l16, sc, lo, n);
    int2* slot = cand + g * KP + l16;
    const uint2 raw = *reinterpret_cast<const uint2*>(slot);
    bool lost = false;
    for (int e = 0; e < n; ++e) {
      const int c = (int)(((e < 2 ? raw.x : raw.y) >> (16 * (e & 1))) & 0xffffu);
      const int64_t pos = atomicAdd(&cur[c], 1);
      if (pos < cap)
        ent[pos] = make_int2((int)g, c);
      else
        lost = true;
    }
    *slot = make_int2(-1, 0);
    // any lane of the frame's 16 that lost a pair
    const uint64_t bal = __ballot(lost);
    const bool any = (bal >> (threadIdx.x & 48)) & 0xffffull;
    if (l16 == 0) {
      flag[g] = (sc < 0 || any) ? kFallback : 0;
      cMi[g] = INT_MIN;
    }
  }
}

__device__ inline int ordered(float v) {
  const int i = __float_as_int(v);
  return i >= 0 ? i : i ^ 0x7fffffff;
}
__device__ inline float unordered(int i) { return __int_as_float(i >= 0 ? i : i ^ 0x7fffffff); }

// FP32 score cst_c - 1/2 ||L_c^-1 (x - mu_c)||^2 of sorted pairs on
// v_mfma_f32_32x32x2_f32: up to 32 pairs of one component at a time (columns),
// the rows of L_c^-1 as the other operand, held in registers for a run of
// pairs of the component (rows 32..63 over all columns, rows 0..31 over
// columns 0..31: 46 MFMAs).  First pass (score null): the frame's M.  Second
// pass: the pair's score, and the frame's maximum as an ordered integer.
// mu_c is taken in two FP32 parts: rounded to one, features far from the origin
// (1e6 at unit deviations) would move a score by hundreds of nats.
// A wave takes a contiguous range and loads the rows of the next run while it
// scores this one; the ranges fill the device once (2 workgroups per CU).  4 M
// frames, 20 M pairs: 0.9 ms on average for the two passes, near the FP32 MFMA
// time; 3.8 ms when each run's rows were loaded, under guards, after the run
// was known, and 9.4 ms with a pair per lane and L_c^-1 through the scalar cache.
template <bool V4>  // rows of X in whole float4
__global__ void __launch_bounds__(256, 2)
k_bound_quad(const float* __restrict__ X, int D, const int* __restrict__ coff, int C,
             const int2* __restrict__ ent, int64_t cap, const double* __restrict__ mu,
             const float* __restrict__ lquad, const double* __restrict__ cst,
             float* __restrict__ score, float* __restrict__ Mf) {
  const int lane = threadIdx.x & 63, h = lane >> 5, l32 = lane & 31;
  const int64_t total = min((int64_t)coff[C], cap);
  const int64_t nw = (int64_t)gridDim.x * 4;
  const int64_t per = max<int64_t>(8, (total + nw - 1) / nw);
  int64_t e0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * per;
  const int64_t b1 = min(total, e0 + per);
  if (e0 >= b1) return;
  int cur = -1;
  float4 a1[8], a0[4];  // rows l32 + 32 and l32, columns 4 (2 s + h) .. + 3
  __shared__ float4 ms[4][2][16];  // mu_c of the wave, high and low parts
  const int wave = threadIdx.x >> 6;
  float cc = 0.0f;
  const float4 z4 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  // a row's columns 4 (2 s + h) + e; beyond D any value of the row, L_c^-1 is
  // zero there
  auto row = [&](int g, float4* x) {
    const float* xp = X + (int64_t)g * D;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int k = 4 * (2 * s + h);
      if (V4)
        x[s] = *reinterpret_cast<const float4*>(xp + min(k, D - 4));
      else
        x[s] = make_float4(xp[min(k, D - 1)], xp[min(k + 1, D - 1)], xp[min(k + 2, D - 1)],
                           xp[min(k + 3, D - 1)]);
    }
  };
  // the 64 entries from e0 are at hand, so the rows of the next run of pairs
  // are loaded while this one is scored
  int2 win = ent[min(e0 + lane, b1 - 1)];
  float4 x[8], xn[8];
  row(__shfl(win.x, l32), x);
  while (true) {
    const int c = __builtin_amdgcn_readfirstlane(win.y);
    const uint64_t same = __ballot(win.y == c && e0 + lane < b1);
    const int n = min(32, (int)__popcll(same));  // sorted: a run from e0
    const int g = __shfl(win.x, l32);
    const bool more = e0 + n < b1;
    if (more) {
      row(__shfl(win.x, n + l32), xn);
      win = ent[min(e0 + n + lane, b1 - 1)];
    }
    {
      if (c != cur) {
        cur = c;
        const float4* Lq = reinterpret_cast<const float4*>(lquad) + (size_t)c * 1024 + l32;
#pragma unroll
        for (int s = 0; s < 8; ++s) a1[s] = Lq[(2 * s + h) * 64 + 32];
#pragma unroll
        for (int s = 0; s < 4; ++s) a0[s] = Lq[(2 * s + h) * 64];
        const double m = mu[(size_t)c * D + min(lane, D - 1)];
        float* mw = reinterpret_cast<float*>(ms[wave]) + lane;
        mw[0] = (float)m;
        mw[64] = (float)(m - (double)(float)m);
        __builtin_amdgcn_wave_barrier();
        cc = (float)cst[c];
      }
      float4 d[8];
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const float4 m = ms[wave][0][2 * s + h], l = ms[wave][1][2 * s + h];
        d[s] = make_float4((x[s].x - m.x) - l.x, (x[s].y - m.y) - l.y, (x[s].z - m.z) - l.z,
                           (x[s].w - m.w) - l.w);
      }
      floatx16 y1 = floatx16{0}, y0 = floatx16{0};
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const float4 p = s < 4 ? a0[s < 4 ? s : 0] : z4;
        y1 = __builtin_amdgcn_mfma_f32_32x32x2f32(a1[s].x, d[s].x, y1, 0, 0, 0);
        if (s < 4) y0 = __builtin_amdgcn_mfma_f32_32x32x2f32(p.x, d[s].x, y0, 0, 0, 0);
        y1 = __builtin_amdgcn_mfma_f32_32x32x2f32(a1[s].y, d[s].y, y1, 0, 0, 0);
        if (s < 4) y0 = __builtin_amdgcn_mfma_f32_32x32x2f32(p.y, d[s].y, y0, 0, 0, 0);
        y1 = __builtin_amdgcn_mfma_f32_32x32x2f32(a1[s].z, d[s].z, y1, 0, 0, 0);
        if (s < 4) y0 = __builtin_amdgcn_mfma_f32_32x32x2f32(p.z, d[s].z, y0, 0, 0, 0);
        y1 = __builtin_amdgcn_mfma_f32_32x32x2f32(a1[s].w, d[s].w, y1, 0, 0, 0);
        if (s < 4) y0 = __builtin_amdgcn_mfma_f32_32x32x2f32(p.w, d[s].w, y0, 0, 0, 0);
      }
      float q = 0.0f;
#pragma unroll
      for (int r = 0; r < 16; ++r) q = fmaf(y1[r], y1[r], fmaf(y0[r], y0[r], q));
      q += __shfl_xor(q, 32);
      if (h == 0 && l32 < n) {
        const float sv = cc - 0.5f * q;
        if (score) {
          score[e0 + l32] = sv;
          atomicMax(reinterpret_cast<int*>(Mf) + g, ordered(sv));
        } else {
          Mf[g] = sv;
        }
      }
    }
    if (!more) break;
    e0 += n;
#pragma unroll
    for (int s = 0; s < 8; ++s) x[s] = xn[s];
  }
}

// Appends candidate (c, v) to frame g's list (any order; k_bound_final sorts)
__device__ inline void append_cand(int2* cand, int* flag, int g, int c, float v) {
  const int s = atomicAdd(flag + g, 1) & (kReplay - 1);
  if (s < KP) cand[(int64_t)g * KP + s] = make_int2(c, __float_as_int(v));
}

// Which pairs are candidates is the dense kernel's decision, taken from its
// own scores; those differ from the FP32 scores here by less than half of
// `err` nats (and a few parts in 10^6 of their size).  A pair further than that
// inside or outside the margin is decided either way; frames with a pair closer
// than that are marked for the replay.
__device__ inline float pair_err(float err, float M) { return err + kRelErr * fabsf(M); }

__global__ void __launch_bounds__(256)
k_bound_mark(const int* __restrict__ coff, int C, const int2* __restrict__ ent, int64_t cap,
             const float* __restrict__ score, const int* __restrict__ cMi, float margin, float err,
             int* __restrict__ flag) {
  const int64_t total = min((int64_t)coff[C], cap);
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * 256) {
    const int g = ent[e].x;
    const float M = unordered(cMi[g]), d = score[e] - (M - margin);
    if (fabsf(d) <= pair_err(err, M)) atomicOr(flag + g, kReplay);
  }
}

// Candidates of the decided frames; the pairs to replay go to a list, the pairs
// of a component still together.  One addition to the list's length per 2048
// pairs: one per wave was bound by it (20 M pairs, 2.0 ms; now 0.51 ms).
__global__ void __launch_bounds__(256)
k_bound_append(const int* __restrict__ coff, int C, const int2* __restrict__ ent, int64_t cap,
               const float* __restrict__ score, const int* __restrict__ cMi, float margin,
               float err, int2* __restrict__ cand, int* __restrict__ flag, int* __restrict__ nrep,
               int* __restrict__ rep) {
  constexpr int N = 2048;  // pairs per workgroup and addition
  __shared__ int list[N];
  __shared__ int cnt, at;
  const int64_t total = min((int64_t)coff[C], cap);
  for (int64_t e0 = (int64_t)blockIdx.x * N; e0 < total; e0 += (int64_t)gridDim.x * N) {
    if (threadIdx.x == 0) cnt = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; i += 256) {
      const int64_t e = e0 + i + threadIdx.x;
      if (e >= total) break;
      const int2 p = ent[e];
      const float s = score[e], M = unordered(cMi[p.x]);
      if (!(s >= M - margin - pair_err(err, M))) continue;
      const int f = flag[p.x];
      if (f >= kFallback) continue;
      if (f & kReplay)
        list[atomicAdd(&cnt, 1)] = (int)e;
      else
        append_cand(cand, flag, p.x, p.y, s);
    }
    __syncthreads();
    if (threadIdx.x == 0 && cnt > 0) at = atomicAdd(nrep, cnt);
    __syncthreads();
    for (int i = threadIdx.x; i < cnt; i += 256) rep[at + i] = list[i];
    __syncthreads();
  }
}

// The dense kernel's scores of the listed pairs.  FP32: v_mfma_f32_32x32x2_f32
// adds its two products one after the other with fused multiply-adds, so the
// scalar chain over the same products in the same order (features k, k + 4 of
// a chunk of 8 alternating) gives the same bits; one pair per lane.  BF16: the
// same MFMA sequence with the pair's component in row i and its frame in
// column i; the diagonal is the score.
template <bool BF>
__global__ void __launch_bounds__(64)
k_bound_replay(const float* __restrict__ X, int D, const float* __restrict__ shift, int Cpad,
               int Kpad, const int2* __restrict__ ent, const int* __restrict__ nrep,
               const int* __restrict__ rep, const uint16_t* __restrict__ pairs,
               const float* __restrict__ W, const __bf16* __restrict__ W16,
               int2* __restrict__ cand, int* __restrict__ flag) {
  constexpr int NP = BF ? 32 : 64;  // pairs per wave
  extern __shared__ float xs[];     // [D + 1][NP]
  const int lane = threadIdx.x;
  const int total = nrep[0];
  for (int e0 = blockIdx.x * NP; e0 < total; e0 += gridDim.x * NP) {
    const int li = BF ? (lane & 31) : lane, h = lane >> 5;
    const bool valid = e0 + li < total;
    const int2 en = ent[rep[valid ? e0 + li : e0]];
    __syncthreads();  // one wave; the previous pass's reads are done
    for (int k = BF ? h : 0; k <= D; k += BF ? 2 : 1)
      xs[k * NP + li] = k == 0 ? 1.0f : X[(int64_t)en.x * D + k - 1] - shift[k - 1];
    __syncthreads();
    const float* xf = xs + li;
    float my = 0.0f;
    if constexpr (!BF) {
      const float4* w = reinterpret_cast<const float4*>(W + (size_t)en.y * 8);
      const uint4* pr = reinterpret_cast<const uint4*>(pairs);
      const int nq = Kpad / 8;
      float4 wa = w[0], wb = w[1];
      uint4 pw = pr[0];
      for (int q = 0; q < nq; ++q) {
        float4 na = wa, nb = wb;
        uint4 np = pw;
        if (q + 1 < nq) {
          na = w[(size_t)(q + 1) * Cpad * 2];
          nb = w[(size_t)(q + 1) * Cpad * 2 + 1];
          np = pr[q + 1];
        }
        float x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const uint32_t p = (k < 2 ? pw.x : k < 4 ? pw.y : k < 6 ? pw.z : pw.w) >> (16 * (k & 1));
          x[k] = xf[(p & 0xff) * NP] * xf[((p >> 8) & 0xff) * NP];
        }
        my = fmaf(wa.x, x[0], my);
        my = fmaf(wb.x, x[4], my);
        my = fmaf(wa.y, x[1], my);
        my = fmaf(wb.y, x[5], my);
        my = fmaf(wa.z, x[2], my);
        my = fmaf(wb.z, x[6], my);
        my = fmaf(wa.w, x[3], my);
        my = fmaf(wb.w, x[7], my);
        wa = na;
        wb = nb;
        pw = np;
      }
      if (valid) append_cand(cand, flag, en.x, en.y, my);
    } else {
      floatx16 acc = floatx16{0};
      for (int q = 0; q < Kpad / 16; ++q) {
        const __bf16* w = W16 + ((size_t)q * Cpad + en.y) * 32 + 8 * h;
        const bf16x8 wh = *reinterpret_cast<const bf16x8*>(w);
        const bf16x8 wl = *reinterpret_cast<const bf16x8*>(w + 16);
        const uint4 pw = *reinterpret_cast<const uint4*>(pairs + 16 * q + 8 * h);
        bf16x8 bh, bl;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const uint32_t w32 = (e < 2) ? pw.x : (e < 4) ? pw.y : (e < 6) ? pw.z : pw.w;
          const uint32_t pr = w32 >> ((e & 1) * 16);
          const float v = xf[(pr & 0xff) * NP] * xf[((pr >> 8) & 0xff) * NP];
          const __bf16 hi = (__bf16)v;
          bh[e] = hi;
          bl[e] = (__bf16)(v - (float)hi);
        }
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wh, bh, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wh, bl, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wl, bh, acc, 0, 0, 0);
      }
      // diagonal (i, i): register 4 (i / 8) + i % 4 of the lanes with h = (i / 4) % 2
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (r == 4 * (li >> 3) + (li & 3)) my = acc[r];
      if (valid && h == ((li >> 2) & 1)) append_cand(cand, flag, en.x, en.y, my);
    }
  }
}

// The frame's list in the dense kernel's order (components with bit 2 clear,
// ascending, then the others), its maximum, and the overflow flag: more than
// 8 candidates of one half within the margin, or more than KP appended.
// Frames for the dense kernel are listed in fb.  16 lanes per frame.
__global__ void __launch_bounds__(256)
k_bound_final(int64_t F, float margin, int2* __restrict__ cand, int* __restrict__ flag,
              float* __restrict__ cM, const int* __restrict__ Fdev, int* __restrict__ nfb,
              int* __restrict__ fb) {
  if (Fdev && (int64_t)Fdev[0] < F) F = Fdev[0];
  const int l16 = threadIdx.x & 15;
  const int64_t g = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
  if (g >= F) return;  // uniform over the 16 lanes of a frame
  const int fl = flag[g], n = fl & (kReplay - 1);
  if (fl >= kFallback) {
    if (l16 == 0) fb[atomicAdd(nfb, 1)] = (int)g;
    return;
  }
  const int2 e = cand[g * KP + l16];
  const float v = e.x >= 0 ? __int_as_float(e.y) : -INFINITY;
  float M = v;
#pragma unroll
  for (int o = 8; o >= 1; o >>= 1) M = fmaxf(M, __shfl_xor(M, o, 16));
  const bool in = e.x >= 0 && v >= M - margin;
  const uint64_t sh = threadIdx.x & 48;
  const int lowk = __popcll((__ballot(in && !(e.x & 4)) >> sh) & 0xffffull);
  const int high = __popcll((__ballot(in && (e.x & 4)) >> sh) & 0xffffull);
  const int key = e.x < 0 ? INT_MAX : (e.x & 4) ? e.x | (1 << 24) : e.x;
  int rank = 0;
#pragma unroll
  for (int o = 0; o < 16; ++o) {
    const int k = __shfl(key, o, 16);
    rank += k < key || (k == key && o < l16);
  }
  cand[g * KP + rank] = e;
  if (l16 == 0) {
    cM[g] = M;
    flag[g] = (n > KP || n == 0 || lowk > KP / 2 || high > KP / 2) ? 1 : 0;
  }
}

size_t dirs_lds(int D) { return sizeof(double) * ((size_t)D * D + 2 * (size_t)D * BR + BR * BR + BR); }

}  // namespace

int64_t bound_sweep_frames(int Cpad, int64_t maxF) {
  const int64_t n = (int64_t(1) << 30) / Cpad / 512 * 512;
  return n < (int64_t(1) << 17) ? 0 : std::min<int64_t>(n, (maxF + 511) / 512 * 512);
}

// The bound needs D + 2 <= 64 columns and at least 32 dimensions for its rows,
// 16-bit component ids, and enough components that its 20 launches and the sorts
// pay beside the sweeps: 36,000 frames at C = 512 take 403 us against 467 by a dense
// shape at D = 32 and 469 against 1228 at D = 60 (C = 2048: 830 and 1492, 967 and 4547).
bool bound_supported(int C, int D) { return D >= BR && D + 2 <= BK && C >= 512 && C <= 65536; }

bool bound_set_attributes(const ivx_ctx* ctx) {
  if (!ctx->Wf) return true;
  auto set = [](const void* fn, size_t bytes) {
    return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) ==
           hipSuccess;
  };
  return set(reinterpret_cast<const void*>(&k_bound_dirs), dirs_lds(62));
}

// cov_changed: the directions depend on the covariances alone
void launch_bound_prepare(ivx_ctx* ctx, bool cov_changed, hipStream_t s) {
  if (!ctx->Wf) return;
  const int C = ctx->C, D = ctx->D;
  if (cov_changed) {
    k_bound_dirs<<<C, 256, dirs_lds(D), s>>>(ctx->linv, ctx->cst, D, ctx->Wd);
    k_linv_quads<<<2048, 256, 0, s>>>(ctx->linv, C, D, ctx->lquad);
  }
  k_bound_spread<<<(C + 3) / 4, 256, 0, s>>>(ctx->w, ctx->mu, ctx->cov, ctx->cst, ctx->shift, C, D,
                                             ctx->bspread);
  k_bound_scale<<<(C + 3) / 4, 256, 0, s>>>(ctx->Wd, ctx->mu, ctx->cst, ctx->shift, ctx->bspread, C,
                                            D, ctx->wmu, ctx->bnorm, ctx->bmax, ctx->bunit);
  k_bound_pack<<<ctx->Cpad / 2, 256, 0, s>>>(ctx->Wd, ctx->wmu, ctx->bnorm, ctx->cst, C, ctx->Cpad,
                                             D, ctx->bmax, ctx->bunit, ctx->Wf, ctx->cb);
}

void launch_bound_select(ivx_ctx* ctx, const float* X, int64_t F, int prec, hipStream_t s,
                         const int* Fdev, int** fb_count, int** fb_list, int** rest) {
  const bool bf = prec == IVX_BF16;
  const float margin = bf ? ctx->margin_bf16 : ctx->margin;
  // the FP32 dense scores are off by up to 0.4 nats on the workload, the BF16
  // split-form ones by up to ~3
  const float err = bf ? 8.0f : 3.0f;
  // workspace, all in arrays that the rescoring writes later: the FP16 frames
  // in ent, replaced there by the sorted pairs of sweep 2 (at most 14 F); the
  // pairs of sweep 1 and (t^2, g) in lscore, replaced by the pairs' scores,
  // two counters, the dense kernel's frames and the pairs to replay; the
  // sample's decision behind them
  const int64_t cap = kListed * F;
  _Float16* xh = reinterpret_cast<_Float16*>(ctx->ent);
  char* w8 = reinterpret_cast<char*>(ctx->lscore);
  int2* ent1 = reinterpret_cast<int2*>(w8);
  float2* tg = reinterpret_cast<float2*>(w8 + 8 * F);
  float* score = reinterpret_cast<float*>(w8);
  int* cnts = reinterpret_cast<int*>(w8 + 56 * F);
  int* fb = cnts + 2;
  int* rep = fb + F;
  int* dec = reinterpret_cast<int*>(w8 + 120 * F);  // 5 ints; rep ends at 116 F + 8
  static_assert(56 + 4 + 4 * kListed <= 116, "workspace layout");
  static_assert(KP == 16 && sizeof(int2) * KP == 2 * BK, "workspace layout");
  uint16_t* surv = reinterpret_cast<uint16_t*>(ctx->cand);
  int* cMi = reinterpret_cast<int*>(ctx->cM);
  const int fpb = hist_frames(F, ctx->nhist);
  const unsigned nb = (unsigned)((F + fpb - 1) / fpb);
  const size_t ldsc = sizeof(int) * ctx->C;
  const unsigned n16 = (unsigned)((F + 15) / 16);
  const unsigned nq = (unsigned)std::min<int64_t>((F + 31) / 32, 2 * (int64_t)ctx->ncu);
  const unsigned ne = (unsigned)std::min<int64_t>((F + 63) / 64, 8 * (int64_t)ctx->ncu);
  ProfScope ps(ctx, PK_FRAME_SELECT, s);
  k_bound_frames<<<n16, 256, 0, s>>>(X, F, ctx->D, ctx->shift, ctx->bunit, Fdev, xh, tg);
  // the sample's sums, in the candidate or the score buffer (both written later)
  const float k60 = 1891.0f / (float)ctx->K;
  const SampleRule rule = {k60 * (bf ? 0.5f : 0.2f), k60 * (bf ? 5.5e-6f : 2.6e-6f),
                           bf ? 1.5f : 1.85f, 128 * ctx->ncu, (int)scores_frames(ctx)};
  const int64_t room = std::max<int64_t>(128 * F, (int64_t)ctx->scores_bytes);
  float2* sv = 128 * F >= (int64_t)ctx->scores_bytes ? reinterpret_cast<float2*>(ctx->cand)
                                                      : reinterpret_cast<float2*>(ctx->scores);
  const int ns = (int)std::min<int64_t>(kSample, room / (8 * ctx->Cpad) / 32 * 32);
  *rest = nullptr;
  if (ns > 0) {
    k_sample_sums<<<ctx->Cpad / (2 * SP), 256, 0, s>>>(xh, tg, F, ctx->Wf, ctx->bmax, ctx->Cpad, ns,
                                                       sv, dec, Fdev);
    k_sample_count<<<ns, 256, 0, s>>>(X, F, ctx->D, tg, ctx->cb, ctx->bmax, ctx->Cpad,
                                     margin + err - 3.0f, ctx->mu, ctx->lquad, ctx->cst, sv,
                                     rule, dec, Fdev);
    Fdev = dec;
    *rest = dec + 1;
  }
  const bool v4 = ctx->D % 4 == 0 && reinterpret_cast<uintptr_t>(X) % 16 == 0;
  // the sweeps over as many frames as their sums have room for, in equal parts;
  // without sums, all frames at once
  uint2v* sums = reinterpret_cast<uint2v*>(ctx->sums16);
  const int64_t parts = sums ? (F + ctx->sweep_frames - 1) / ctx->sweep_frames : 1;
  const int64_t step = ((F + parts - 1) / parts + 511) / 512 * 512;
  for (int64_t f0 = 0; f0 < F; f0 += step) {
    const int64_t f1 = std::min(F, f0 + step), n = f1 - f0;
    // frames per tile: 256 FB; two blocks per wave halve the LDS reads per MFMA,
    // one fills the device with half the frames
    const int64_t slots = 2 * (int64_t)ctx->ncu;
    const int64_t t2 = (n + 511) / 512, t1 = (n + 255) / 256;
    const bool two =
        2.0 * (double)((t2 + slots - 1) / slots) <= 1.3 * (double)((t1 + slots - 1) / slots);
    const unsigned nblk = (unsigned)std::min<int64_t>(two ? t2 : t1, slots);
    const int fpp = hist_frames(n, ctx->nhist);
    const unsigned np = (unsigned)((n + fpp - 1) / fpp);
    auto* best = !sums ? (two ? &k_bound_best<2, false> : &k_bound_best<1, false>)
                       : (two ? &k_bound_best<2, true> : &k_bound_best<1, true>);
    best<<<nblk, 64 * BW, 0, s>>>(
        xh, tg, f0, f1, ctx->Wf, ctx->cb, ctx->bmax, ctx->Cpad / 2, ctx->cflag, sums, Fdev);
    k_best_hist<<<np, 256, ldsc, s>>>(f0, f1, fpp, ctx->C, ctx->cflag, Fdev, ctx->hist);
    launch_hist_scan((int)np, ctx->C, ctx->hist, ctx->coff, s);
    k_best_scatter<<<np, 256, ldsc, s>>>(f0, f1, fpp, ctx->C, ctx->cflag, Fdev, ctx->hist,
                                         ctx->coff, ent1);
    const unsigned nq1 = (unsigned)std::min<int64_t>((n + 31) / 32, 2 * (int64_t)ctx->ncu);
    (v4 ? k_bound_quad<true> : k_bound_quad<false>)<<<nq1, 256, 0, s>>>(
        X, ctx->D, ctx->coff, ctx->C, ent1, n, ctx->mu, ctx->lquad, ctx->cst, nullptr, ctx->cM);
    auto* list = !sums ? (two ? &k_bound_list<2, false> : &k_bound_list<1, false>)
                       : (two ? &k_bound_list<2, true> : &k_bound_list<1, true>);
    list<<<nblk, 64 * BW, 0, s>>>(
        xh, tg, f0, f1, ctx->Wf, ctx->cb, ctx->bmax, ctx->Cpad / 2, margin + err - 3.0f, ctx->cM,
        sums, surv, ctx->cflag, Fdev);
  }
  k_bound_hist<<<nb, 256, ldsc, s>>>(F, fpb, ctx->C, surv, ctx->cflag, Fdev, ctx->hist, cnts);
  launch_hist_scan((int)nb, ctx->C, ctx->hist, ctx->coff, s);
  k_bound_scatter<<<nb, 256, ldsc, s>>>(F, fpb, ctx->C, ctx->cand, ctx->cflag, Fdev, ctx->hist,
                                        ctx->coff, cap, ctx->ent, cMi);
  (v4 ? k_bound_quad<true> : k_bound_quad<false>)<<<nq, 256, 0, s>>>(
      X, ctx->D, ctx->coff, ctx->C, ctx->ent, cap, ctx->mu, ctx->lquad, ctx->cst, score, ctx->cM);
  k_bound_mark<<<ne, 256, 0, s>>>(ctx->coff, ctx->C, ctx->ent, cap, score, cMi, margin, err,
                                  ctx->cflag);
  k_bound_append<<<ne, 256, 0, s>>>(ctx->coff, ctx->C, ctx->ent, cap, score, cMi, margin, err,
                                    ctx->cand, ctx->cflag, cnts + 1, rep);
  const unsigned nr = (unsigned)std::min<int64_t>((F + 31) / 32, 16 * (int64_t)ctx->ncu);
  const size_t lr = sizeof(float) * (bf ? 32 : 64) * (size_t)(ctx->D + 1);
  (bf ? k_bound_replay<true> : k_bound_replay<false>)<<<nr, 64, lr, s>>>(
      X, ctx->D, ctx->shift, ctx->Cpad, ctx->Kpad, ctx->ent, cnts + 1, rep, ctx->pairs, ctx->Wexp,
      ctx->W16, ctx->cand, ctx->cflag);
  k_bound_final<<<n16, 256, 0, s>>>(F, margin, ctx->cand, ctx->cflag, ctx->cM, Fdev, cnts, fb);
  *fb_count = cnts;
  *fb_list = fb;
}

}  // namespace ivx
