// Scoring back-end of Sec. 4.1 on the GPU: centring / whitening / length
// normalisation, class scatter, LDA, two-covariance PLDA and trial scoring.
//
//  k_class_sums      per-class sums and counts (FP64 atomics)
//  gemm64_tn         second moment X^T X (FP64 MFMA, k_gemm64.hip)
//  k_scatter         Sw, Sb (divisor N) from the second moment and class sums
//  k_jacobi_step     symmetric eigendecomposition by cyclic Jacobi with
//                    round-robin ordering: n/2 disjoint rotations per step, one
//                    kernel per step (one workgroup per pair); the host checks the off-diagonal norm
//                    after every sweep
//  k_dgemm           small FP64 products (n <= 512) through LDS tiles
//  k_lnorm, k_lnorm_white  y = W (x - mean) scaled to unit length
//  k_plda_score, k_plda_matrix  llr of (z1, z2) in the space where W = I and
//                    B = diag(psi), trial by trial or for all pairs
#include <algorithm>
#include <cmath>

#include "ivx_backend.h"

namespace ivx {
namespace {

__global__ void __launch_bounds__(256)
k_class_sums(const float* __restrict__ X, int64_t n, int dim, const int* __restrict__ labels,
             int K, double* __restrict__ sums, double* __restrict__ counts,
             int* __restrict__ bad) {
  const int64_t i = blockIdx.x;
  if (i >= n) return;
  const int k = labels ? labels[i] : 0;
  if (k < 0 || k >= K) {
    if (threadIdx.x == 0) atomicAdd(bad, 1);
    return;
  }
  for (int d = threadIdx.x; d < dim; d += blockDim.x)
    atomicAdd(&sums[(size_t)k * dim + d], (double)X[i * dim + d]);
  if (threadIdx.x == 0) atomicAdd(&counts[k], 1.0);
}

// Sw = (M2 - G) / N, Sb = (G - N m m^T) / N with G = sum_k s_k s_k^T / n_k and
// m = sum_k s_k / N (classes without members contribute nothing).
__global__ void __launch_bounds__(256)
k_scatter(const double* __restrict__ M2, const double* __restrict__ sums,
          const double* __restrict__ counts, int K, int dim, double* __restrict__ Sw,
          double* __restrict__ Sb, double* __restrict__ mean) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= (int64_t)dim * dim) return;
  const int i = (int)(e / dim), j = (int)(e - (int64_t)i * dim);
  double G = 0.0, si = 0.0, sj = 0.0, N = 0.0;
  for (int k = 0; k < K; ++k) {
    const double nk = counts[k];
    if (nk <= 0.0) continue;
    const double a = sums[(size_t)k * dim + i], b = sums[(size_t)k * dim + j];
    G += a * b / nk;
    si += a;
    sj += b;
    N += nk;
  }
  const double mi = si / N, mj = sj / N;
  Sw[e] = (M2[e] - G) / N;
  Sb[e] = (G - N * mi * mj) / N;
  if (i == j && mean) mean[i] = mi;
}

// Round-robin pairing of n (even) indices, step r in [0, n-1): pair 0 is
// (n-1, r); pair k >= 1 is ((r + k) mod (n-1), (r - k) mod (n-1)).
__device__ inline void rr_pair(int n, int r, int k, int& p, int& q) {
  const int m = n - 1;
  if (k == 0) {
    p = r;
    q = m;
  } else {
    p = (r + k) % m;
    q = (r - k + m) % m;
  }
  if (p > q) {
    const int t = p;
    p = q;
    q = t;
  }
}

// Cyclic Jacobi on the symmetric A [n][n] (n even): the n/2 disjoint pairs of
// round-robin step r rotate at once, A <- J^T A J, V <- V J.  One launch does
// the column rotations of step r0 (rot0; none if r0 < 0) and the row rotations
// of step r1 (written to rot1; none if r1 < 0).  A workgroup owns the rows p, q
// of a pair of step r1: the column rotations act inside a row, the pair's own
// rotation comes from the 2 x 2 block inside its two rows, and so does the row
// rotation, so a step needs no other exchange than the rotations of the one
// before.  A step is bound by its latency (launch, one round of loads, the
// rotation): 4.3 us at n = 400, and 6.6 us as two kernels, rows then columns.
// The products are rounded as they were there (a rotation sequence that differs
// in the last bit ends in other signs and another order).
__global__ void __launch_bounds__(256)
k_jacobi_step(double* __restrict__ A, double* __restrict__ V, int n, int r0,
              const double2* __restrict__ rot0, int r1, double2* __restrict__ rot1) {
  __shared__ double row[2][512];
  __shared__ double s_c, s_s;
  const int k = threadIdx.x;  // column pair of step r0
  int p, q;
  rr_pair(n, r1 < 0 ? 0 : r1, blockIdx.x, p, q);
  if (k < n / 2) {
    int cp, cq;
    rr_pair(n, r0 < 0 ? 0 : r0, k, cp, cq);
    const double2 cs = r0 < 0 ? make_double2(1.0, 0.0) : rot0[k];
    double a[2][2], v[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const size_t o = (size_t)(i ? q : p) * n;
      a[i][0] = A[o + cp];
      a[i][1] = A[o + cq];
      v[i][0] = V[o + cp];
      v[i][1] = V[o + cq];
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if (cs.y == 0.0) {
        row[i][cp] = a[i][0];
        row[i][cq] = a[i][1];
      } else {
        const double ap = a[i][0], aq = a[i][1];
        row[i][cp] = cs.x * ap - cs.y * aq;
        row[i][cq] = cs.y * ap + cs.x * aq;
        const double vp = v[i][0], vq = v[i][1];
        const size_t o = (size_t)(i ? q : p) * n;
        V[o + cp] = cs.x * vp - cs.y * vq;
        V[o + cq] = cs.y * vp + cs.x * vq;
      }
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const double apq = row[0][q];
    double c = 1.0, t = 0.0;
    if (r1 >= 0 && apq != 0.0) {
      const double theta = (row[1][q] - row[0][p]) / (2.0 * apq);
      t = (theta >= 0.0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
      c = 1.0 / sqrt(t * t + 1.0);
    }
    s_c = c;
    s_s = t * c;
    if (r1 >= 0) rot1[blockIdx.x] = make_double2(c, t * c);
  }
  __syncthreads();
  const double c = s_c, sv = s_s;
  for (int j = threadIdx.x; j < n; j += 256) {
    const double ap = row[0][j], aq = row[1][j];
    A[(size_t)p * n + j] = sv == 0.0 ? ap : c * ap - sv * aq;
    A[(size_t)q * n + j] = sv == 0.0 ? aq : sv * ap + c * aq;
  }
}

// part[b] = partial sums of the squared off-diagonal (and, with diag, all)
// entries of A [n][n]; one value per workgroup, two slots per workgroup.
__global__ void __launch_bounds__(256)
k_offnorm_part(const double* __restrict__ A, int n, double* __restrict__ part) {
  __shared__ double r0[256], r1[256];
  double off = 0.0, all = 0.0;
  for (int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x; e < (int64_t)n * n;
       e += (int64_t)gridDim.x * 256) {
    const double v = A[e] * A[e];
    all += v;
    if (e / n != e % n) off += v;
  }
  r0[threadIdx.x] = off;
  r1[threadIdx.x] = all;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) {
      r0[threadIdx.x] += r0[threadIdx.x + o];
      r1[threadIdx.x] += r1[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = r0[0];
    part[2 * blockIdx.x + 1] = r1[0];
  }
}

__global__ void k_eye_diag(double* __restrict__ V, int n, const double* __restrict__ A,
                           double* __restrict__ w, int mode) {
  for (int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x; e < (int64_t)n * n;
       e += (int64_t)gridDim.x * 256) {
    if (mode == 0)
      V[e] = (e / n == e % n) ? 1.0 : 0.0;
    else if (e < n)
      w[e] = A[e * n + e];
  }
}

// C[M][N] = sum_k op(A)[m][k] op(B)[k][n] - colsub[n], FP64 sums, 16 x 16 tiles.
// op(A)[m][k] = A[m*lda + k] (ta = 0) or A[k*lda + m] (ta = 1); same for B.
template <typename TA>
__global__ void __launch_bounds__(256)
k_dgemm(const TA* __restrict__ A, int64_t lda, int ta, const double* __restrict__ B, int64_t ldb,
        int tb, void* __restrict__ Cv, int64_t ldc, int c_float, int M, int N, int K,
        const double* __restrict__ colsub) {
  __shared__ double As[16][17], Bs[16][17];
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const int64_t m = (int64_t)blockIdx.y * 16 + ty;
  const int nn = blockIdx.x * 16 + tx;
  double acc = 0.0;
  for (int k0 = 0; k0 < K; k0 += 16) {
    {
      const int64_t mm = (int64_t)blockIdx.y * 16 + ty;
      const int kk = k0 + tx;
      double v = 0.0;
      if (mm < M && kk < K) v = (double)(ta ? A[(int64_t)kk * lda + mm] : A[mm * lda + kk]);
      As[ty][tx] = v;
      const int kb = k0 + ty, nb = blockIdx.x * 16 + tx;
      double u = 0.0;
      if (kb < K && nb < N) u = tb ? B[(int64_t)nb * ldb + kb] : B[(int64_t)kb * ldb + nb];
      Bs[ty][tx] = u;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) acc += As[ty][k] * Bs[k][tx];
    __syncthreads();
  }
  if (m < M && nn < N) {
    if (colsub) acc -= colsub[nn];
    if (c_float)
      static_cast<float*>(Cv)[m * ldc + nn] = (float)acc;
    else
      static_cast<double*>(Cv)[m * ldc + nn] = acc;
  }
}

// Wh[:, j] = Q[:, j] / sqrt(lam_j) for the columns j < dim of Q [ld][ld]
// (trans: stored transposed, Wh[j][i]); an eigenvalue <= floor * max makes
// the matrix singular: flagged.
__global__ void __launch_bounds__(256)
k_whiten_cols(const double* __restrict__ Q, int ld, const double* __restrict__ lam, int dim,
              double floor_rel, int trans, double* __restrict__ Wh, int* __restrict__ bad) {
  __shared__ double s_max;
  if (threadIdx.x == 0) {
    double mx = 0.0;
    for (int j = 0; j < dim; ++j) mx = fmax(mx, lam[j]);
    s_max = mx;
  }
  __syncthreads();
  for (int64_t e = blockIdx.x * 256 + threadIdx.x; e < (int64_t)dim * dim;
       e += (int64_t)gridDim.x * 256) {
    const int i = (int)(e / dim), j = (int)(e - (int64_t)i * dim);
    const double l = lam[j];
    const int64_t o = trans ? (int64_t)j * dim + i : e;
    if (!(l > floor_rel * s_max)) {
      if (i == 0) atomicAdd(bad, 1);
      Wh[o] = 0.0;
    } else {
      Wh[o] = Q[(size_t)i * ld + j] / sqrt(l);
    }
  }
}

// Ranks of w [n] in decreasing order (ties: lower index first); idx[rank] = i
// for the first `keep` ranks, among the first `valid` entries only.
__global__ void __launch_bounds__(256)
k_rank_desc(const double* __restrict__ w, int valid, int keep, int* __restrict__ idx) {
  for (int i = blockIdx.x * 256 + threadIdx.x; i < valid; i += gridDim.x * 256) {
    const double v = w[i];
    int r = 0;
    for (int j = 0; j < valid; ++j) r += (w[j] > v) || (w[j] == v && j < i);
    if (r < keep) idx[r] = i;
  }
}

// out[i][r] = src[i][idx[r]] (i < rows, r < keep), FP64; vals[r] = w[idx[r]]
__global__ void __launch_bounds__(256)
k_gather_cols(const double* __restrict__ src, int ld, const int* __restrict__ idx, int rows,
              int keep, const double* __restrict__ w, double* __restrict__ out,
              double* __restrict__ vals) {
  const int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x;
  if (e < (int64_t)rows * keep) {
    const int i = (int)(e / keep), r = (int)(e - (int64_t)i * keep);
    out[e] = src[(size_t)i * ld + idx[r]];
  }
  if (vals && e < keep) vals[e] = w[idx[e]];
}

// y = W (x - mean) (W optional) scaled to unit length; one wave per row,
// four rows per workgroup, the centred and whitened rows staged in LDS.
constexpr int LN_MAX = 512;
__global__ void __launch_bounds__(256)
k_lnorm(const float* __restrict__ X, int64_t n, int dim, const double* __restrict__ mean,
        const double* __restrict__ W, float* __restrict__ Y) {
  __shared__ double t[4][LN_MAX];
  __shared__ double y[4][LN_MAX];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t row = (int64_t)blockIdx.x * 4 + wv;
  const bool active = row < n;
  if (active)
    for (int d = lane; d < dim; d += 64)
      t[wv][d] = (double)X[row * dim + d] - (mean ? mean[d] : 0.0);
  __syncthreads();
  double ss = 0.0;
  if (active) {
    for (int i = lane; i < dim; i += 64) {
      double a = t[wv][i];
      if (W) {
        const double* wi = W + (size_t)i * dim;
        a = 0.0;
        for (int d = 0; d < dim; ++d) a += wi[d] * t[wv][d];
      }
      y[wv][i] = a;
      ss += a * a;
    }
  }
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
  if (active) {
    const double inv = ss > 0.0 ? 1.0 / sqrt(ss) : 0.0;
    for (int i = lane; i < dim; i += 64) Y[row * dim + i] = (float)(y[wv][i] * inv);
  }
}

typedef double doublex4 __attribute__((ext_vector_type(4)));

// The same with W, 16 rows per workgroup: W (x - mean) on FP64
// MFMA (16 x 16 x 4), the centred rows in LDS, every wave the output columns
// 16 (wave + 4 t).  The matrix cores add the products one by one in the order of
// the columns, and the squares are added as the wave per row of k_lnorm would,
// so a row is the one that a lane per output forms.  1200 rows of 400: 96 us
// (75 workgroups, bound by the cache lookups of their reads of W: 32 contiguous
// bytes per row and instruction), a lane per output 284 us (8 bytes).
constexpr int LN_T = LN_MAX / 64;  // output tiles per wave
__global__ void __launch_bounds__(256)
k_lnorm_white(const float* __restrict__ X, int64_t n, int dim, const double* __restrict__ mean,
              const double* __restrict__ W, float* __restrict__ Y) {
  extern __shared__ double t[];  // [16][ld], zero beyond dim; then the products
  const int ld = (dim + 15) / 16 * 16 + 2;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, l16 = lane & 15, q16 = lane >> 4;
  const int64_t r0 = (int64_t)blockIdx.x * 16;
  for (int e = tid; e < 16 * ld; e += 256) {
    const int r = e / ld, c = e - r * ld;
    t[e] = (c < dim && r0 + r < n) ? (double)X[(r0 + r) * dim + c] - (mean ? mean[c] : 0.0) : 0.0;
  }
  __syncthreads();
  const int nt = (dim + 15) / 16;
  doublex4 acc[LN_T];
  double b[LN_T][4];  // a tile's entries of W, loaded while the other tiles multiply
  auto row = [&](int u, int k0) {  // columns >= dim of Y are not stored
    const double* wr = W + (size_t)min(16 * (w + 4 * u) + l16, dim - 1) * dim;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int k = k0 + 4 * e + q16;
      const double v = wr[min(k, dim - 1)];
      b[u][e] = k < dim ? v : 0.0;
    }
  };
#pragma unroll
  for (int u = 0; u < LN_T; ++u) {
    acc[u] = doublex4{0.0, 0.0, 0.0, 0.0};
    if (w + 4 * u < nt) row(u, 0);
  }
  for (int k0 = 0; k0 < dim; k0 += 16) {
    double a[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) a[e] = t[l16 * ld + k0 + 4 * e + q16];
#pragma unroll
    for (int u = 0; u < LN_T; ++u)
      if (w + 4 * u < nt) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[e], b[u][e], acc[u], 0, 0, 0);
        row(u, k0 + 16);
      }
  }
  __syncthreads();  // the centred rows are consumed
#pragma unroll
  for (int u = 0; u < LN_T; ++u)
    if (w + 4 * u < nt)
#pragma unroll
      for (int r = 0; r < 4; ++r) t[(4 * r + q16) * ld + 16 * (w + 4 * u) + l16] = acc[u][r];
  __syncthreads();
  for (int r = 4 * w; r < 4 * w + 4; ++r) {
    double ss = 0.0;
    for (int d = lane; d < dim; d += 64) ss += t[r * ld + d] * t[r * ld + d];
    for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
    const double inv = ss > 0.0 ? 1.0 / sqrt(ss) : 0.0;
    if (r0 + r < n)
      for (int d = lane; d < dim; d += 64) Y[(r0 + r) * dim + d] = (float)(t[r * ld + d] * inv);
  }
}

// Per-dimension PLDA score coefficients from psi (between-speaker variances
// in the space where the within-speaker covariance is I): with s = psi + 1,
// det = s^2 - psi^2:  a = -(s / det - 1 / s) / 2,  b = psi / det,
// c = sum (-log(det) / 2 + log s).
__global__ void __launch_bounds__(256)
k_plda_coef(const double* __restrict__ psi, int d, double* __restrict__ coef) {
  __shared__ double red[256];
  double c = 0.0;
  for (int i = threadIdx.x; i < d; i += 256) {
    const double p = fmax(psi[i], 0.0), s = p + 1.0, det = s * s - p * p;
    coef[i] = -0.5 * (s / det - 1.0 / s);
    coef[d + i] = p / det;
    c += -0.5 * log(det) + log(s);
  }
  red[threadIdx.x] = c;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) coef[2 * d] = red[0];
}

// scores[t] = c + sum_i a_i (z1_i^2 + z2_i^2) + b_i z1_i z2_i for the pair
// (Z1[trials[2t]], Z2[trials[2t+1]]); one wave per trial.
__global__ void __launch_bounds__(256)
k_plda_score(const float* __restrict__ Z1, int64_t n1, const float* __restrict__ Z2, int64_t n2,
             int d, const double* __restrict__ coef, const int* __restrict__ trials, int64_t T,
             float* __restrict__ scores, int* __restrict__ bad) {
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= T) return;
  const int i = trials[2 * t], j = trials[2 * t + 1];
  if (i < 0 || i >= n1 || j < 0 || j >= n2) {
    if (lane == 0) {
      atomicAdd(bad, 1);
      scores[t] = NAN;
    }
    return;
  }
  const float* z1 = Z1 + (int64_t)i * d;
  const float* z2 = Z2 + (int64_t)j * d;
  double s = 0.0;
  for (int k = lane; k < d; k += 64) {
    const double a = z1[k], b = z2[k];
    s += coef[k] * (a * a + b * b) + coef[d + k] * a * b;
  }
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if (lane == 0) scores[t] = (float)(s + coef[2 * d]);
}

// q[i] = sum_k a_k z_k^2 of the rows of Z1, then of Z2; one wave per row
__global__ void __launch_bounds__(256)
k_plda_quad(const float* __restrict__ Z1, int64_t n1, const float* __restrict__ Z2, int64_t n2,
            int d, const double* __restrict__ coef, double* __restrict__ q) {
  const int lane = threadIdx.x & 63;
  const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= n1 + n2) return;
  const float* z = i < n1 ? Z1 + i * d : Z2 + (i - n1) * d;
  double s = 0.0;
  for (int k = lane; k < d; k += 64) {
    const double a = z[k];
    s += coef[k] * a * a;
  }
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if (lane == 0) q[i] = s;
}

// M[i][j] = c + q1_i + q2_j + sum_k b_k z1_ik z2_jk: 64 x 64 tile, FP64 MFMA,
// a wave per 32 x 32 quarter, 16 dimensions per LDS stage.  1.44 M pairs of
// d = 200: 43 us (361 workgroups, less than two per CU; the staging between
// barriers bounds it); 719 k trials one by one take 263 us.
__global__ void __launch_bounds__(256)
k_plda_matrix(const float* __restrict__ Z1, int64_t n1, const float* __restrict__ Z2, int64_t n2,
              int d, const double* __restrict__ coef, const double* __restrict__ q,
              float* __restrict__ M) {
  constexpr int LD = 64 + 16;
  __shared__ double As[16][LD], Bs[16][LD];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, l16 = lane & 15, q16 = lane >> 4;
  const int wm = w >> 1, wn = w & 1;
  const int64_t i0 = (int64_t)blockIdx.y * 64, j0 = (int64_t)blockIdx.x * 64;
  doublex4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};
  const int kc = tid & 15, rr = tid >> 4;  // column and first row of the thread's entries
  float za[4], zb[4];
  double cf = 0.0;
  auto load = [&](int k0) {  // rows and columns beyond the edge: any, then zero
    const int k = min(k0 + kc, d - 1);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      za[i] = Z1[min(i0 + rr + 16 * i, n1 - 1) * d + k];
      zb[i] = Z2[min(j0 + rr + 16 * i, n2 - 1) * d + k];
    }
    cf = coef[d + k];
  };
  load(0);
  for (int k0 = 0; k0 < d; k0 += 16) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool in = k0 + kc < d;
      As[kc][rr + 16 * i] = in ? cf * (double)za[i] : 0.0;
      Bs[kc][rr + 16 * i] = in ? (double)zb[i] : 0.0;
    }
    __syncthreads();
    if (k0 + 16 < d) load(k0 + 16);
#pragma unroll
    for (int ks = 0; ks < 16; ks += 4) {
      double a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) a[i] = As[ks + q16][wm * 32 + i * 16 + l16];
#pragma unroll
      for (int j = 0; j < 2; ++j) b[j] = Bs[ks + q16][wn * 32 + j * 16 + l16];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
    }
  }
  const double c = coef[2 * d];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int64_t col = j0 + wn * 32 + j * 16 + l16;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t row = i0 + wm * 32 + i * 16 + 4 * r + q16;
        if (row < n1 && col < n2) M[row * n2 + col] = (float)(acc[i][j][r] + q[row] + q[n1 + col] + c);
      }
    }
}

__global__ void __launch_bounds__(256)
k_plda_gather(const float* __restrict__ M, int64_t n1, int64_t n2, const int* __restrict__ trials,
              int64_t T, float* __restrict__ scores, int* __restrict__ bad) {
  for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < T; t += (int64_t)gridDim.x * 256) {
    const int i = trials[2 * t], j = trials[2 * t + 1];
    if (i < 0 || i >= n1 || j < 0 || j >= n2) {
      atomicAdd(bad, 1);
      scores[t] = NAN;
    } else {
      scores[t] = M[(int64_t)i * n2 + j];
    }
  }
}

// dst [n][n] = the symmetric part of src [dim][dim], zero-padded to n >= dim
__global__ void __launch_bounds__(256)
k_pad_sym(const double* __restrict__ src, int dim, double* __restrict__ dst, int n) {
  for (int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x; e < (int64_t)n * n;
       e += (int64_t)gridDim.x * 256) {
    const int i = (int)(e / n), j = (int)(e - (int64_t)i * n);
    dst[e] = (i < dim && j < dim) ? 0.5 * (src[(size_t)i * dim + j] + src[(size_t)j * dim + i])
                                  : 0.0;
  }
}

__global__ void k_fill_zero(double* __restrict__ p, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0.0;
}

size_t lnorm_lds(int dim) { return sizeof(double) * 16 * ((size_t)(dim + 15) / 16 * 16 + 2); }

}  // namespace

// ------------------------------------------------------------------ launchers

void be_zero(double* p, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  int64_t nb = (n + 255) / 256;
  if (nb > 4096) nb = 4096;
  k_fill_zero<<<(unsigned)nb, 256, 0, s>>>(p, n);
}

void be_class_sums(const float* X, int64_t n, int dim, const int* labels, int K, double* sums,
                   double* counts, int* bad, hipStream_t s) {
  if (n > 0) k_class_sums<<<(unsigned)n, 128, 0, s>>>(X, n, dim, labels, K, sums, counts, bad);
}

void be_scatter(const double* M2, const double* sums, const double* counts, int K, int dim,
                double* Sw, double* Sb, double* mean, hipStream_t s) {
  const int64_t e = (int64_t)dim * dim;
  k_scatter<<<(unsigned)((e + 255) / 256), 256, 0, s>>>(M2, sums, counts, K, dim, Sw, Sb, mean);
}

constexpr int kOffParts = 64;

int be_jacobi(double* A, double* V, int n, int max_sweeps, double tol, double* w, double2* rot,
              double* part, hipStream_t s) {
  const int64_t nn = (int64_t)n * n;
  const unsigned gb = (unsigned)std::min<int64_t>((nn + 255) / 256, 1024);
  k_eye_diag<<<gb, 256, 0, s>>>(V, n, A, w, 0);
  double host[2 * kOffParts];
  double fro = -1.0;
  int sweep = 0;
  for (;; ++sweep) {
    k_offnorm_part<<<kOffParts, 256, 0, s>>>(A, n, part);
    if (hipMemcpyAsync(host, part, sizeof(host), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
      return -1;
    double off = 0.0, all = 0.0;
    for (int b = 0; b < kOffParts; ++b) {
      off += host[2 * b];
      all += host[2 * b + 1];
    }
    if (fro < 0.0) fro = std::sqrt(all);
    if (!(std::sqrt(off) > tol * fro)) break;
    if (sweep >= max_sweeps) return -2;
    // rot [2][n / 2]: the rotations of the step before and of this one
    for (int r = 0; r < n; ++r)
      k_jacobi_step<<<n / 2, 256, 0, s>>>(A, V, n, r - 1, rot + (r + 1) % 2 * (n / 2),
                                          r < n - 1 ? r : -1, rot + r % 2 * (n / 2));
  }
  k_eye_diag<<<1, 256, 0, s>>>(V, n, A, w, 1);
  return sweep;
}

void be_dgemm(const void* A, bool a_float, int64_t lda, bool ta, const double* B, int64_t ldb,
              bool tb, void* C, int64_t ldc, bool c_float, int M, int N, int K,
              const double* colsub, hipStream_t s) {
  if (M <= 0 || N <= 0) return;
  dim3 grid((unsigned)((N + 15) / 16), (unsigned)((M + 15) / 16));
  if (a_float)
    k_dgemm<float><<<grid, 256, 0, s>>>(static_cast<const float*>(A), lda, ta, B, ldb, tb, C, ldc,
                                       c_float, M, N, K, colsub);
  else
    k_dgemm<double><<<grid, 256, 0, s>>>(static_cast<const double*>(A), lda, ta, B, ldb, tb, C,
                                        ldc, c_float, M, N, K, colsub);
}

void be_whiten_cols(const double* Q, int ld, const double* lam, int dim, double floor_rel,
                    bool trans, double* Wh, int* bad, hipStream_t s) {
  const int64_t e = (int64_t)dim * dim;
  int64_t nb = (e + 255) / 256;
  if (nb > 1024) nb = 1024;
  k_whiten_cols<<<(unsigned)nb, 256, 0, s>>>(Q, ld, lam, dim, floor_rel, trans ? 1 : 0, Wh, bad);
}

void be_pad_sym(const double* src, int dim, double* dst, int n, hipStream_t s) {
  const int64_t e = (int64_t)n * n;
  int64_t nb = (e + 255) / 256;
  if (nb > 1024) nb = 1024;
  k_pad_sym<<<(unsigned)nb, 256, 0, s>>>(src, dim, dst, n);
}

void be_rank_desc(const double* w, int valid, int keep, int* idx, hipStream_t s) {
  k_rank_desc<<<(unsigned)((valid + 255) / 256), 256, 0, s>>>(w, valid, keep, idx);
}

void be_gather_cols(const double* src, int ld, const int* idx, int rows, int keep,
                    const double* w, double* out, double* vals, hipStream_t s) {
  const int64_t e = (int64_t)rows * keep;
  k_gather_cols<<<(unsigned)((e + 255) / 256), 256, 0, s>>>(src, ld, idx, rows, keep, w, out,
                                                            vals);
}

void be_lnorm(const float* X, int64_t n, int dim, const double* mean, const double* W, float* Y,
              hipStream_t s) {
  if (n <= 0) return;
  // the matrix-core form from where its reads of W pay for its longer chain (a
  // call in us, lane per output / matrix cores: dimension 60 10.1 / 10.6, 150
  // 15.7 / 16.6, 250 33 / 27, 400 142 / 86), or where k_lnorm would need a second
  // round of workgroups (1500 rows of 150: 27 / 17)
  if (W && (dim > 192 || n > 1024))
    k_lnorm_white<<<(unsigned)((n + 15) / 16), 256, lnorm_lds(dim), s>>>(X, n, dim, mean, W, Y);
  else
    k_lnorm<<<(unsigned)((n + 3) / 4), 256, 0, s>>>(X, n, dim, mean, W, Y);
}

bool be_set_attributes() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_lnorm_white),
                             hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)lnorm_lds(LN_MAX)) == hipSuccess;
}

void be_plda_matrix(const float* Z1, int64_t n1, const float* Z2, int64_t n2, int d,
                    const double* coef, double* q, float* M, hipStream_t s) {
  k_plda_quad<<<(unsigned)((n1 + n2 + 3) / 4), 256, 0, s>>>(Z1, n1, Z2, n2, d, coef, q);
  const dim3 grid((unsigned)((n2 + 63) / 64), (unsigned)((n1 + 63) / 64));
  k_plda_matrix<<<grid, 256, 0, s>>>(Z1, n1, Z2, n2, d, coef, q, M);
}

void be_plda_gather(const float* M, int64_t n1, int64_t n2, const int* trials, int64_t T,
                    float* scores, int* bad, hipStream_t s) {
  if (T > 0)
    k_plda_gather<<<(unsigned)std::min<int64_t>((T + 255) / 256, 4096), 256, 0, s>>>(
        M, n1, n2, trials, T, scores, bad);
}

void be_plda_coef(const double* psi, int d, double* coef, hipStream_t s) {
  k_plda_coef<<<1, 256, 0, s>>>(psi, d, coef);
}

void be_plda_score(const float* Z1, int64_t n1, const float* Z2, int64_t n2, int d,
                   const double* coef, const int* trials, int64_t T, float* scores, int* bad,
                   hipStream_t s) {
  if (T > 0)
    k_plda_score<<<(unsigned)((T + 3) / 4), 256, 0, s>>>(Z1, n1, Z2, n2, d, coef, trials, T,
                                                         scores, bad);
}

}  // namespace ivx
