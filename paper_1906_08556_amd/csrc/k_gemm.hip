// Dense FP32 GEMM on MFMA (v_mfma_f32_32x32x2_f32) for the E-step and M-step
// contractions: C = op(A) op(B), M x N x K.
//
//  * BM x BN output tile per workgroup of 4 waves (WM along M), each wave MI x
//    NJ blocks of 32 x 32, K staged 16 at a time through LDS with a register
//    double buffer for the next global tile.  Every shape adds the products of
//    an element in the same order (k ascending, fused), so the results do not
//    depend on the shape.
//  * op(A)(m, k) = A[m*lda + k] (TA = false) or A[k*lda + m] (TA = true);
//    op(B)(k, n) = B[k*ldb + n] (TB = false) or B[n*ldb + k] (TB = true).
//  * blockIdx.z = batch * ksplit + split; split s covers K range
//    [s*kchunk, min(K, (s+1)*kchunk)).
//  * Tile order: the larger operand is streamed once -- with m_fast the M
//    tiles of one column block of B are consecutive, otherwise the N tiles of
//    one row block of A.
//  * Epilogues: store FP32 (per split to its own slice), or store FP32 into
//    the tile-packed symmetric layout (lower 16 x 16 tiles only).
#include <algorithm>

#include "ivx_internal.h"
#include "k_gemm.h"

namespace ivx {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef floatx16 floatx16_t;

constexpr int BK = 16;

template <int MI, int WM, int NJ, bool TA, bool TB, int EPI>
__global__ void __launch_bounds__(256, 4) k_gemm(GemmArgs g) {
  constexpr int WN = 4 / WM, BM = 32 * MI * WM, BN = 32 * NJ * WN;
  constexpr int LDA_S = BM + 32;  // LDS row stride (floats) of the [k][m] tile
  constexpr int LDB_S = BN + 32;  // LDS row stride (floats) of the [k][n] tile
  constexpr int VA = BM * 4, VB = BN * 4;               // float4 per staged tile
  constexpr int JA = VA / 256, JB = VB / 256;
  __shared__ __attribute__((aligned(16))) float As[2][BK][LDA_S];
  __shared__ __attribute__((aligned(16))) float Bs[2][BK][LDB_S];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int h = lane >> 5, l32 = lane & 31;
  const int batch = blockIdx.z / g.ksplit, split = blockIdx.z % g.ksplit;
  const int m0 = (g.m_fast ? blockIdx.x : blockIdx.y) * BM;
  const int n0 = (g.m_fast ? blockIdx.y : blockIdx.x) * BN;
  if (EPI == GEMM_STORE_TP) {
    // skip workgroups whose tiles all lie strictly above the diagonal
    const int mlast = min(m0 + BM, g.M) - 1;
    if ((mlast >> 4) < (n0 >> 4)) return;
  }
  const float* A = g.A + batch * g.sA;
  const float* B = g.B + batch * g.sB;
  const int kb = split * g.kchunk;
  const int ke = min(g.K, kb + g.kchunk);

  // global tile loader: lanes run along the contiguous dimension of each
  // operand (coalesced), four consecutive elements per load (float4 where
  // the rows are 16-byte aligned); float4 number v = tid + 256 j covers
  //  !TA  A[m][k]: m = v / 4,        k = 4 (v % 4)
  //   TA  A[k][m]: k = v / (BM / 4), m = 4 (v % (BM / 4))
  // and the same for B with n in place of m
  const bool vecA = g.lda % 4 == 0 && g.sA % 4 == 0 && reinterpret_cast<uintptr_t>(g.A) % 16 == 0;
  const bool vecB = g.ldb % 4 == 0 && g.sB % 4 == 0 && reinterpret_cast<uintptr_t>(g.B) % 16 == 0;
  float4 ra[JA], rb[JB];
  // nval: how many of the four consecutive elements at p lie in bounds
  auto ld4 = [](const float* p, int nval, bool vec) -> float4 {
    float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (nval >= 4 && vec) {
      v = *reinterpret_cast<const float4*>(p);
    } else {
      if (nval > 0) v.x = p[0];
      if (nval > 1) v.y = p[1];
      if (nval > 2) v.z = p[2];
      if (nval > 3) v.w = p[3];
    }
    return v;
  };
  // aligned rows, whole float4 along M and N: loads without guards, at a uniform
  // base and a fixed offset per lane (rows and columns beyond the edge repeat
  // the last ones, their results are not stored); only the last K block is
  // guarded.  FP32 MFMAs and vector instructions take turns on the SIMD, so an
  // address or a guard per load costs MFMA time: 128 x 128 tiles at 4000 x
  // 80200 x 2048 take 11.4 ms (115 TFLOP/s, the clock near 2.1 GHz), with 64-bit
  // addresses and guards 12.6 ms; 64 x 64 tiles wait for their loads either way.
  const bool fast = vecA && vecB && (!TA || g.M % 4 == 0) && (TB || g.N % 4 == 0) &&
                    g.lda < (1 << 22) && g.ldb < (1 << 22);
  unsigned oa[JA], ob[JB];  // byte offsets
#pragma unroll
  for (int j = 0; j < JA; ++j) {
    const int v = tid + 256 * j;
    oa[j] = 4 * (TA ? (v / (BM / 4)) * (unsigned)g.lda + min(4 * (v % (BM / 4)), g.M - 4 - m0)
                    : min(v >> 2, g.M - 1 - m0) * (unsigned)g.lda + 4 * (v & 3));
  }
#pragma unroll
  for (int j = 0; j < JB; ++j) {
    const int v = tid + 256 * j;
    ob[j] = 4 * (TB ? min(v >> 2, g.N - 1 - n0) * (unsigned)g.ldb + 4 * (v & 3)
                    : (v / (BN / 4)) * (unsigned)g.ldb + min(4 * (v % (BN / 4)), g.N - 4 - n0));
  }
  auto load = [&](int k0) {
    if (fast && k0 + BK <= ke) {
      const char* pa = reinterpret_cast<const char*>(A + (TA ? (int64_t)k0 * g.lda + m0
                                                             : (int64_t)m0 * g.lda + k0));
      const char* pb = reinterpret_cast<const char*>(B + (TB ? (int64_t)n0 * g.ldb + k0
                                                             : (int64_t)k0 * g.ldb + n0));
#pragma unroll
      for (int j = 0; j < JA; ++j) ra[j] = *reinterpret_cast<const float4*>(pa + oa[j]);
#pragma unroll
      for (int j = 0; j < JB; ++j) rb[j] = *reinterpret_cast<const float4*>(pb + ob[j]);
      return;
    }
#pragma unroll
    for (int j = 0; j < JA; ++j) {
      const int v = tid + 256 * j;
      const int m = m0 + (TA ? 4 * (v % (BM / 4)) : v >> 2), k = k0 + (TA ? v / (BM / 4) : 4 * (v & 3));
      const float* p = A + (TA ? (int64_t)k * g.lda + m : (int64_t)m * g.lda + k);
      ra[j] = ld4(p, TA ? (k < ke ? min(4, g.M - m) : 0) : (m < g.M ? min(4, ke - k) : 0), vecA);
    }
#pragma unroll
    for (int j = 0; j < JB; ++j) {
      const int v = tid + 256 * j;
      const int n = n0 + (TB ? v >> 2 : 4 * (v % (BN / 4))), k = k0 + (TB ? 4 * (v & 3) : v / (BN / 4));
      const float* p = B + (TB ? (int64_t)n * g.ldb + k : (int64_t)k * g.ldb + n);
      rb[j] = ld4(p, TB ? (n < g.N ? min(4, ke - k) : 0) : (k < ke ? min(4, g.N - n) : 0), vecB);
    }
  };
  // rows k of a transposed tile are stored with bits 4 and 5 of the column
  // flipped by k / 4: the four lanes that write rows 4 apart meet four
  // different groups of banks (without it all four met the same one)
  auto sw = [](int k, int m, int width) { return width % 64 ? m : m ^ (16 * ((k >> 2) & 3)); };
  auto put = [&](float* S, int ld, int width, bool t, int v, const float4& r) {
    if (t) {  // four consecutive k of one row
      const int m = v >> 2, k = 4 * (v & 3), c = sw(k, m, width);
      S[k * ld + c] = r.x;
      S[(k + 1) * ld + c] = r.y;
      S[(k + 2) * ld + c] = r.z;
      S[(k + 3) * ld + c] = r.w;
    } else {
      const int k = v / (width / 4), m = 4 * (v % (width / 4));
      *reinterpret_cast<float4*>(S + k * ld + sw(k, m, width)) = r;
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int j = 0; j < JA; ++j) {
      const int v = tid + 256 * j;
      put(&As[buf][0][0], LDA_S, BM, !TA, v, ra[j]);
    }
#pragma unroll
    for (int j = 0; j < JB; ++j) {
      const int v = tid + 256 * j;
      put(&Bs[buf][0][0], LDB_S, BN, TB, v, rb[j]);
    }
  };

  floatx16 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = floatx16{0};

  const int nk = (ke > kb) ? (ke - kb + BK - 1) / BK : 0;
  if (nk > 0) {
    load(kb);
    store(0);
  }
  __syncthreads();
  auto step = [&](int it, int cur) {  // cur is a constant: fixed LDS addresses
    if (it + 1 < nk) load(kb + (it + 1) * BK);
#pragma unroll
    for (int s = 0; s < BK / 2; ++s) {
      const int k = 2 * s + h;
      float av[MI], bv[NJ];
#pragma unroll
      for (int i = 0; i < MI; ++i) av[i] = As[cur][k][sw(2 * s, (wm * MI + i) * 32 + l32, BM)];
#pragma unroll
      for (int j = 0; j < NJ; ++j) bv[j] = Bs[cur][k][sw(2 * s, (wn * NJ + j) * 32 + l32, BN)];
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i], bv[j], acc[i][j], 0, 0, 0);
    }
    if (it + 1 < nk) store(cur ^ 1);
    __syncthreads();
  };
  for (int it = 0; it < nk; it += 2) {
    step(it, 0);
    if (it + 1 < nk) step(it + 1, 1);
  }

  // epilogue: acc[i][j][r] is C[m][n] with m = mbase + 8*(r/4) + 4*h + r%4, n = nbase + l32
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int n = n0 + (wn * NJ + j) * 32 + l32;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = m0 + (wm * MI + i) * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
        if (m >= g.M || n >= g.N) continue;
        const float v = acc[i][j][r];
        float* C = g.C + batch * g.sC;
        if (EPI == GEMM_STORE) {
          C[split * g.sS + (int64_t)m * g.ldc + n] = v;
        } else {  // GEMM_STORE_TP: m, n are matrix row / column
          const int bi = m >> 4, bj = n >> 4;
          if (bi >= bj)
            C[(int64_t)(bi * (bi + 1) / 2 + bj) * 256 + (m & 15) * 16 + (n & 15)] = v;
        }
      }
    }
}

// At most UM rows (the E-step of a few utterances): C = A B with one column of
// B per lane, a wave per workgroup, the rows of A broadcast from LDS.  Bound by
// the one read of B; 32 rows of it are requested ahead (8 KB per wave in
// flight).  The same products in the same order as the MFMA tiles, which
// would compute 32 rows whatever M is.  U = 1 at C = 2048, R = 400 (681 MB of
// U_c): 256-row tile 677 us.
template <int UM>
__global__ void __launch_bounds__(64) k_gemm_rows(GemmArgs g) {
  constexpr int KC = 256, PF = 32;
  __shared__ __attribute__((aligned(16))) float As[KC][UM];
  const int lane = threadIdx.x, n = blockIdx.x * 64 + lane;
  const int kb = blockIdx.z * g.kchunk, ke = min(g.K, kb + g.kchunk);
  const float* B = g.B + min(n, g.N - 1);
  float acc[UM];
#pragma unroll
  for (int u = 0; u < UM; ++u) acc[u] = 0.0f;
  float nb[PF];
#pragma unroll
  for (int p = 0; p < PF; ++p) nb[p] = B[(int64_t)min(kb + p, g.K - 1) * g.ldb];
  for (int k0 = kb; k0 < ke; k0 += KC) {
    const int kc = min(KC, ke - k0);
    __syncthreads();  // one wave; the previous rows of A are consumed
    for (int i = lane; i < UM * KC; i += 64) {
      const int u = i / KC, k = i % KC;
      As[k][u] = (u < g.M && k < kc) ? g.A[(int64_t)u * g.lda + k0 + k] : 0.0f;
    }
    __syncthreads();
    for (int k1 = 0; k1 < kc; k1 += PF) {
      float b[PF];
#pragma unroll
      for (int p = 0; p < PF; ++p) b[p] = nb[p];
#pragma unroll
      for (int p = 0; p < PF; ++p)
        nb[p] = B[(int64_t)min(k0 + k1 + PF + p, g.K - 1) * g.ldb];
      if (k1 + PF <= kc) {
#pragma unroll
        for (int p = 0; p < PF; ++p)
#pragma unroll
          for (int u = 0; u < UM; ++u) acc[u] = fmaf(As[k1 + p][u], b[p], acc[u]);
      } else {
#pragma unroll
        for (int p = 0; p < PF; ++p)
          if (k1 + p < kc) {
#pragma unroll
            for (int u = 0; u < UM; ++u) acc[u] = fmaf(As[k1 + p][u], b[p], acc[u]);
          }
      }
    }
  }
  if (n < g.N) {
#pragma unroll
    for (int u = 0; u < UM; ++u)
      if (u < g.M) g.C[blockIdx.z * g.sS + (int64_t)u * g.ldc + n] = acc[u];
  }
}

// out[i] = sum over the splits of part[s][i], in order
__global__ void k_add_splits(const float* __restrict__ part, int ns, int64_t n, int64_t ncol,
                             int64_t ldo, float* __restrict__ out) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    float s = part[i];
    for (int k = 1; k < ns; ++k) s += part[k * n + i];
    out[i / ncol * ldo + i % ncol] = s;
  }
}

// 64 x 64 tiles where they leave less of the padded output empty: per element
// of the padded output they take 1.06 times what 128 x 128 tiles take (1000 x
// 83200 x 2048: 3.26 against 3.08 ms; 400 rows: 1.45 against 1.64 ms; 64 rows:
// 0.27 against 0.47 ms).  256 x 128 tiles took 12.1 ms for 4000 rows against
// 11.9 ms, 1.81 ms for 400; 32 x 256 tiles are bound by their loads (1.70 ms).
// Fewer than 512 large tiles leave CUs without two (64 rows of the linear term,
// 256 tiles: 0.23 against 0.12 ms).
bool small_tiles(int M, int N, int64_t z) {
  if ((int64_t)((M + 127) / 128) * ((N + 127) / 128) * z < 512) return true;
  auto area = [&](int64_t t) { return (double)(((M + t - 1) / t) * ((N + t - 1) / t) * t * t); };
  return 1.06 * area(64) < area(128);
}

template <bool TA, bool TB, int EPI>
void launch(GemmArgs g, int batches, hipStream_t s) {
  const int64_t z = (int64_t)batches * g.ksplit, t = small_tiles(g.M, g.N, z) ? 64 : 128;
  const int64_t mt = (g.M + t - 1) / t, nt = (g.N + t - 1) / t;
  // stream the larger operand (per K) once; y-dimension limits apply
  g.m_fast = ((int64_t)g.N > (int64_t)g.M && nt <= 65535) || mt > 65535 ? 1 : 0;
  const dim3 grid = g.m_fast ? dim3((unsigned)mt, (unsigned)nt, (unsigned)z)
                             : dim3((unsigned)nt, (unsigned)mt, (unsigned)z);
  if (t == 64)
    k_gemm<1, 2, 1, TA, TB, EPI><<<grid, 256, 0, s>>>(g);
  else
    k_gemm<2, 2, 2, TA, TB, EPI><<<grid, 256, 0, s>>>(g);
}

}  // namespace

bool gemm_f32(const GemmArgs& g0, bool ta, bool tb, int epi, int batches, hipStream_t s) {
  GemmArgs g = g0;
  if (g.ksplit < 1) g.ksplit = 1;
  if (g.ksplit == 1 || g.kchunk <= 0) {
    g.ksplit = 1;
    g.kchunk = g.K;
  }
  if (g.M <= 0 || g.N <= 0 || batches <= 0) return true;
  if (!ta && !tb && epi == GEMM_STORE && batches == 1 && g.M <= 16 && g.K > 0) {
    const dim3 grid((unsigned)((g.N + 63) / 64), 1, (unsigned)g.ksplit);
    auto* k = g.M <= 1 ? &k_gemm_rows<1>
              : g.M <= 2 ? &k_gemm_rows<2>
              : g.M <= 4 ? &k_gemm_rows<4>
              : g.M <= 8 ? &k_gemm_rows<8> : &k_gemm_rows<16>;
    k<<<grid, 64, 0, s>>>(g);
    return true;
  }
#define IVX_GEMM_CASE(TA_, TB_, EPI_)                 \
  if (ta == TA_ && tb == TB_ && epi == EPI_) {        \
    launch<TA_, TB_, EPI_>(g, batches, s);            \
    return true;                                      \
  }
  IVX_GEMM_CASE(false, false, GEMM_STORE)
  IVX_GEMM_CASE(true, false, GEMM_STORE_TP)
  IVX_GEMM_CASE(false, true, GEMM_STORE)
  IVX_GEMM_CASE(true, false, GEMM_STORE)
#undef IVX_GEMM_CASE
  return false;
}

bool gemm_f32_splitk(const GemmArgs& g0, bool ta, bool tb, float* ws, int64_t ws_elems,
                     hipStream_t s) {
  GemmArgs g = g0;
  if (g.M <= 0 || g.N <= 0) return true;
  // splits of at least 256 until there are 512 tiles of 128 x 128
  const int64_t tiles = (int64_t)((g.M + 127) / 128) * ((g.N + 127) / 128), n = (int64_t)g.M * g.N;
  int64_t ns = std::min<int64_t>({(512 + tiles - 1) / tiles, g.K / 256, ws_elems / n});
  if (ns < 2) return gemm_f32(g, ta, tb, GEMM_STORE, 1, s);
  g.kchunk = (int)(((g.K + ns - 1) / ns + 15) / 16 * 16);
  g.ksplit = (g.K + g.kchunk - 1) / g.kchunk;
  float* out = g.C;
  const int64_t ldo = g.ldc;
  g.C = ws;
  g.ldc = g.N;
  g.sS = n;
  if (!gemm_f32(g, ta, tb, GEMM_STORE, 1, s)) return false;
  k_add_splits<<<(unsigned)std::min<int64_t>((n + 255) / 256, 2048), 256, 0, s>>>(ws, g.ksplit, n,
                                                                                 g.N, ldo, out);
  return true;
}

}  // namespace ivx

// ------------------------------------------------------------ BF16 split form
// C[m][n] = sum_k A[m][k] B[n][k] (FP32 result) on v_mfma_f32_32x32x16_bf16
// from operands stored pre-split as BF16 high and low parts (v = hi + lo,
// both K-contiguous): hi*hi + hi*lo + lo*hi are accumulated in FP32.  Used
// for the precision assembly L(u) = I + N U in the BF16 form.  128 x 128
// output tile per workgroup, K staged 16 at a time, double-buffered LDS.
namespace ivx {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
constexpr int SR = 24;  // LDS row stride (bf16) of a staged 16-k row (48 B)

__global__ void __launch_bounds__(256, 2)
k_gemm_bf16x3_nt(const __bf16* __restrict__ Ahi, const __bf16* __restrict__ Alo, int64_t lda,
                 const __bf16* __restrict__ Bhi, const __bf16* __restrict__ Blo, int64_t ldb,
                 float* __restrict__ C, int64_t ldc, int M, int N, int K, int m_fast) {
  // [buf][operand: A hi, A lo, B hi, B lo][128 rows][SR]
  __shared__ __bf16 St[2][4][128 * SR];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int h = lane >> 5, l32 = lane & 31;
  // m_fast: the M tiles of one column block of B run consecutively
  const int64_t m0 = (int64_t)(m_fast ? blockIdx.x : blockIdx.y) * 128;
  const int64_t n0 = (int64_t)(m_fast ? blockIdx.y : blockIdx.x) * 128;
  // loader: thread covers row tid / 2 and k half (tid & 1) * 8 of each operand
  const int lr = tid >> 1, lk = (tid & 1) * 8;
  uint4 rg[4];
  auto load = [&](int k0) {
    const int64_t am = m0 + lr, bn = n0 + lr;
    const int k = k0 + lk;
    const bool ka = k < K;  // K is a multiple of 8
    rg[0] = (am < M && ka) ? *reinterpret_cast<const uint4*>(Ahi + am * lda + k) : make_uint4(0, 0, 0, 0);
    rg[1] = (am < M && ka) ? *reinterpret_cast<const uint4*>(Alo + am * lda + k) : make_uint4(0, 0, 0, 0);
    rg[2] = (bn < N && ka) ? *reinterpret_cast<const uint4*>(Bhi + bn * ldb + k) : make_uint4(0, 0, 0, 0);
    rg[3] = (bn < N && ka) ? *reinterpret_cast<const uint4*>(Blo + bn * ldb + k) : make_uint4(0, 0, 0, 0);
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int o = 0; o < 4; ++o) *reinterpret_cast<uint4*>(&St[buf][o][lr * SR + lk]) = rg[o];
  };
  floatx16_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = floatx16_t{0};
  const int nk = (K + 15) / 16;
  load(0);
  store(0);
  __syncthreads();
  for (int it = 0; it < nk; ++it) {
    const int cur = it & 1;
    if (it + 1 < nk) load((it + 1) * 16);
    bf16x8_t ah[2], al[2], bh[2], bl[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int ra = (wm * 64 + i * 32 + l32) * SR + 8 * h;
      const int rb = (wn * 64 + i * 32 + l32) * SR + 8 * h;
      ah[i] = *reinterpret_cast<const bf16x8_t*>(&St[cur][0][ra]);
      al[i] = *reinterpret_cast<const bf16x8_t*>(&St[cur][1][ra]);
      bh[i] = *reinterpret_cast<const bf16x8_t*>(&St[cur][2][rb]);
      bl[i] = *reinterpret_cast<const bf16x8_t*>(&St[cur][3][rb]);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], bh[j], acc[i][j], 0, 0, 0);
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], bl[j], acc[i][j], 0, 0, 0);
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[i], bh[j], acc[i][j], 0, 0, 0);
      }
    if (it + 1 < nk) store(cur ^ 1);
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int64_t n = n0 + wn * 64 + j * 32 + l32;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t m = m0 + wm * 64 + i * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
        if (m < M && n < N) C[m * ldc + n] = acc[i][j][r];
      }
    }
}

// src [rows][cols] FP32 -> hi / lo [rows][ldo] BF16 (cols <= ldo; padding 0)
__global__ void k_split_bf16(const float* __restrict__ src, int64_t rows, int64_t cols,
                             int64_t ldo, __bf16* __restrict__ hi, __bf16* __restrict__ lo) {
  const int64_t n = rows * ldo;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = i / ldo, c = i - r * ldo;
    const float v = (c < cols) ? src[r * cols + c] : 0.0f;
    const __bf16 vh = (__bf16)v;
    hi[i] = vh;
    lo[i] = (__bf16)(v - (float)vh);
  }
}

// src [rows][cols] FP32 -> hi / lo [cols][ldo] BF16 transposed (rows <= ldo;
// padding 0), through 64 x 64 LDS tiles
__global__ void __launch_bounds__(256)
k_split_bf16_t(const float* __restrict__ src, int64_t rows, int64_t cols, int64_t ldo,
               __bf16* __restrict__ hi, __bf16* __restrict__ lo) {
  __shared__ float t[64][65];
  const int64_t r0 = (int64_t)blockIdx.y * 64, c0 = (int64_t)blockIdx.x * 64;
  for (int e = threadIdx.x; e < 64 * 64; e += 256) {
    const int rr = e >> 6, cc = e & 63;
    const int64_t r = r0 + rr, c = c0 + cc;
    t[rr][cc] = (r < rows && c < cols) ? src[r * cols + c] : 0.0f;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 64 * 64; e += 256) {
    const int cc = e >> 6, rr = e & 63;
    const int64_t r = r0 + rr, c = c0 + cc;
    if (c < cols && r < ldo) {
      const float v = t[rr][cc];
      const __bf16 vh = (__bf16)v;
      hi[c * ldo + r] = vh;
      lo[c * ldo + r] = (__bf16)(v - (float)vh);
    }
  }
}

}  // namespace

void split_bf16(const float* src, int64_t rows, int64_t cols, int64_t ldo, __bf16* hi, __bf16* lo,
                hipStream_t s) {
  if (rows <= 0) return;
  k_split_bf16<<<2048, 256, 0, s>>>(src, rows, cols, ldo, hi, lo);
}

void split_bf16_transposed(const float* src, int64_t rows, int64_t cols, int64_t ldo, __bf16* hi,
                           __bf16* lo, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return;
  dim3 grid((unsigned)((cols + 63) / 64), (unsigned)((ldo + 63) / 64));
  k_split_bf16_t<<<grid, 256, 0, s>>>(src, rows, cols, ldo, hi, lo);
}

void gemm_bf16x3_nt(const __bf16* Ahi, const __bf16* Alo, int64_t lda, const __bf16* Bhi,
                    const __bf16* Blo, int64_t ldb, float* C, int64_t ldc, int M, int N, int K,
                    hipStream_t s) {
  if (M <= 0 || N <= 0) return;
  const unsigned mt = (unsigned)((M + 127) / 128), nt = (unsigned)((N + 127) / 128);
  const int m_fast = (N > M && nt <= 65535u) || mt > 65535u ? 1 : 0;  // stream B once
  const dim3 grid = m_fast ? dim3(mt, nt) : dim3(nt, mt);
  k_gemm_bf16x3_nt<<<grid, 256, 0, s>>>(Ahi, Alo, lda, Bhi, Blo, ldb, C, ldc, M, N, K, m_fast);
}

}  // namespace ivx
