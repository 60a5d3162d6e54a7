// Frame scores of small batches: the dense kernel's expanded-feature product
// split over components as well as frames.
//
// The persistent dense kernel (k_frame.hip) gives a 128-frame tile to one
// workgroup, which sweeps all C components: 2.2 ms at C = 2048, D = 60 however
// few frames there are, on 1 of 256 CUs for 100 frames.  Here a wave forms one
// block of 16 (FP32) or 32 (BF16) components for 16 NF or 32 frames, so that
// 100 frames already give 900 waves, and writes the scores [F][Cpad]; a second
// kernel takes every frame's maximum and its candidates in the dense kernel's
// order.
//
// The scores are the dense kernel's bit for bit: v_mfma_f32_16x16x4_f32 adds
// its four products one after the other with fused multiply-adds, as
// v_mfma_f32_32x32x2_f32 does its two, so the features taken in the same order
// (0, 4, 1, 5, 2, 6, 3, 7 of every chunk of 8) give the same sums; the BF16
// form uses the same instruction.
#include <algorithm>
#include <cmath>

#include "ivx_internal.h"

namespace ivx {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// Frames [Fdev[0] or F] (numbers flist[i] where given); more than fcap: nothing
// (they do not fit the score buffer and are left to the dense kernel).
__device__ inline int64_t batch(int64_t F, const int* Fdev, int64_t fcap) {
  if (Fdev && (int64_t)Fdev[0] < F) F = Fdev[0];
  return F <= fcap ? F : 0;
}

// One workgroup unit: 16 NF frames x 64 components, a block of 16 components
// per wave.  Units of one frame group are consecutive, so the XCDs (workgroups
// are dealt to them in turn) each keep one part of W in their L2.  The features
// of a slab of 64 / NF chunks are formed once for the four waves and kept in LDS
// in operand order; two MFMAs then take one 8-byte read.  Bound by the cache
// lookups of W's coefficients: C = 2048, D = 60, 100 frames take 36 us, 1013
// frames 130 us (24 us when every chunk of the 100 read the same coefficients, 60
// and 238 us with two 4-byte loads per lane and chunk and 16 or 32 frames per
// wave); the chain of 474 dependent MFMAs at NF = 1 is 7 us.
template <int NF>
__global__ void __launch_bounds__(256)
k_scores_f32(const float* __restrict__ X, int64_t F, int D, const float* __restrict__ shift,
             const float* __restrict__ W, int C, int Cpad, int Kpad,
             const uint16_t* __restrict__ pairs, const int* __restrict__ Fdev,
             const int* __restrict__ flist, int64_t fcap, float* __restrict__ scores) {
  constexpr int SQ = 64 / NF;  // chunks per slab
  extern __shared__ float sm[];
  const int DS = (D + 1) | 1, nq = Kpad / 8;
  float2* fe = reinterpret_cast<float2*>(sm);                      // [SQ][NF][64]
  float* xs = sm + 2 * 64 * 64;                                    // [16 NF][DS]
  uint32_t* tab = reinterpret_cast<uint32_t*>(xs + 16 * NF * DS);  // [nq][4]
  const int64_t n = batch(F, Fdev, fcap);
  const int ncg = (C + 63) / 64;
  const int64_t units = (n + 16 * NF - 1) / (16 * NF) * ncg;
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // lane group g takes features 4 (g % 2) + g / 2 and the next but one of a chunk
  if ((int64_t)blockIdx.x < units)
    for (int i = tid; i < nq * 4; i += 256) {
      const int k = 8 * (i >> 2) + 4 * (i & 1) + ((i >> 1) & 1);
      tab[i] = (uint32_t)pairs[k] | ((uint32_t)pairs[k + 2] << 16);
    }
  for (int64_t u = blockIdx.x; u < units; u += gridDim.x) {
    const int64_t f0 = u / ncg * (16 * NF);
    const int c0 = (int)(u % ncg) * 64 + wave * 16;  // Cpad is a multiple of 256
    __syncthreads();  // the previous unit's frames are consumed
    for (int i = tid; i < 16 * NF * (D + 1); i += 256) {
      const int fr = i / (D + 1), a = i - fr * (D + 1);
      const int64_t f = f0 + fr;
      float v = a == 0 ? 1.0f : 0.0f;
      if (a > 0 && f < n) v = X[(flist ? flist[f] : f) * D + a - 1] - shift[a - 1];
      xs[fr * DS + a] = v;
    }
    const size_t ws = (size_t)Cpad * 8;
    // a lane's two coefficients out of one 16-byte load: as two loads of 4 bytes at
    // a stride of 32 the cache lookups of a chunk take longer than its MFMAs
    const unsigned wl = l16 * 8 + 4 * (g & 1);
    const bool odd = g >> 1;
    floatx4 acc[NF];
#pragma unroll
    for (int j = 0; j < NF; ++j) acc[j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    // chunks requested ahead (L2 latency against 64 NF cycles per chunk)
    constexpr int PF = NF == 4 ? 4 : 8;
    const float* const wend = W + (size_t)(nq - 1) * ws + (size_t)c0 * 8;
    const float* wn = W + (size_t)c0 * 8;  // the next chunk to request; stays at the last
    float4 wv[PF];
    auto request = [&](int p) {
      wv[p] = *reinterpret_cast<const float4*>(wn + wl);
      wn = wn < wend ? wn + ws : wend;
    };
#pragma unroll
    for (int p = 0; p < PF; ++p) request(p);
    for (int s0 = 0; s0 < nq; s0 += SQ) {
      __syncthreads();  // the frames are staged, the previous slab is consumed
      // entry (chunk i / NF, frame block i % NF): a wave's 64 lanes in operand order
#pragma unroll 4
      for (int i = wave; i < 64; i += 4) {
        const int q = min(s0 + i / NF, nq - 1);
        const uint32_t t = tab[q * 4 + g];
        const float* x = xs + ((i % NF) * 16 + l16) * DS;
        fe[i * 64 + lane] = make_float2(x[t & 0xff] * x[(t >> 8) & 0xff],
                                        x[(t >> 16) & 0xff] * x[t >> 24]);
      }
      __syncthreads();
      const int q1 = min(s0 + SQ, nq);
      for (int q0 = s0; q0 < q1; q0 += PF) {
        const float2* fq = fe + (q0 - s0) * NF * 64 + lane;
        float2 b[PF][NF];
#pragma unroll
        for (int p = 0; p < PF; ++p)
#pragma unroll
          for (int j = 0; j < NF; ++j) b[p][j] = fq[(p * NF + j) * 64];
#pragma unroll
        for (int p = 0; p < PF; ++p) {
          const float a0 = odd ? wv[p].y : wv[p].x, a1 = odd ? wv[p].w : wv[p].z;
          request(p);
          if (q0 + p < nq) {
#pragma unroll
            for (int j = 0; j < NF; ++j)
              acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, b[p][j].x, acc[j], 0, 0, 0);
#pragma unroll
            for (int j = 0; j < NF; ++j)
              acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, b[p][j].y, acc[j], 0, 0, 0);
          }
        }
      }
    }
    // acc[j][r]: component c0 + 4 g + r, frame f0 + 16 j + l16
#pragma unroll
    for (int j = 0; j < NF; ++j) {
      const int64_t f = f0 + 16 * j + l16;
      if (f < n && c0 < C)
        *reinterpret_cast<float4*>(scores + f * Cpad + c0 + 4 * g) =
            make_float4(acc[j][0], acc[j][1], acc[j][2], acc[j][3]);
    }
  }
}

// The same with the BF16 split form: 32 frames x 128 components per unit, 32
// components per wave.
__global__ void __launch_bounds__(256)
k_scores_bf16(const float* __restrict__ X, int64_t F, int D, const float* __restrict__ shift,
              const __bf16* __restrict__ W16, int C, int Cpad, int Kpad,
              const uint16_t* __restrict__ pairs, const int* __restrict__ Fdev,
              const int* __restrict__ flist, int64_t fcap, float* __restrict__ scores) {
  extern __shared__ float sm[];
  const int DS = (D + 1) | 1, nq = Kpad / 16;
  float* xs = sm;                                              // [32][DS]
  uint32_t* prs = reinterpret_cast<uint32_t*>(xs + 32 * DS);   // [Kpad / 2], 16-byte aligned
  const int64_t n = batch(F, Fdev, fcap);
  const int ncg = (C + 127) / 128;
  const int64_t units = (n + 31) / 32 * ncg;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
  if ((int64_t)blockIdx.x < units)
    for (int i = tid; i < Kpad / 2; i += 256) prs[i] = reinterpret_cast<const uint32_t*>(pairs)[i];
  for (int64_t u = blockIdx.x; u < units; u += gridDim.x) {
    const int64_t f0 = u / ncg * 32;
    const int c0 = (int)(u % ncg) * 128 + (tid >> 6) * 32;
    __syncthreads();  // the previous unit's frames are consumed
    for (int i = tid; i < 32 * (D + 1); i += 256) {
      const int fr = i / (D + 1), a = i - fr * (D + 1);
      const int64_t f = f0 + fr;
      float v = a == 0 ? 1.0f : 0.0f;
      if (a > 0 && f < n) v = X[(flist ? flist[f] : f) * D + a - 1] - shift[a - 1];
      xs[fr * DS + a] = v;
    }
    __syncthreads();
    if (c0 >= C) continue;
    const __bf16* w = W16 + ((size_t)c0 + l32) * 32 + 8 * h;
    const size_t ws = (size_t)Cpad * 32;
    const float* xf = xs + l32 * DS;
    floatx16 acc = floatx16{0};
    bf16x8 nh = *reinterpret_cast<const bf16x8*>(w), nl = *reinterpret_cast<const bf16x8*>(w + 16);
    for (int q = 0; q < nq; ++q) {
      const bf16x8 wh = nh, wl = nl;
      const size_t o = (size_t)min(q + 1, nq - 1) * ws;
      nh = *reinterpret_cast<const bf16x8*>(w + o);
      nl = *reinterpret_cast<const bf16x8*>(w + o + 16);
      const uint4 pw = *reinterpret_cast<const uint4*>(prs + 8 * q + 4 * h);
      bf16x8 bh, bl;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t w32 = (e < 2) ? pw.x : (e < 4) ? pw.y : (e < 6) ? pw.z : pw.w;
        const uint32_t pr = w32 >> ((e & 1) * 16);
        const float v = xf[pr & 0xff] * xf[(pr >> 8) & 0xff];
        const __bf16 hi = (__bf16)v;
        bh[e] = hi;
        bl[e] = (__bf16)(v - (float)hi);
      }
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wh, bh, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wh, bl, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wl, bh, acc, 0, 0, 0);
    }
    // acc[4 b + e]: component c0 + 8 b + 4 h + e, frame f0 + l32
    const int64_t f = f0 + l32;
    if (f < n) {
#pragma unroll
      for (int b = 0; b < 4; ++b)
        *reinterpret_cast<float4*>(scores + f * Cpad + c0 + 8 * b + 4 * h) =
            make_float4(acc[4 * b], acc[4 * b + 1], acc[4 * b + 2], acc[4 * b + 3]);
    }
  }
}

// Candidate lists, maximum and overflow flag of every frame from its scores:
// one wave per frame, four consecutive components per lane and pass.  Slots as
// the dense kernel fills them: components with bit 2 clear (even lanes) from
// slot 0, the others from slot 8, ascending.
__global__ void __launch_bounds__(256)
k_scores_select(int64_t F, int C, int Cpad, const int* __restrict__ Fdev,
                const int* __restrict__ flist, int64_t fcap, const float* __restrict__ scores,
                float margin, int2* __restrict__ cand, float* __restrict__ cM,
                int* __restrict__ cflag) {
  const int64_t n = batch(F, Fdev, fcap);
  const int lane = threadIdx.x & 63;
  for (int64_t f = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); f < n; f += (int64_t)gridDim.x * 4) {
    const float* sc = scores + f * Cpad;
    float mx = -INFINITY;
    for (int c = 4 * lane; c < C; c += 256) {
      const float4 v = *reinterpret_cast<const float4*>(sc + c);
      mx = fmaxf(mx, v.x);
      if (c + 1 < C) mx = fmaxf(mx, v.y);
      if (c + 2 < C) mx = fmaxf(mx, v.z);
      if (c + 3 < C) mx = fmaxf(mx, v.w);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    const float thr = mx - margin;
    const int64_t g = flist ? flist[f] : f;
    int2* lst = cand + g * KP;
    if (lane < KP) lst[lane] = make_int2(-1, 0);
    const uint64_t half = (lane & 1) ? 0xaaaaaaaaaaaaaaaaull : 0x5555555555555555ull;
    const uint64_t below = half & ((1ull << lane) - 1ull);
    int cnt = 0;  // of the lane's half
    for (int cb = 0; cb < C; cb += 256) {
      const int c = cb + 4 * lane;
      float v[4];
      int m = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = c + e < C ? sc[c + e] : -INFINITY;
        if (c + e < C && v[e] >= thr) m |= 1 << e;
      }
      if (__ballot(m != 0) == 0) continue;
      int before = 0, all = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint64_t b = __ballot((m >> e) & 1);
        before += __popcll(b & below);
        all += __popcll(b & half);
      }
      int at = cnt + before;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if ((m >> e) & 1) {
          if (at < KP / 2) lst[(lane & 1) * (KP / 2) + at] = make_int2(c + e, __float_as_int(v[e]));
          ++at;
        }
      cnt += all;
    }
    const uint64_t ov = __ballot(cnt > KP / 2);
    if (lane == 0) {
      cM[g] = mx;
      cflag[g] = ov ? 1 : 0;
    }
  }
}

size_t scores_lds(int nf16, int D, int Kpad) {
  return sizeof(float) * ((size_t)16 * nf16 * ((D + 1) | 1) + (size_t)Kpad / 2);
}

constexpr size_t kSlabBytes = 64 * 64 * sizeof(float2);

}  // namespace

int64_t scores_frames(const ivx_ctx* ctx) {
  return ctx->scores ? (int64_t)(ctx->scores_bytes / (sizeof(float) * (size_t)ctx->Cpad)) : 0;
}

void launch_scores_select(ivx_ctx* ctx, const float* X, int64_t F, int prec, hipStream_t s,
                          const int* Fdev, const int* flist) {
  const int64_t fcap = scores_frames(ctx), Fm = std::min(F, fcap);
  if (Fm <= 0) return;
  const int C = ctx->C, D = ctx->D, Kpad = ctx->Kpad;
  const int64_t most = 8 * (int64_t)ctx->ncu;
  ProfScope ps(ctx, PK_FRAME_SELECT, s);
  if (prec == IVX_BF16) {
    const int64_t units = (Fm + 31) / 32 * ((C + 127) / 128);
    k_scores_bf16<<<(unsigned)std::min(units, most), 256, scores_lds(2, D, Kpad), s>>>(
        X, F, D, ctx->shift, ctx->W16, C, ctx->Cpad, Kpad, ctx->pairs, Fdev, flist, fcap,
        ctx->scores);
  } else {
    // 16 frames per wave while four workgroups per CU hold all (also for the
    // left-over frames of the bound, whose count only the device knows), else 64,
    // which read W a quarter as often.  C = 2048, D = 60, whole selection in us
    // with 16 / 32 / 64 / 128 frames: 100 frames 71 / 91 / 121 / 187, 512 frames
    // 116 / 123 / 138 / 205, 1013 frames 176 / 184 / 169 / 208, 4000 frames 506 /
    // 501 / 451 / 484.
    auto units = [&](int nf) { return (Fm + 16 * nf - 1) / (16 * nf) * ((C + 63) / 64); };
    const int nf = Fdev || units(1) <= 4 * (int64_t)ctx->ncu ? 1 : 4;
    auto* k = nf == 4 ? &k_scores_f32<4> : &k_scores_f32<1>;
    k<<<(unsigned)std::min(units(nf), most), 256, scores_lds(nf, D, Kpad) + kSlabBytes, s>>>(
        X, F, D, ctx->shift, ctx->Wexp, C, ctx->Cpad, Kpad, ctx->pairs, Fdev, flist, fcap,
        ctx->scores);
  }
  k_scores_select<<<(unsigned)std::min<int64_t>((Fm + 3) / 4, most), 256, 0, s>>>(
      F, C, ctx->Cpad, Fdev, flist, fcap, ctx->scores,
      prec == IVX_BF16 ? ctx->margin_bf16 : ctx->margin, ctx->cand, ctx->cM, ctx->cflag);
}

}  // namespace ivx
