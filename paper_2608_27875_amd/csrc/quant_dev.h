// Device helpers of per-block symmetric quantization (Algorithm 2, Stage 2),
// shared by the prefill quantizer and the decode cache's block merges.
#pragma once

#include "hyq_internal.h"
#include "recip_quotient.h"

#include <type_traits>

namespace hyq {

constexpr int kQuantThreads = 256;

// Maximum over the kQuantThreads threads of a workgroup (every thread gets it).
__device__ __forceinline__ float block_max(float v, float* sh) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) sh[w] = v;
  __syncthreads();
  float r = sh[0];
  for (int i = 1; i < kQuantThreads / 64; ++i) r = fmaxf(r, sh[i]);
  __syncthreads();
  return r;
}

// 32 bf16 values (64 bytes) as float.
__device__ __forceinline__ void load32(const uint16_t* p, float* x) {
  const uint4* q = reinterpret_cast<const uint4*>(p);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const uint4 w = q[u];
    const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      x[u * 8 + 2 * e] = bf16_lo(ww[e]);
      x[u * 8 + 2 * e + 1] = bf16_hi(ww[e]);
    }
  }
}

// Codes of a quotient y = fl32(x / s), s > 0.
__device__ __forceinline__ int code_int(float y, float c) {
  return (int)fminf(fmaxf(__builtin_rintf(y), -c), c);
}

// E4M3 bit pattern; the clamp keeps -0 and bounds the quotient by the largest
// finite value.
__device__ __forceinline__ int code_fp8(float y) {
  y = fminf(fmaxf(y, -448.0f), 448.0f);
  return __builtin_amdgcn_cvt_pk_fp8_f32(y, 0.0f, 0, false) & 0xff;
}

// E2M1 code (0..15): the nearest of the magnitudes 0, 0.5, 1, 1.5, 2, 3, 4, 6
// (codes 0..7), a tie going to the even code, beyond 5 the largest; bit 3 is
// the sign of the quotient (so -0 gives 8).
__device__ __forceinline__ int code_fp4(float y) {
  const float a = fabsf(y);
  const int c = (a > 0.25f) + (a >= 0.75f) + (a > 1.25f) + (a >= 1.75f) + (a > 2.5f) +
                (a >= 3.5f) + (a > 5.0f);
  return c | (int)((__float_as_uint(y) >> 31) << 3);
}

// E2M3 code (0..63): the nearest of the 32 magnitudes (eighths below 2,
// quarters up to 4, halves up to 7.5), a tie going to the even code, beyond
// 7.5 the largest; bit 5 is the sign of the quotient.  Within each binade
// [0,1), [1,2), [2,4), [4,8) the magnitudes are evenly spaced and start at an
// even code, so the nearest one is the binade's first code plus
// rint((a - base) / step), computed exactly.
__device__ __forceinline__ int code_fp6(float y) {
  const float a = fabsf(y);
  const float base = a < 1.0f ? 0.0f : a < 2.0f ? 1.0f : a < 4.0f ? 2.0f : 4.0f;
  const float inv = a < 2.0f ? 8.0f : a < 4.0f ? 4.0f : 2.0f;
  const int c0 = a < 1.0f ? 0 : a < 2.0f ? 8 : a < 4.0f ? 16 : 24;
  const int c = min(31, c0 + (int)__builtin_rintf(fminf(a - base, 8.0f) * inv));
  return c | (int)((__float_as_uint(y) >> 31) << 5);
}

template <int FMT>
__device__ __forceinline__ int code_of(float y, float c) {
  if (FMT == HYQ_FMT_FP8) return code_fp8(y);
  if (FMT == HYQ_FMT_FP4) return code_fp4(y);
  if (FMT == HYQ_FMT_FP4Q6) return code_fp6(y);
  return code_int(y, c);
}

// Code of x with the correctly rounded IEEE quotient x / s (s > 0).
template <int FMT>
__device__ __forceinline__ int quant_code(float x, float s, float c) {
  return code_of<FMT>(x / s, c);
}

// The same quotient by the block's reciprocal r = fl32(1 / s) where
// recip_ok(s): three operations (and the sign of x, which the floating-point
// codes keep for -0) instead of about twelve, which held the quantization
// kernels back as much as memory did (Q at 32k, 32 heads, 402 MB: 76.1 us
// before, 62.9 us now, each in a launch of its own; K and V at 32k, 8 heads,
// int4: 42.5 us before, 36.7 us although the partition and Freeze's gather
// joined the launch).
template <int FMT>
__device__ __forceinline__ float quot(float x, float s, float r) {
  const float y = recip_quotient(x, s, r);
  return FMT == HYQ_FMT_INT ? y : __builtin_copysignf(y, x);
}

// Eight codes, one per byte of o[0], o[1], of the eight bf16 values in w.
template <int FMT, bool RECIP>
__device__ __forceinline__ void codes8(const uint32_t (&w)[4], float s, float r, float c,
                                       uint32_t (&o)[2]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    float y[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float x = e & 1 ? bf16_hi(w[2 * h + (e >> 1)]) : bf16_lo(w[2 * h + (e >> 1)]);
      y[e] = RECIP ? quot<FMT>(x, s, r) : x / s;
    }
    if constexpr (FMT == HYQ_FMT_FP8) {   // two conversions fill the word
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = fminf(fmaxf(y[e], -448.0f), 448.0f);
      int v = __builtin_amdgcn_cvt_pk_fp8_f32(y[0], y[1], 0, false);
      v = __builtin_amdgcn_cvt_pk_fp8_f32(y[2], y[3], v, true);
      o[h] = (uint32_t)v;
    } else {
      uint32_t v = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) v |= (uint32_t)(code_of<FMT>(y[e], c) & 0xff) << (8 * e);
      o[h] = v;
    }
  }
}

// Bound c of the query codes of a format.
template <int FMT>
constexpr float query_bound() {
  return FMT == HYQ_FMT_FP8 ? 448.0f : FMT == HYQ_FMT_FP4Q6 ? 7.5f : 127.0f;
}

// Block `blk` of a share of Q blocks (64 rows of one head) by a workgroup of
// kQuantThreads threads: codes and scale.  Thread t takes the 16-byte chunks
// t % 16 of rows t / 16 + 16i, so every load instruction of a wave reads 1 KB
// and every store writes 512 contiguous bytes.  (One wave per block instead,
// without LDS, streams as fast but takes four times as long per block, which
// a short prompt waits for.)
template <int FMT>
__device__ __forceinline__ void quant_q_block(const QuantQ& a, int blk, float* red) {
  constexpr float C = query_bound<FMT>();
  const int bh = blk / a.n_qblk, qb = blk - bh * a.n_qblk;
  const int r0 = qb * kBlock + ((int)threadIdx.x >> 4), ch = threadIdx.x & 15;
  constexpr int kRowsPer = kQuantThreads / 16, kN = kBlock / kRowsPer;
  const uint16_t* src = a.Q + (size_t)bh * a.L * kHeadDim;
  uint4 w[kN];
#pragma unroll
  for (int i = 0; i < kN; ++i) {   // rows past L re-read the last one (the maximum is the same)
    const int t = min(r0 + kRowsPer * i, a.L - 1);
    w[i] = reinterpret_cast<const uint4*>(src + (size_t)t * kHeadDim)[ch];
  }
  float m = 0.0f;
#pragma unroll
  for (int i = 0; i < kN; ++i) {
    const uint32_t ww[4] = {w[i].x, w[i].y, w[i].z, w[i].w};
#pragma unroll
    for (int e = 0; e < 4; ++e) m = fmaxf(m, fmaxf(fabsf(bf16_lo(ww[e])), fabsf(bf16_hi(ww[e]))));
  }
  const float s = block_max(m, red) / C;
  if (threadIdx.x == 0) a.qs[blk] = s;
  const float r = 1.0f / s;
  int8_t* dst = a.qc + (size_t)bh * a.L * kHeadDim + ch * 8;
  auto emit = [&](auto kind) {   // 0: all codes zero, 1: by the reciprocal, 2: by division
    constexpr int KIND = decltype(kind)::value;
#pragma unroll
    for (int i = 0; i < kN; ++i) {
      const int t = r0 + kRowsPer * i;
      const uint32_t ww[4] = {w[i].x, w[i].y, w[i].z, w[i].w};
      uint32_t o[2] = {0u, 0u};
      if constexpr (KIND != 0) codes8<FMT, KIND == 1>(ww, s, r, C, o);
      if (t < a.L) *reinterpret_cast<uint2*>(dst + (size_t)t * kHeadDim) = make_uint2(o[0], o[1]);
    }
  };
  if (recip_ok(s)) emit(std::integral_constant<int, 1>{});
  else if (s > 0.0f) emit(std::integral_constant<int, 2>{});
  else emit(std::integral_constant<int, 0>{});
}

// c_B of a code format and bit-width (Algorithm 2, Stage 2).
template <int BITS, int FMT>
constexpr float code_bound() {
  return FMT == HYQ_FMT_FP8 ? 448.0f : FMT == HYQ_FMT_FP4 ? 6.0f : (BITS == 8 ? 127.0f : 7.0f);
}

}  // namespace hyq
