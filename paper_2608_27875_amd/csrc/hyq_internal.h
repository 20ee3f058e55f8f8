// Internal declarations shared by the libhyq translation units (host launch
// wrappers and small device helpers).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "hyq.h"

namespace hyq {

// ---- host-side launch wrappers (each returns a hipError_t) ----------------

// Compute units of the current device (cached per device).
int device_cus();

// The Q blocks of a call (64 rows of one head each), head-major.
struct QuantQ {
  const uint16_t* Q;
  int8_t* qc;
  float* qs;
  int L, n_qblk;
  int fmt;   // query codes: HYQ_FMT_INT (int8), HYQ_FMT_FP8 (E4M3) or HYQ_FMT_FP4Q6 (E2M3)
  int count;
};
QuantQ quant_q_all(const hyq_shape& s, const hyq_sizes& z, const uint16_t* Q, int8_t* q_codes,
                   float* q_scale);
void launch_quant_q(const QuantQ& q, hipStream_t st);

// Selection (Algorithm 1, or the column mass) into idx.  Scratch: scores
// ([B][Hkv][P], may be the caller's output), qsum (the per-head tail sums,
// [B][Hq][D]), hist ([B][Hkv][kSelHistBins] key counts), tws
// (select_topk_ws_bytes of top-k candidates and bitmaps), cm_ws (the column
// mass's scratch).  With qq (only where prefill_fuses: both then fit one grid
// dimension) also those Q blocks, beside the selection's own work.  A no-op
// when k = 0.
size_t select_topk_ws_bytes(int BH, int P);
bool prefill_fuses(const hyq_shape& s, const QuantQ& qq);
hipError_t launch_select(const hyq_shape& s, const hyq_sizes& z, const uint16_t* Q,
                         const uint16_t* K, int32_t* idx, float* scores, float* qsum,
                         uint32_t* hist, uint32_t* tws, float* cm_ws, const QuantQ* qq,
                         hipStream_t st);

// Column-mass scores (eq. vl_score) into scores[B][Hkv][P] and their key
// histograms into hist; clears the candidate count of each head (word
// bj * tws_words of tws).  cm_ws holds colmass_ws_bytes(s) bytes of scratch.
size_t colmass_ws_bytes(const hyq_shape& s);
hipError_t launch_colmass_scores(const hyq_shape& s, const hyq_sizes& z, const uint16_t* Q,
                                 const uint16_t* K, float* scores, uint32_t* hist, uint32_t* tws,
                                 size_t tws_words, float* cm_ws, hipStream_t st);

hipError_t launch_quantize(const hyq_shape& s, const hyq_sizes& z, const uint16_t* Q,
                           const uint16_t* K, const uint16_t* V, const int32_t* idx,
                           int8_t* q_codes, float* q_scale, uint8_t* k_codes, float* k_scale,
                           uint8_t* v_codes, float* v_scale, int32_t* kq_pos, hipStream_t st);

hipError_t launch_attn_prefill(const hyq_shape& s, const hyq_sizes& z, const uint16_t* Q,
                               const uint16_t* K, const uint16_t* V, const int32_t* idx,
                               const int8_t* q_codes, const float* q_scale,
                               const uint8_t* k_codes, const float* k_scale,
                               const uint8_t* v_codes, const float* v_scale,
                               const int32_t* kq_pos, float softmax_scale, void* out,
                               int out_dtype, hipStream_t st);

// The partition and the K/V block quantization of a prefill: kq_pos (the
// non-vertical prefix positions, ascending, then padding markers), codes and
// scales of z.n_kvblk blocks per (b, j).
void launch_quant_kv(const hyq_shape& s, const hyq_sizes& z, const uint16_t* K, const uint16_t* V,
                     const int32_t* idx, int32_t* kq_pos, uint8_t* k_codes, float* k_scale,
                     uint8_t* v_codes, float* v_scale, hipStream_t st);

// Decode: split of the sequence axis (quantized splits S_q, full-precision
// splits S_f, per KV head), workspace size, and the launches.
struct DecodeSplit {
  int nbq, S_q, S_f;   // quantized blocks; quantized and full-precision workgroups per KV head
};
constexpr int kDecodePartFloats = 132;   // one partial: acc[128], m, l, padding
DecodeSplit decode_split(const hyq_dcache& c);
size_t decode_ws_bytes(const hyq_dcache& c);
// Partials (bytes) that one decode attention launch writes for the cache's
// current state.
size_t decode_part_bytes(const hyq_dcache& c);
// Device address of the allocation-free call's scratch on the current device.
hipError_t noalloc_scratch(float** out);
// Freeze's partition, quantization and gather of the bf16 rows, as one launch.
hipError_t launch_freeze_kv(const hyq_dcache& c, const hyq_sizes& z, int N, const uint16_t* K,
                            const uint16_t* V, hipStream_t st);
hipError_t launch_decode_append(const hyq_dcache& c, const uint16_t* k_new, const uint16_t* v_new,
                                bool merge, int slot, hipStream_t st);
hipError_t launch_decode_attn(const hyq_dcache& c, const uint16_t* q, float softmax_scale,
                              void* out, int out_dtype, float* part, hipStream_t st);

// ---- device helpers -------------------------------------------------------

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t b) {
  return __uint_as_float(b << 16);
}

// Low / high bf16 of a packed pair, widened exactly.
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

constexpr int kHeadDim = 128;
constexpr int kBlock = 64;
// Top-k key histogram: bins of the top kSelHistBits bits of the score order key.
constexpr int kSelHistBits = 12;
constexpr int kSelHistBins = 1 << kSelHistBits;
// Number of i in [0, n) for which holds(i), a predicate that turns false once
// (wave-cooperative 64-ary search; every lane returns the same value).
template <class Pred>
__device__ __forceinline__ int wave_search(int n, Pred holds) {
  const int lane = threadIdx.x & 63;
  int lo = 0, hi = n;   // answer in [lo, hi]
  while (hi > lo) {
    const int step = (hi - lo + 63) / 64;
    const int i = lo + (lane + 1) * step - 1;
    const bool pred = i < hi && holds(i);
    lo += (int)__popcll(__ballot(pred)) * step;
    hi = min(hi, lo + step - 1);
    if (step == 1) break;
  }
  return lo;
}
// Order-preserving map float -> uint32 (larger float, larger key); -0 -> +0.
__device__ __forceinline__ uint32_t order_key(float f) {
  uint32_t u = __float_as_uint(f + 0.0f);   // -0 + 0 = +0
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
// Workgroup-local key histogram (top kSelHistBits bits of the order key),
// flushed into the KV head's histogram in global memory.
constexpr int kHistShift = 32 - kSelHistBits;   // the histogram bin is key >> kHistShift
__device__ __forceinline__ void hist_clear(uint32_t* lh) {
  for (int i = threadIdx.x; i < kSelHistBins; i += blockDim.x) lh[i] = 0u;
}
__device__ __forceinline__ void hist_flush(const uint32_t* lh, uint32_t* __restrict__ gh) {
  for (int i = threadIdx.x; i < kSelHistBins; i += blockDim.x) {
    const uint32_t c = lh[i];
    if (c) atomicAdd(gh + i, c);
  }
}

}  // namespace hyq
