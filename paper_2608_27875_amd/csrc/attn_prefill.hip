// Hybrid-precision causal prefill attention: Algorithm 2, Stage 3 (App. A.2)
// and eq. (prefill_hybrid) of Section 4.2 of HyQuant.
//
// One workgroup = one KV head (b, j) x 8 work units, a unit being (32 query
// rows, one query head of the group); with g = 4 that is two 32-row tiles of
// the 4 heads.  The 8 waves (two per SIMD) share every K/V tile staged in
// LDS.  Each wave keeps one online-softmax state per query row and scans
//   segment A: the quantized keys (compacted K_Q order) in tiles of 64 =
//              one quantization block: S^T = K_codes * Qcodes^T with the int8
//              MFMA (exact int32) or, for FP8 codes, the E4M3 MFMA (float32),
//              or, for FP4 codes, the scaled MFMA with E2M1 keys against
//              E4M3 queries; logits scaled by alpha*log2(e)*sQ*sK; P V with
//              the f16 MFMA on the V codes (int8, E4M3 and E2M1 values are
//              exact in f16);
//   segments B and C: the full-precision keys (vertical lines, then the
//              window), 64 at a time gathered into two alternating LDS
//              buffers a tile ahead through registers: S^T with the bf16
//              MFMA; P V with the f16 MFMA on V / sVref converted to f16
//              (exact for bf16 values of that range); a tile whose V / sVref
//              leaves the f16 range raises sVref (the accumulator rescaled
//              exactly) and is staged again.
// Causality is by original key position in every segment.  With the
// per-query window (HYQ_WIN_BAND) row t sees keys t+1-W .. t in full
// precision and a quantized key only once it is older than that: segment A
// compares positions with t - W, and the full-precision list also carries the
// quantizable keys of the workgroup's band, each seen by W rows.
//
// Launches too small to fill the chip that way split the keys as well, or
// take smaller workgroups (attn_shape.h): two groups of 4 waves per
// workgroup, each with its own LDS rings and every other tile of the same 4
// units, merged at the end; 4-wave workgroups, two per CU; or one unit per
// workgroup with the keys split over its 8 waves (attn_prefill_split_kernel).
//
// Register layout (32x32 MFMA, wave64): lane l, accumulator register r holds
// row (r/4)*8 + (l/32)*4 + r%4 and column l%32.  With keys as rows (S^T),
// each lane owns one query (column) and 16 keys per 32-key half; those 16
// values are reused directly as the B operand of the P V product, and the
// V^T tile in LDS stores each 16-key group in the matching order
// [0-3, 8-11, 4-7, 12-15].
//
// Quantized tiles run through LDS rings fed from registers (K four
// buffers, V two): while tile c is computed, K(c+2) and V(c) (loaded into
// registers during tile c-1) are converted and written to LDS and K(c+3),
// V(c+1) are loaded, so global latency is covered by a whole tile and each
// barrier waits only for LDS writes.  The P V product of tile c-1 is issued
// interleaved with the softmax of tile c (one MFMA per weight pair) so that
// the matrix cores and the vector ALUs overlap within each wave.
//
// V scales: with sVref a power of two >= every sV of the head, the ratio
// sV/sVref = fm * 2^e is split into its mantissa fm in [1/2, 1) and its
// power of two.  2^e is applied exactly to the V codes when they are
// staged as f16 (a block with a small scale only ever gives small V values,
// whose rounding stays small against the output); fm is folded into the
// exponent, P' = 2^(y - m + log2 fm), so the f16 weights never lose range.
// The accumulator holds O * l / sVref; the row sum l adds P' / fm per tile
// (from the same f16 values that enter the MFMA).  An all-zero V block
// (sV = 0) folds nothing.
#include "attn_shape.h"
#include "codes_dev.h"
#include "hyq_internal.h"

#include <type_traits>

namespace hyq {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v2f __attribute__((ext_vector_type(2)));

constexpr int kTile = 64;
// 16-byte chunks of one staged tile: 8-bit K and V tiles are 512 chunks, 4-bit 256
constexpr int kChunks8 = kTile * kHeadDim / 16;
constexpr int kChunks4 = kChunks8 / 2;
constexpr float kLazy = 8.0f;             // general path: rescale only when the max grows by > 2^8
constexpr float kFastMax = 32768.0f;      // fast path: largest accepted weight sum of a lane
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kMinusBig = -1.0e30f;

// Key/value codes of the two FP4 formats are the same E2M1 nibbles; they
// differ only in the query codes (E4M3, or E2M3 for HYQ_FMT_FP4Q6).
constexpr bool kv_fp4(int fmt) { return fmt == HYQ_FMT_FP4 || fmt == HYQ_FMT_FP4Q6; }

// LDS row pitches (bytes).  +16 keeps the 16-byte reads of 8 consecutive
// rows on distinct banks.
// int8 K tile: 64 rows of 128 B with no padding; the 16-byte chunk j of row r
// is stored at slot j ^ ((r / 2) % 8): a 256-byte bank row holds two K rows,
// so the 16 lanes of one 16-byte read phase (16 consecutive rows, one chunk)
// land on distinct banks.
constexpr int kKRowI8 = kHeadDim;
constexpr int kKPitchBf = kHeadDim * 2 + 16;    // bf16 K row
constexpr int kVPitch = kTile * 2 + 16;          // one channel of 64 f16/bf16 keys
constexpr int kVBytes = kHeadDim * kVPitch;

// Tile metadata: kq_pos of the 64 slots, the bits of sK and sV (read from
// LDS rather than with scalar loads, whose counter would also wait for every
// pending LDS read), and one slot that absorbs the stores of the other
// staging threads so that staging needs no branch.
constexpr int kMetaSK = kTile, kMetaSV = kTile + 1, kMetaSink = kTile + 2;
struct KBuf {                       // K codes and metadata of one quantized tile
  alignas(16) uint8_t k[kTile * kKRowI8];
  int32_t pos[kTile + 4];
};
struct VBuf {                       // V of one quantized tile as f16 V^T
  alignas(16) uint8_t v[kVBytes];
};
// Quantized segment: tile c multiplies K(c) (fragments read from kb[c%4] at
// the end of tile c-1) and V(c-1) from vb[(c-1)%2]; it writes K(c+2) to
// kb[(c+2)%4] and V(c) to vb[c%2], and reads the fragments of K(c+1) from
// kb[(c+1)%4] (published one barrier earlier) before its closing barrier.
constexpr int kKRing = 4;
struct QRing {
  KBuf kb[kKRing];
  VBuf vb[2];
};
struct FBuf {                       // one full-precision tile
  alignas(16) uint8_t k[kTile * kKPitchBf];   // bf16 K rows
  alignas(16) uint8_t v[kVBytes];             // V^T as f16 V / sVref
  alignas(16) int32_t pos[kTile];             // rows t >= pos see the key ...
  alignas(16) int32_t hi[kTile];              // ... up to row hi
  int32_t ovf;     // (f << 8) | E: tile f staged here had a V / sVref outside the f16
                   // range, E the largest biased float exponent of its V values
};
// Nothing quantized: tile c multiplies K(c) and V(c-1), as the quantized
// segment does, while K(c+1) and V(c) are written.
struct DRing {
  alignas(16) uint8_t k[2][kTile * kKPitchBf];   // bf16 K rows
  VBuf vb[2];                                    // V^T as f16 V / sVref
  int32_t ovf[2];                                // as FBuf's, of the V tile beside it
};
// Full-precision tiles alternate between two buffers: tile f+1 is written
// while tile f is computed.
union Smem {
  QRing q;
  FBuf f[2];
  DRing d;
};

__device__ __forceinline__ float xhalf_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float xhalf_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Number of entries <= x in the ascending array a[0, n).
__device__ int count_le(const int32_t* __restrict__ a, int n, int x) {
  return wave_search(n, [=](int i) { return a[i] <= x; });
}

// Slot of key e (0..63) in the permuted V^T row.
__device__ __forceinline__ int vslot(int e) {
  const int r = e & 15, c4 = r >> 2;
  const int sc = (c4 == 1) ? 2 : (c4 == 2) ? 1 : c4;
  return (e & ~15) + sc * 4 + (r & 3);
}

// ---------------------------------------------------------------------------
// Quantized tiles, staged through registers: K codes (compacted order), V
// codes (channel-major), kq_pos and the two block scales of one tile.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int kswz(int row, int chunk) {
  return row * kKRowI8 + ((chunk ^ ((row >> 1) & 7)) << 4);
}
// E2M1 K tile: 64 rows of 64 B (four 16-byte chunks); a 256-byte bank row
// holds four K rows, so chunk j of row r sits at slot j ^ ((r / 4) % 4) and
// the 16 rows of one read phase land on distinct banks.
__device__ __forceinline__ int kswz4(int row, int chunk) {
  return row * (kHeadDim / 2) + ((chunk ^ ((row >> 2) & 3)) << 4);
}

// (native vectors: aggregate copies of HIP's uint4 would go through memory)
// Chunks per thread of an NT-thread workgroup: 8-bit tiles split evenly; a
// 4-bit tile has one chunk for each of its first 256 threads, and the other
// threads (if any) repeat them (same data to the same LDS bytes), which keeps
// staging branch-free.
template <int BITS, int NT>
constexpr int chunks_per_thread() {
  static_assert(kChunks8 % NT == 0 && NT >= kChunks4, "tile chunks must split evenly");
  return BITS == 8 ? kChunks8 / NT : 1;
}
template <int BITS, int NT>
__device__ __forceinline__ int chunk_id(int tid, int i) {
  return BITS == 8 ? tid + i * NT : (tid & (kChunks4 - 1));
}

template <int BITS, int NT>
struct StageRegs {
  v4u k[chunks_per_thread<BITS, NT>()];   // 16-byte chunks chunk_id(tid, i) of a K tile
  v4u v[chunks_per_thread<BITS, NT>()];   // same for a V tile
  int32_t meta;                 // threads 0..63: kq_pos; 64, 65: sK, sV bits (K's tile)
};

// K fragments of one tile for the S^T product (A operands of the two 32-key
// halves).  int8: 4 steps of v_mfma_i32_32x32x32_i8, lane half h holding
// channels 32*step + 16h .. +16; E4M3: 2 steps of
// v_mfma_scale_f32_32x32x64_f8f6f4, lane half h holding channels
// 64*step + 32h .. +32.  Q fragments (the B operands) split the channels the
// same way, which is all the dot product needs.
// E2M1 keys against E4M3 queries (2 steps of the same scaled MFMA): the
// 4-bit A operand of lane half h takes the products 16h .. +16 and
// 32 + 16h .. +16 of the step's 64, the 8-bit B operand of half h the
// products 32h .. +32; channels are assigned so that the K fragment is the
// 16 contiguous bytes of channels 64*step + 32h .. +32, and the Q fragment
// the two 16-byte runs at channels 64*step + 16h and 64*step + 32 + 16h.
// E2M1 keys against E2M3 queries (HYQ_FMT_FP4Q6): the 6-bit B operand of
// lane half h pairs element n with element n of the 4-bit A operand's half
// h (measured with one-hot operands), its 32 codes packed 6 bits apart in
// six registers; so the Q fragment is channels 64*step + 32h .. +32, the
// same channels as the K fragment, packed from one code byte each.
template <int FMT>
struct KFrag {
  v4i f[2][4];
};
template <>
struct KFrag<HYQ_FMT_FP8> {
  v8i f[2][2];
};
template <>
struct KFrag<HYQ_FMT_FP4> {
  v4i f[2][2];
};
template <>
struct KFrag<HYQ_FMT_FP4Q6> {
  v4i f[2][2];
};
template <int FMT>
struct QFrag {
  v4i f[4];
};
template <>
struct QFrag<HYQ_FMT_FP8> {
  v8i f[2];
};
template <>
struct QFrag<HYQ_FMT_FP4> {
  v8i f[2];
};
template <>
struct QFrag<HYQ_FMT_FP4Q6> {   // six registers of packed E2M3 codes per step
  v8i f[2];
};

template <int FMT>
__device__ __forceinline__ void read_kfrag(KFrag<FMT>& kf, const KBuf& b, int col, int half) {
#pragma unroll
  for (int kh = 0; kh < 2; ++kh) {
    if constexpr (FMT == HYQ_FMT_FP8) {
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const v4i lo = *reinterpret_cast<const v4i*>(b.k + kswz(kh * 32 + col, kk * 4 + half * 2));
        const v4i hi = *reinterpret_cast<const v4i*>(b.k + kswz(kh * 32 + col, kk * 4 + half * 2 + 1));
        kf.f[kh][kk] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      }
    } else if constexpr (kv_fp4(FMT)) {
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
        kf.f[kh][kk] = *reinterpret_cast<const v4i*>(b.k + kswz4(kh * 32 + col, kk * 2 + half));
    } else {
#pragma unroll
      for (int k4 = 0; k4 < 4; ++k4)
        kf.f[kh][k4] = *reinterpret_cast<const v4i*>(b.k + kswz(kh * 32 + col, k4 * 2 + half));
    }
  }
}

template <int FMT>
__device__ __forceinline__ void read_qfrag(QFrag<FMT>& qf, const int8_t* qrow, bool ok, int half) {
  if constexpr (FMT == HYQ_FMT_FP8) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
      qf.f[kk] = ok ? *reinterpret_cast<const v8i*>(qrow + kk * 64 + half * 32) : v8i{};
  } else if constexpr (FMT == HYQ_FMT_FP4) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const v4i lo = ok ? *reinterpret_cast<const v4i*>(qrow + kk * 64 + half * 16) : v4i{};
      const v4i hi = ok ? *reinterpret_cast<const v4i*>(qrow + kk * 64 + 32 + half * 16) : v4i{};
      qf.f[kk] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
  } else if constexpr (FMT == HYQ_FMT_FP4Q6) {
    // 32 code bytes (channels 64*kk + 32*half ..) -> 6-bit slots 0..31 of six
    // registers (slot n at bits 6n .. 6n+5); done once per wave
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const v4u lo = ok ? *reinterpret_cast<const v4u*>(qrow + kk * 64 + half * 32) : v4u{};
      const v4u hi = ok ? *reinterpret_cast<const v4u*>(qrow + kk * 64 + half * 32 + 16) : v4u{};
      const uint32_t w[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
      uint32_t r[6] = {0u, 0u, 0u, 0u, 0u, 0u};
#pragma unroll
      for (int n = 0; n < 32; ++n) {
        const uint32_t code = (w[n >> 2] >> (8 * (n & 3))) & 0x3Fu;
        const int bit = 6 * n;
        r[bit >> 5] |= code << (bit & 31);
        if ((bit & 31) > 26) r[(bit >> 5) + 1] |= code >> (32 - (bit & 31));
      }
      qf.f[kk] = v8i{(int)r[0], (int)r[1], (int)r[2], (int)r[3], (int)r[4], (int)r[5], 0, 0};
    }
  } else {
#pragma unroll
    for (int k4 = 0; k4 < 4; ++k4)
      qf.f[k4] = ok ? *reinterpret_cast<const v4i*>(qrow + k4 * 32 + half * 16) : v4i{};
  }
}

// S^T of one tile: int32 (int8 codes) or float32 (E4M3, E2M1 codes) logits.
template <int FMT>
using SVec = std::conditional_t<FMT == HYQ_FMT_INT, v16i, v16f>;

template <int FMT>
__device__ __forceinline__ void qk_tile(SVec<FMT> (&s)[2], const KFrag<FMT>& kf,
                                        const QFrag<FMT>& qf) {
#pragma unroll
  for (int kh = 0; kh < 2; ++kh) {
    s[kh] = SVec<FMT>{};
    if constexpr (FMT == HYQ_FMT_FP8) {
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)   // format 0 = E4M3 for both operands, unit scales
        s[kh] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(kf.f[kh][kk], qf.f[kk], s[kh], 0,
                                                                0, 0, 127, 0, 127);
    } else if constexpr (FMT == HYQ_FMT_FP4) {
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {   // A format 4 = E2M1 (4 registers), B format 0 = E4M3
        const v8i ka = __builtin_shufflevector(kf.f[kh][kk], v4i{}, 0, 1, 2, 3, 4, 5, 6, 7);
        s[kh] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(ka, qf.f[kk], s[kh], 4, 0, 0, 127,
                                                                0, 127);
      }
    } else if constexpr (FMT == HYQ_FMT_FP4Q6) {
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {   // A format 4 = E2M1, B format 2 = E2M3 (6 registers)
        const v8i ka = __builtin_shufflevector(kf.f[kh][kk], v4i{}, 0, 1, 2, 3, 4, 5, 6, 7);
        s[kh] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(ka, qf.f[kk], s[kh], 4, 2, 0, 127,
                                                                0, 127);
      }
    } else {
#pragma unroll
      for (int k4 = 0; k4 < 4; ++k4)
        s[kh] = __builtin_amdgcn_mfma_i32_32x32x32_i8(kf.f[kh][k4], qf.f[k4], s[kh], 0, 0, 0);
    }
  }
}

// Everything one wave needs for the quantized segment.
struct SegA {
  const uint8_t* kc0;
  const uint8_t* vc0;
  const int32_t* kq0;
  const float* ks0;
  const float* vs0;
  int n;              // quantized tiles to scan, of which this group takes
  int grp;            // grp, grp + S, ...
  int t0;             // first query row of the wave
  float cq;           // alpha * log2(e) * s_Q
  float inv_vref;
  int lane, half, col;
};

// K codes and metadata of tile tk, V codes of tile tv.
template <int BITS, int NT>
__device__ __forceinline__ void stage_load(StageRegs<BITS, NT>& r, const SegA& a, int tk, int tv,
                                           int tid) {
  constexpr int kRow = BITS == 8 ? kHeadDim : kHeadDim / 2;
  constexpr int vRow = BITS == 8 ? kTile : kTile / 2;
  constexpr int n = chunks_per_thread<BITS, NT>();
  const int t = tk;
  const v4u* kc = reinterpret_cast<const v4u*>(a.kc0 + (size_t)tk * kTile * kRow);
  const v4u* vc = reinterpret_cast<const v4u*>(a.vc0 + (size_t)tv * kHeadDim * vRow);
#pragma unroll
  for (int i = 0; i < n; ++i) r.k[i] = kc[chunk_id<BITS, NT>(tid, i)];
#pragma unroll
  for (int i = 0; i < n; ++i) r.v[i] = vc[chunk_id<BITS, NT>(tid, i)];
  // wave 0: kq_pos; wave 1: lane 0 sK, lane 1 sV; the rest reload sV
  // (choices uniform per wave or between two uniform addresses: no branch)
  const int w = tid >> 6, lane = tid & 63;
  const int32_t* pk = a.kq0 + (size_t)t * kTile + lane;
  const int32_t* psk = reinterpret_cast<const int32_t*>(a.ks0 + t);
  const int32_t* psv = reinterpret_cast<const int32_t*>(a.vs0 + t);
  const int32_t* ps = (w == 1 && lane == 0) ? psk : psv;
  r.meta = *(w == 0 ? pk : ps);
}

// int8 K: chunk q = row*8 + j goes to the swizzled slot of (row, j).  4-bit
// K: chunk tid holds 32 channels of row tid/4, expanded to int8 (16*code)
// and stored as two chunks.  V: f16 [128][kVPitch] in the permuted key order.
template <int BITS, int FMT, int NT>
__device__ __forceinline__ void stage_store(KBuf& kb, VBuf& vb, const StageRegs<BITS, NT>& r, int tid,
                                            const VScale& vs) {
  if (BITS == 8) {
#pragma unroll
    for (int i = 0; i < chunks_per_thread<BITS, NT>(); ++i) {
      const int q = chunk_id<BITS, NT>(tid, i);
      *reinterpret_cast<v4u*>(kb.k + kswz(q >> 3, q & 7)) = r.k[i];
    }
#pragma unroll
    for (int i = 0; i < chunks_per_thread<BITS, NT>(); ++i) {
      const int q = chunk_id<BITS, NT>(tid, i);
      const int d = q >> 2, kg = q & 3;   // channel d, keys kg*16 .. +16
      const v4u w = r.v[i];
      uint32_t h[8];
      codes4_to_h<FMT>(w.x, h[0], h[1], vs);   // keys 0..3
      codes4_to_h<FMT>(w.y, h[2], h[3], vs);   // keys 4..7
      codes4_to_h<FMT>(w.z, h[4], h[5], vs);   // keys 8..11
      codes4_to_h<FMT>(w.w, h[6], h[7], vs);   // keys 12..15
      uint8_t* dst = vb.v + d * kVPitch + kg * 32;
      *reinterpret_cast<v4u*>(dst) = v4u{h[0], h[1], h[4], h[5]};
      *reinterpret_cast<v4u*>(dst + 16) = v4u{h[2], h[3], h[6], h[7]};
    }
  } else if constexpr (kv_fp4(FMT)) {
    // E2M1 K: the 16-byte chunk as it is (the MFMA reads 4-bit operands);
    // V: E2M1 -> f16 times 2^e, two codes per conversion, exact
    const int q4 = chunk_id<BITS, NT>(tid, 0);
    *reinterpret_cast<v4u*>(kb.k + kswz4(q4 >> 2, q4 & 3)) = r.k[0];
    const int d = q4 >> 1, kh = q4 & 1;   // channel d, keys kh*32 .. +32 (16 B packed)
    const v4u w = r.v[0];
    const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int g16 = 0; g16 < 2; ++g16) {
      uint32_t h[8];   // h[e]: keys 2e, 2e + 1 of the 16
      e2m1x8_to_h(ww[2 * g16], *reinterpret_cast<uint32_t(*)[4]>(&h[0]), vs.f32);
      e2m1x8_to_h(ww[2 * g16 + 1], *reinterpret_cast<uint32_t(*)[4]>(&h[4]), vs.f32);
      uint8_t* dst = vb.v + d * kVPitch + (kh * 2 + g16) * 32;
      *reinterpret_cast<v4u*>(dst) = v4u{h[0], h[1], h[4], h[5]};
      *reinterpret_cast<v4u*>(dst + 16) = v4u{h[2], h[3], h[6], h[7]};
    }
  } else {
    const int q4 = chunk_id<BITS, NT>(tid, 0);
    {
      const int row = q4 >> 2, j4 = q4 & 3;
      const v4u w = r.k[0];
      uint32_t o[8];
      i4x8_to_i8(w.x, o[0], o[1]);
      i4x8_to_i8(w.y, o[2], o[3]);
      i4x8_to_i8(w.z, o[4], o[5]);
      i4x8_to_i8(w.w, o[6], o[7]);
      *reinterpret_cast<v4u*>(kb.k + kswz(row, 2 * j4)) = v4u{o[0], o[1], o[2], o[3]};
      *reinterpret_cast<v4u*>(kb.k + kswz(row, 2 * j4 + 1)) = v4u{o[4], o[5], o[6], o[7]};
    }
    const int d = q4 >> 1, kh = q4 & 1;   // channel d, keys kh*32 .. +32 (16 B packed)
    const v4u w = r.v[0];
    const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int g16 = 0; g16 < 2; ++g16) {
      uint32_t bb[4];
      i4x8_to_i8(ww[2 * g16], bb[0], bb[1]);
      i4x8_to_i8(ww[2 * g16 + 1], bb[2], bb[3]);
      uint32_t h[8];
      i8x4_to_h(bb[0], h[0], h[1], vs);
      i8x4_to_h(bb[1], h[2], h[3], vs);
      i8x4_to_h(bb[2], h[4], h[5], vs);
      i8x4_to_h(bb[3], h[6], h[7], vs);
      uint8_t* dst = vb.v + d * kVPitch + (kh * 2 + g16) * 32;
      *reinterpret_cast<v4u*>(dst) = v4u{h[0], h[1], h[4], h[5]};
      *reinterpret_cast<v4u*>(dst + 16) = v4u{h[2], h[3], h[6], h[7]};
    }
  }
  const int w = tid >> 6, lane = tid & 63;
  kb.pos[w == 0 ? lane : (w == 1 ? min(kMetaSK + lane, kMetaSink) : kMetaSink)] = r.meta;
}

// The full-precision key list of a workgroup: nvl vertical lines (idx, seen
// from their position on), then nqb quantizable keys of the per-query band
// (kq[nq0 ..], each seen by the W rows from its position on), then the
// window positions base .. (seen from their position on; in band mode by W
// rows, which is every later row).  Entries at or beyond `count` are padding
// (position HYQ_KQ_POS_PAD, seen by no row, zero rows).
struct FpList {
  const int32_t* vl;
  const int32_t* kq;
  const int32_t* dummy;   // any readable word (entries whose position is computed)
  int nvl, nq0, nqb, base, count, band_w;
};
// Entry e's position comes from a load (vertical lines, band keys) or is
// computed (window); fp_src gives the word to load, always readable, and
// fp_resolve turns the loaded word into (position, last row).
__device__ __forceinline__ const int32_t* fp_src(const FpList& f, int e) {
  return e < f.nvl ? f.vl + e : (e < f.nvl + f.nqb ? f.kq + (f.nq0 + (e - f.nvl)) : f.dummy);
}
__device__ __forceinline__ void fp_resolve(const FpList& f, int e, int32_t w, int& p, int& hi) {
  if (e >= f.count) {
    p = HYQ_KQ_POS_PAD;
    hi = -1;
  } else if (e < f.nvl) {
    p = w;
    hi = INT32_MAX;
  } else if (e < f.nvl + f.nqb) {
    p = w;
    hi = w + f.band_w - 1;
  } else {
    p = f.base + (e - f.nvl - f.nqb);
    hi = f.band_w > 0 ? p + f.band_w - 1 : INT32_MAX;
  }
}

// A full-precision tile in registers.  K: thread tid holds the 16-byte
// chunks q = tid + i * NT (key q / 16, channels 8 * (q % 16) ..), with
// the key's position and last row.  V: item q = tid + i * NT is the
// chunk q / 32 of the key pair (2 * (q % 32), +1), so that one LDS store
// writes both keys of a channel (adjacent V^T slots) and the 64 lanes of a
// wave (32 pairs, two chunks) hit distinct banks.  Also the position words of
// the same keys of the following tile.
// Thread index within its group of NT threads (a workgroup is one or two groups).
template <int NT>
__device__ __forceinline__ int group_tid() { return (int)threadIdx.x & (NT - 1); }
template <int NT>
struct FpRegs {
  static constexpr int kPairs = kTile * 16 / NT, kVItems = (kTile / 2) * 16 / NT;
  static_assert((kTile * 16) % NT == 0 && ((kTile / 2) * 16) % NT == 0,
                "full-precision chunks must split evenly");
  v4u k[kPairs], v[2 * kVItems];
  int32_t pos[kPairs], hi[kPairs], vpos[2 * kVItems];
  int32_t wnext[kPairs], vwnext[2 * kVItems];
};
template <int NT>
__device__ __forceinline__ int fp_kkey(int i) { return (group_tid<NT>() + i * NT) >> 4; }
template <int NT>
__device__ __forceinline__ int fp_vkey(int i, int s) {
  return 2 * ((group_tid<NT>() + i * NT) & 31) + s;
}
template <int NT>
__device__ __forceinline__ int fp_vchunk(int i) { return (group_tid<NT>() + i * NT) >> 5; }

// Position words of tile ft (before its first fp_load).
template <int NT>
__device__ __forceinline__ void fp_load_words(FpRegs<NT>& r, const FpList& f, int ft) {
#pragma unroll
  for (int i = 0; i < FpRegs<NT>::kPairs; ++i) r.wnext[i] = *fp_src(f, ft * kTile + fp_kkey<NT>(i));
#pragma unroll
  for (int i = 0; i < FpRegs<NT>::kVItems; ++i)
#pragma unroll
    for (int s = 0; s < 2; ++s) r.vwnext[2 * i + s] = *fp_src(f, ft * kTile + fp_vkey<NT>(i, s));
}

// Load the rows of tile ft (padding rows read row 0, zeroed at the store)
// from the position words loaded earlier, then the words of the group's next
// tile ft + S.
// Tiles past the end are all padding.
template <int NT, int S>
__device__ __forceinline__ void fp_load(FpRegs<NT>& r, const FpList& f, const uint16_t* __restrict__ Kh,
                                        const uint16_t* __restrict__ Vh, int ft, int L) {
#pragma unroll
  for (int i = 0; i < FpRegs<NT>::kPairs; ++i) {
    int p, hi;
    fp_resolve(f, ft * kTile + fp_kkey<NT>(i), r.wnext[i], p, hi);
    r.pos[i] = p;
    r.hi[i] = hi;
    const size_t row = (unsigned)p < (unsigned)L ? (size_t)p : 0;
    r.k[i] = reinterpret_cast<const v4u*>(Kh + row * kHeadDim)[(group_tid<NT>() + i * NT) & 15];
  }
#pragma unroll
  for (int i = 0; i < FpRegs<NT>::kVItems; ++i)
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      int p, hi;
      fp_resolve(f, ft * kTile + fp_vkey<NT>(i, s), r.vwnext[2 * i + s], p, hi);
      r.vpos[2 * i + s] = p;
      const size_t row = (unsigned)p < (unsigned)L ? (size_t)p : 0;
      r.v[2 * i + s] = reinterpret_cast<const v4u*>(Vh + row * kHeadDim)[fp_vchunk<NT>(i)];
    }
  fp_load_words<NT>(r, f, ft + S);
}

// V^T stores of one key pair (adjacent slots from `slot` on) and one
// 16-byte chunk: channel d gets the 32-bit word (f16 of key 2m, of key 2m+1)
// of V / sVref (sVref a power of two: exact for bf16 values of that range,
// down to the f16 subnormals).  Returns the largest |V| of the pair's chunk.
__device__ __forceinline__ float fp_store_vpair(uint8_t* vt, v4u v0, v4u v1, int slot, int chunk,
                                                float inv_vref) {
  float mx = 0.0f;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int d = chunk * 8 + 2 * j;
    const float a0 = __uint_as_float(v0[j] << 16), a1 = __uint_as_float(v1[j] << 16);
    const float b0 = __uint_as_float(v0[j] & 0xffff0000u), b1 = __uint_as_float(v1[j] & 0xffff0000u);
    mx = fmaxf(mx, fmaxf(fabsf(a0), fabsf(a1)));
    mx = fmaxf(mx, fmaxf(fabsf(b0), fabsf(b1)));
    const v2f lo = {a0 * inv_vref, a1 * inv_vref}, hi = {b0 * inv_vref, b1 * inv_vref};
    *reinterpret_cast<v2h*>(vt + d * kVPitch + slot * 2) = __builtin_convertvector(lo, v2h);
    *reinterpret_cast<v2h*>(vt + (d + 1) * kVPitch + slot * 2) = __builtin_convertvector(hi, v2h);
  }
  return mx;
}

// Write a loaded tile to LDS: K rows as bf16, V^T as f16 V / sVref,
// positions and last rows.  A V ratio outside the f16 range records
// (tile << 8) | (largest biased exponent of |V|) in ovf (a NaN is not
// recorded: it stays a NaN in f16).
template <int NT>
__device__ __forceinline__ void fp_store(FBuf& b, const FpRegs<NT>& r, float inv_vref, int tag, int L) {
#pragma unroll
  for (int i = 0; i < FpRegs<NT>::kPairs; ++i) {
    const int e = fp_kkey<NT>(i), col = (group_tid<NT>() + i * NT) & 15;
    const unsigned keep = (unsigned)r.pos[i] < (unsigned)L ? 0xffffffffu : 0u;
    *reinterpret_cast<v4u*>(b.k + e * kKPitchBf + col * 16) = r.k[i] & keep;
    if (col == 0) {
      b.pos[e] = r.pos[i];
      b.hi[e] = r.hi[i];
    }
  }
  float mx = 0.0f;
#pragma unroll
  for (int i = 0; i < FpRegs<NT>::kVItems; ++i) {
    const unsigned k0 = (unsigned)r.vpos[2 * i] < (unsigned)L ? 0xffffffffu : 0u;
    const unsigned k1 = (unsigned)r.vpos[2 * i + 1] < (unsigned)L ? 0xffffffffu : 0u;
    mx = fmaxf(mx, fp_store_vpair(b.v, r.v[2 * i] & k0, r.v[2 * i + 1] & k1,
                                  vslot(fp_vkey<NT>(i, 0)), fp_vchunk<NT>(i), inv_vref));
  }
  if (!(mx * inv_vref <= 65504.0f)) atomicMax(&b.ovf, (tag << 8) | (int)(__float_as_uint(mx) >> 23));
}

// Rewrite the V^T of a published tile with a new sVref (positions from LDS).
template <int NT>
__device__ __forceinline__ void fp_restage_v(FBuf& b, const uint16_t* __restrict__ Vh, int L,
                                             float inv_vref) {
#pragma unroll
  for (int i = 0; i < FpRegs<NT>::kVItems; ++i) {
    v4u vw[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int p = b.pos[fp_vkey<NT>(i, s)];
      vw[s] = v4u{0u, 0u, 0u, 0u};
      if ((unsigned)p < (unsigned)L)
        vw[s] = reinterpret_cast<const v4u*>(Vh + (size_t)p * kHeadDim)[fp_vchunk<NT>(i)];
    }
    fp_store_vpair(b.v, vw[0], vw[1], vslot(fp_vkey<NT>(i, 0)), fp_vchunk<NT>(i), inv_vref);
  }
}

// Visibility of this lane's 32 keys of a full-precision tile to row tq, bit
// kh * 16 + r for accumulator register r of half-tile kh.  Without the band
// every listed key is seen from its position on (padding has a position
// past every row), so only the positions are read.
__device__ __forceinline__ uint32_t fp_vis_mask(const FBuf& b, int tq, int half, bool band) {
  uint32_t m = 0;
#pragma unroll
  for (int kh = 0; kh < 2; ++kh)
#pragma unroll
    for (int rg = 0; rg < 4; ++rg) {
      const int e = kh * 32 + rg * 8 + half * 4;
      const v4i p4 = *reinterpret_cast<const v4i*>(&b.pos[e]);
#pragma unroll
      for (int j = 0; j < 4; ++j) m |= (uint32_t)(p4[j] <= tq) << (kh * 16 + rg * 4 + j);
    }
  if (band) {
    uint32_t mh = 0;
#pragma unroll
    for (int kh = 0; kh < 2; ++kh)
#pragma unroll
      for (int rg = 0; rg < 4; ++rg) {
        const int e = kh * 32 + rg * 8 + half * 4;
        const v4i h4 = *reinterpret_cast<const v4i*>(&b.hi[e]);
#pragma unroll
        for (int j = 0; j < 4; ++j) mh |= (uint32_t)(tq <= h4[j]) << (kh * 16 + rg * 4 + j);
      }
    m &= mh;
  }
  return m;
}

// Online-softmax state of one 32-query block of a wave (each lane owns one
// query and the keys of its half of every 32-key group).
struct NState {
  float m;        // reference max (log2 domain); the true max is <= m + kLazy
  float l;        // this lane's part of the row sum, relative to m
  float corr;     // rescale of acc still to apply: 2^(m_before - m)
  v16f acc[4];    // O^T accumulator, 4 groups of 32 channels
};

__device__ __forceinline__ void init_state(NState& st) {
  st.m = kMinusBig;
  st.l = 0.0f;
  st.corr = 1.0f;
#pragma unroll
  for (int dg = 0; dg < 4; ++dg)
#pragma unroll
    for (int r = 0; r < 16; ++r) st.acc[dg][r] = 0.0f;
}

// Key index (0..63) of accumulator register r of half-tile kh for this lane.
__device__ __forceinline__ int key_of(int kh, int r, int half) {
  return kh * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
}

// Raise the reference max of every lane of the wave when some lane's tile
// max exceeds it by more than kLazy (2^kLazy bounds the unnormalized
// weights).  Branch-free: the row sum is rescaled now, the accumulator before
// the next P V product that adds to it.
__device__ __forceinline__ void lazy_max(NState& ns, float mt) {
  const bool any = __ballot(mt > ns.m + kLazy) != 0;
  const float mn = any ? fmaxf(ns.m, mt) : ns.m;
  const float c = __builtin_amdgcn_exp2f(ns.m - mn);   // 1 when unchanged
  ns.l *= c;
  ns.corr = c;
  ns.m = mn;
}

__device__ __forceinline__ void apply_corr(NState& ns) {
  if (__ballot(ns.corr != 1.0f)) {
#pragma unroll
    for (int dg = 0; dg < 4; ++dg)
#pragma unroll
      for (int r = 0; r < 16; ++r) ns.acc[dg][r] *= ns.corr;
  }
  ns.corr = 1.0f;
}

// General path: causal mask by original position, or a tile whose maximum
// outgrew the reference max.  Raises m to the masked tile
// maximum when needed and rescales l and the accumulator at once (the
// accumulator already holds every P V product of earlier tiles).  No
// per-lane branches, so the cross-lane swap sees every lane's operand; the
// visibility test is evaluated twice rather than kept in registers.
template <typename SV>
__device__ __forceinline__ void softmax_general(NState& ns, const SV (&s)[2], v8h (&p)[4],
                                             float cqk, float fm, bool diag, const int32_t* pos,
                                             int tq, int half) {
  float mx = -INFINITY;
#pragma unroll
  for (int kh = 0; kh < 2; ++kh)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const bool vis = (!diag) | (pos[key_of(kh, r, half)] <= tq);
      mx = fmaxf(mx, vis ? (float)s[kh][r] : -INFINITY);
    }
  mx = xhalf_max(mx);
  lazy_max(ns, mx == -INFINITY ? -INFINITY : mx * cqk);
  apply_corr(ns);
  // the row sum adds the same f16 weights the MFMA uses, divided by fm
  float ps = 0.0f;
#pragma unroll
  for (int kh = 0; kh < 2; ++kh)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const bool vis = (!diag) | (pos[key_of(kh, r, half)] <= tq);
      const float ex = __builtin_amdgcn_exp2f((float)s[kh][r] * cqk - ns.m);
      const _Float16 hp = (_Float16)((vis ? ex : 0.0f) * fm);
      ps += (float)hp;
      p[kh * 2 + (r >> 3)][r & 7] = hp;
    }
  ns.l += ps * __builtin_amdgcn_rcpf(fm);
}

// Softmax of one full-precision tile (logits of hidden keys already -inf):
// raise the reference max when the tile's exceeds it by more than kLazy,
// weights 2^(s * alpha * log2(e) - m) as f16 into p (the B operands of P V),
// and their f16 sum into the row sum.  alpha > 0, so the tile max of the
// scaled logits is the scaled max of the raw ones.
__device__ __forceinline__ void fp_softmax(NState& st, const v16f (&sf)[2], float alpha_log2e,
                                           v8h (&p)[4]) {
  float mx = -INFINITY;
#pragma unroll
  for (int kh = 0; kh < 2; ++kh)
#pragma unroll
    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sf[kh][r]);
  lazy_max(st, xhalf_max(mx) * alpha_log2e);
  apply_corr(st);
  const v2h one2 = {(_Float16)1.0f, (_Float16)1.0f};
  float ps = 0.0f;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int kh = i >> 3, r = (i & 7) * 2;
    v2f e;
    e[0] = __builtin_amdgcn_exp2f(__builtin_fmaf(sf[kh][r], alpha_log2e, -st.m));
    e[1] = __builtin_amdgcn_exp2f(__builtin_fmaf(sf[kh][r + 1], alpha_log2e, -st.m));
    const v2h pk = __builtin_convertvector(e, v2h);
    ps = __builtin_amdgcn_fdot2(pk, one2, ps, false);
    p[kh * 2 + (r >> 3)][r & 7] = pk[0];
    p[kh * 2 + (r >> 3)][(r & 7) + 1] = pk[1];
  }
  st.l += ps;
}

// One tile of the quantized segment:
//   publish tile c+1 (registers -> LDS) and load tile c+2 into registers;
//   S^T of tile c (int8 MFMA);
//   P V of tile c-1 (weights pprev; zeros when c = 0) interleaved with the
//   fast-path softmax of tile c -> pcur;
//   the general path instead when the tile touches the diagonal, its V
//   scale ratio is tiny, or some weight overflowed the fast-path bound.
// The accumulator never carries a pending rescale between tiles: only the
// general path moves the reference max, and it rescales on the spot.
// PH = c % 4 is a template argument so that every LDS address is a per-lane
// constant plus an immediate offset.
template <int BITS, int FMT, int NT, int S, int PH>
__device__ __forceinline__ void segA_tile(Smem& sm, const SegA& a, int c, const QFrag<FMT>& qf,
                                          NState& st, const v8h (&pprev)[4], v8h (&pcur)[4],
                                          StageRegs<BITS, NT>& sr, KFrag<FMT>& kf) {
  // 4-bit integer codes are staged as 16*code
  constexpr float kSub = (BITS == 8 || kv_fp4(FMT)) ? 1.0f : 0.0625f;
  const int tid = group_tid<NT>();
  // the group's c-th tile; past the end (loads, and with S = 2 the whole last
  // step of the second group) the last tile again, in that step all hidden
  auto tile = [&](int i) { return min(i * S + a.grp, a.n - 1); };
  const bool dead = S > 1 && c * S + a.grp >= a.n;
  const KBuf& cur = sm.q.kb[PH];
  const VBuf& prv = sm.q.vb[(PH + 1) & 1];
  const float sk = __int_as_float(cur.pos[kMetaSK]) * kSub;
  const float sv = __int_as_float(cur.pos[kMetaSV]) * kSub;
  const int last = __builtin_amdgcn_readfirstlane(cur.pos[kTile - 1]);
  // sV / sVref = fm * 2^ev (sVref a power of two: the product is exact)
  int ev;
  float fm = __builtin_frexpf(sv * a.inv_vref, &ev);
  if (!(sv > 0.0f)) {   // all-zero V block: its V codes are 0, fold nothing
    fm = 1.0f;
    ev = 0;
  }
  const VScale vs = make_vscale(__builtin_ldexpf(1.0f, ev));

  // S^T of tile c (its K fragments arrived during the previous tile)
  SVec<FMT> s[2];
  qk_tile<FMT>(s, kf, qf);
  // publish K(c+2) and V(c) (registers loaded during tile c-1) and load K(c+3)
  // and V(c+1); the conversion runs in the shadow of the MFMAs above.  Past
  // the end the last tile is staged again into the free buffers (no branch).
  stage_store<BITS, FMT, NT>(sm.q.kb[(PH + 2) % kKRing], sm.q.vb[PH & 1], sr, tid, vs);
  stage_load<BITS, NT>(sr, a, tile(c + 3), tile(c + 1), tid);

  // Fast path: weights against the current reference max, without the tile
  // max; accepted unless some lane's weights sum above kFastMax (then some
  // weight may have left the f16 range).  Step i issues the MFMA of
  // (channel group i%4, key group i/4) of P V(c-1) and the weight pair i.
  const float cqk = a.cq * sk;
  const float bias = __builtin_amdgcn_logf(fm) - st.m;   // log2
  const v2h one2 = {(_Float16)1.0f, (_Float16)1.0f};
  // The wave in this loop issues ahead of its SIMD partner while that one
  // stages and runs its S^T MFMAs (measured: 1-2% faster than equal
  // priorities; raising the S^T part instead is slower).
  __builtin_amdgcn_s_setprio(1);
  float ps = 0.0f;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int dg = i & 3, ks = i >> 2;
    const v8h va = *reinterpret_cast<const v8h*>(prv.v + (dg * 32 + a.col) * kVPitch + ks * 32 +
                                                 a.half * 16);
    st.acc[dg] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va, pprev[ks], st.acc[dg], 0, 0, 0);
    const int kh = i >> 3, r = (i & 7) * 2;
    const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf((float)s[kh][r], cqk, bias));
    const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf((float)s[kh][r + 1], cqk, bias));
    v2h pk;
    pk[0] = (_Float16)p0;
    pk[1] = (_Float16)p1;
    ps = __builtin_amdgcn_fdot2(pk, one2, ps, false);
    pcur[kh * 2 + (r >> 3)][r & 7] = pk[0];
    pcur[kh * 2 + (r >> 3)][(r & 7) + 1] = pk[1];
  }
  // keep the fast-path weights computed here, next to the MFMAs, rather
  // than sunk into the branch below that consumes them
  asm volatile("" : "+v"(pcur[0]), "+v"(pcur[1]), "+v"(pcur[2]), "+v"(pcur[3]), "+v"(ps));
  __builtin_amdgcn_s_setprio(0);
  const bool diag = dead || last > a.t0;
  const bool redo = diag || __ballot(!(ps <= kFastMax)) != 0;
  if (redo) {
    softmax_general(st, s, pcur, cqk, fm, diag, cur.pos, dead ? -1 : a.t0 + a.col, a.half);
  } else {
    st.l = __builtin_fmaf(ps, __builtin_amdgcn_rcpf(fm), st.l);   // 1-ulp reciprocal
  }
  // K fragments of tile c+1 (published by the previous barrier); past the
  // end they read a staged copy and are not used
  read_kfrag<FMT>(kf, sm.q.kb[(PH + 1) % kKRing], a.col, a.half);
  __syncthreads();
}

// ---------------------------------------------------------------------------
// Every key in full precision (bits 16): consecutive rows, so no key list, and
// the quantized segment's pipeline.  Tile c: S^T(c) with the bf16 MFMA; K(c+1)
// and V(c) from registers to LDS (V converted to f16 V / sVref and transposed)
// and the loads of K(c+2), V(c+1) in its shadow; then P V(c-1) interleaved
// with the fast-path softmax of tile c.  One barrier per tile.  What bounds
// it is the chip's power under matrix work, then vector instructions (about
// 170 per tile and wave beside 32 MFMAs; the key-list stage, which computes
// each row's position, tile maximum and visibility and runs its products and
// its softmax one after the other, takes 296).  GQA 32q/8kv at 32k: 9.47 ms
// with the key-list stage, 8.33 ms (1056 TFLOP/s) here; at 8k 622 and 549 us.
// ---------------------------------------------------------------------------
struct SegD {
  const uint8_t* k0;
  const uint8_t* v0;
  int n, grp;
  int rows;           // keys that some row of the workgroup sees: [0, rows)
  int t0;             // first query row of the wave
  float alpha_log2e;
  int half, col;
};
template <int NT>
struct DenseRegs {
  static constexpr int kK = kTile * 16 / NT, kV = (kTile / 2) * 16 / NT;
  v4u k[kK], v[2 * kV];
};
// 16-byte chunk of a row of tile t.  Past the workgroup's last row, that row
// again: a row that none of the queries sees must not be read, for its V meets
// a zero weight (0 * inf) and takes part in the choice of sVref.
__device__ __forceinline__ v4u dense_chunk(const uint8_t* base, int t, int key, int chunk, int rows) {
  const uint32_t row = (uint32_t)min(t * kTile + key, rows - 1);
  return *reinterpret_cast<const v4u*>(base + (size_t)(row * (uint32_t)(kHeadDim * 2) + chunk * 16));
}
template <int NT>
__device__ __forceinline__ void dense_load_k(DenseRegs<NT>& r, const SegD& a, int t) {
#pragma unroll
  for (int i = 0; i < DenseRegs<NT>::kK; ++i)
    r.k[i] = dense_chunk(a.k0, t, fp_kkey<NT>(i), (group_tid<NT>() + i * NT) & 15, a.rows);
}
template <int NT>
__device__ __forceinline__ void dense_load_v(DenseRegs<NT>& r, const SegD& a, int t) {
#pragma unroll
  for (int i = 0; i < DenseRegs<NT>::kV; ++i)
#pragma unroll
    for (int x = 0; x < 2; ++x)
      r.v[2 * i + x] = dense_chunk(a.v0, t, fp_vkey<NT>(i, x), fp_vchunk<NT>(i), a.rows);
}
template <int NT>
__device__ __forceinline__ void dense_store_k(uint8_t* kb, const DenseRegs<NT>& r) {
#pragma unroll
  for (int i = 0; i < DenseRegs<NT>::kK; ++i)
    *reinterpret_cast<v4u*>(kb + fp_kkey<NT>(i) * kKPitchBf +
                            ((group_tid<NT>() + i * NT) & 15) * 16) = r.k[i];
}
// V of tile t; a ratio outside the f16 range is recorded as fp_store does.
template <int NT>
__device__ __forceinline__ void dense_store_v(VBuf& vb, int32_t& ovf, const DenseRegs<NT>& r, int t,
                                              float inv_vref) {
  float mx = 0.0f;
#pragma unroll
  for (int i = 0; i < DenseRegs<NT>::kV; ++i)
    mx = fmaxf(mx, fp_store_vpair(vb.v, r.v[2 * i], r.v[2 * i + 1], vslot(fp_vkey<NT>(i, 0)),
                                  fp_vchunk<NT>(i), inv_vref));
  if (!(mx * inv_vref <= 65504.0f)) atomicMax(&ovf, (t << 8) | (int)(__float_as_uint(mx) >> 23));
}

// V(c-1), staged one tile ago, outside the f16 range at the sVref of then:
// raise sVref to 2^(E - 134) (every |V| / sVref of the tile below 2^8),
// rescale the accumulator (exact) and stage that tile's V again (also for the
// last tile that an all-hidden step staged in its place: its zero weights must
// not meet an infinity).  Uniform over the workgroup; with S = 2 the barrier
// is for both groups.
template <int NT, int S>
__device__ __forceinline__ void dense_check_v(Smem (&sms)[S], const SegD& a, int c, NState& st,
                                              float& vref, float& inv_vref) {
  DRing& d = sms[a.grp].d;
  const int b = c & 1, t = min(c * S + a.grp, a.n - 1), ov = d.ovf[b];
  const bool mine = (ov >> 8) == t;
  bool any = false;   // S = 2: either group's tile
  if (S == 2) {
    const int o = S - 1 - a.grp;
    any = mine || (sms[o].d.ovf[b] >> 8) == min(c * S + o, a.n - 1);
  }
  if (mine) {
    const float nv = fmaxf(vref, __builtin_ldexpf(1.0f, max(-100, (ov & 0xff) - 134)));
    const float f = vref / nv;
#pragma unroll
    for (int dg = 0; dg < 4; ++dg)
#pragma unroll
      for (int r = 0; r < 16; ++r) st.acc[dg][r] *= f;
    vref = nv;
    inv_vref = 1.0f / nv;
    DenseRegs<NT> again;
    dense_load_v<NT>(again, a, t);
#pragma unroll
    for (int i = 0; i < DenseRegs<NT>::kV; ++i)
      fp_store_vpair(d.vb[b].v, again.v[2 * i], again.v[2 * i + 1], vslot(fp_vkey<NT>(i, 0)),
                     fp_vchunk<NT>(i), inv_vref);
    if (S == 1) __syncthreads();
  }
  if (any) __syncthreads();
}

template <int NT, int S, int PH>
__device__ __forceinline__ void segD_tile(Smem (&sms)[S], const SegD& a, int c, const v8bf (&qb)[8],
                                          NState& st, const v8h (&pprev)[4], v8h (&pcur)[4],
                                          DenseRegs<NT>& dr, float& vref, float& inv_vref) {
  DRing& d = sms[a.grp].d;
  auto tile = [&](int i) { return min(i * S + a.grp, a.n - 1); };
  const bool dead = S > 1 && c * S + a.grp >= a.n;
  const uint8_t* kb = d.k[PH];
  v16f s[2];
#pragma unroll
  for (int kh = 0; kh < 2; ++kh) {
    s[kh] = v16f{};
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const v8bf ka = *reinterpret_cast<const v8bf*>(kb + (kh * 32 + a.col) * kKPitchBf + ks * 32 +
                                                     a.half * 16);
      s[kh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qb[ks], s[kh], 0, 0, 0);
    }
  }
  if (c > 0) dense_check_v<NT, S>(sms, a, c - 1, st, vref, inv_vref);
  dense_store_k<NT>(d.k[PH ^ 1], dr);
  dense_store_v<NT>(d.vb[PH], d.ovf[PH], dr, tile(c), inv_vref);
  dense_load_k<NT>(dr, a, tile(c + 2));
  dense_load_v<NT>(dr, a, tile(c + 1));
  const VBuf& prv = d.vb[PH ^ 1];
  const v2h one2 = {(_Float16)1.0f, (_Float16)1.0f};
  __builtin_amdgcn_s_setprio(1);
  float ps = 0.0f;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int dg = i & 3, ks = i >> 2;
    const v8h va = *reinterpret_cast<const v8h*>(prv.v + (dg * 32 + a.col) * kVPitch + ks * 32 +
                                                 a.half * 16);
    st.acc[dg] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va, pprev[ks], st.acc[dg], 0, 0, 0);
    const int kh = i >> 3, r = (i & 7) * 2;
    v2h pk;
    pk[0] = (_Float16)__builtin_amdgcn_exp2f(__builtin_fmaf(s[kh][r], a.alpha_log2e, -st.m));
    pk[1] = (_Float16)__builtin_amdgcn_exp2f(__builtin_fmaf(s[kh][r + 1], a.alpha_log2e, -st.m));
    ps = __builtin_amdgcn_fdot2(pk, one2, ps, false);
    pcur[kh * 2 + (r >> 3)][r & 7] = pk[0];
    pcur[kh * 2 + (r >> 3)][(r & 7) + 1] = pk[1];
  }
  // keep the fast-path weights next to the MFMAs (see segA_tile)
  asm volatile("" : "+v"(pcur[0]), "+v"(pcur[1]), "+v"(pcur[2]), "+v"(pcur[3]), "+v"(ps));
  __builtin_amdgcn_s_setprio(0);
  const int p0 = (c * S + a.grp) * kTile;   // position of the tile's first key
  if (dead || p0 + kTile - 1 > a.t0 || __ballot(!(ps <= kFastMax)) != 0) {
    const int last = dead ? -1 : a.t0 + a.col - p0;   // last key of the tile the row sees
#pragma unroll
    for (int kh = 0; kh < 2; ++kh)
#pragma unroll
      for (int r = 0; r < 16; ++r) s[kh][r] = key_of(kh, r, a.half) <= last ? s[kh][r] : -INFINITY;
    fp_softmax(st, s, a.alpha_log2e, pcur);
  } else {
    st.l += ps;
  }
  __syncthreads();
}

// Which keys the rows [t_first, t_last] of a workgroup see, and the reference
// sVref of their head's V scales.  A quantized key at position p is seen by
// rows t >= p + shift: shift = 0 for the fixed window, W for the per-query
// band (whose rows see p in full precision instead).
struct KeyPlan {
  int shift, nvl, nq_tiles, fp_count, fp_base, nq0, nqb;
  float vref;
};
template <int BITS, int FMT>
__device__ __forceinline__ KeyPlan key_plan(const int32_t* __restrict__ vl,
                                            const float* __restrict__ v_scale, int k, int P, int nQ,
                                            int n_kvblk, int t_first, int t_last, int band_w) {
  KeyPlan pl;
  pl.shift = BITS == 16 ? 0 : band_w;
  pl.nq0 = pl.nqb = 0;
  pl.vref = 1.0f;
  if (BITS == 16) {
    pl.nvl = 0;
    pl.nq_tiles = 0;
    pl.fp_base = 0;
    pl.fp_count = t_last + 1;
    return pl;
  }
  const int lane = threadIdx.x & 63;
  pl.nvl = count_le(vl, k, t_last);
  const int tq_last = t_last - pl.shift;        // last quantized position any row sees
  // (for the fixed window tq_last = t_last: the count is nvl, no second search)
  const int nq_vis = tq_last < 0 ? 0 : (tq_last < P ? (tq_last + 1) -
                                        (pl.shift == 0 ? pl.nvl : count_le(vl, k, tq_last)) : nQ);
  pl.nq_tiles = min((nq_vis + kTile - 1) / kTile, n_kvblk);
  pl.fp_base = P;
  if (band_w > 0) {
    // band keys of the workgroup's rows: positions [lo, t_last], lo from its first row
    const int lo = max(0, t_first + 1 - band_w);
    const int hi_q = min(t_last, P - 1);    // quantizable band keys: non-vertical in [lo, hi_q]
    if (lo <= hi_q) {
      pl.nq0 = lo - count_le(vl, k, lo - 1);    // non-vertical positions below lo
      pl.nqb = (hi_q + 1) - count_le(vl, k, hi_q) - pl.nq0;
    }
    pl.fp_base = max(P, lo);
  }
  pl.fp_count = pl.nvl + pl.nqb + max(0, t_last + 1 - pl.fp_base);
  // sVref: smallest power of two >= every V scale of this head
  float mx = 0.0f;
  for (int i = lane; i < n_kvblk; i += 64) mx = fmaxf(mx, v_scale[i]);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
  if (BITS == 4 && FMT == HYQ_FMT_INT) mx *= 0.0625f;
  if (mx > 0.0f) {
    int e;
    frexpf(mx, &e);
    e = max(-100, min(100, e));
    pl.vref = ldexpf(1.0f, e);
  }
  return pl;
}

// The full-precision key list of a plan.
__device__ __forceinline__ FpList fp_list(const KeyPlan& pl, const int32_t* vl, const int32_t* kq,
                                          const uint16_t* Kh) {
  FpList fl;
  fl.vl = vl;
  fl.kq = kq;
  fl.dummy = reinterpret_cast<const int32_t*>(Kh);
  fl.nvl = pl.nvl;
  fl.nq0 = pl.nq0;
  fl.nqb = pl.nqb;
  fl.base = pl.fp_base;
  fl.count = pl.fp_count;
  fl.band_w = pl.shift;
  return fl;
}

// Four consecutive output channels (values * sc) at element offset `at`.
template <int OUT_BF16>
__device__ __forceinline__ void store_out4(void* out, size_t at, float o0, float o1, float o2,
                                           float o3) {
  if (OUT_BF16) {
    uint16_t* o = reinterpret_cast<uint16_t*>(out) + at;
    const __bf16 b0 = (__bf16)o0, b1 = (__bf16)o1, b2 = (__bf16)o2, b3 = (__bf16)o3;
    const uint32_t w0 = (uint32_t)__builtin_bit_cast(uint16_t, b0) |
                        ((uint32_t)__builtin_bit_cast(uint16_t, b1) << 16);
    const uint32_t w1 = (uint32_t)__builtin_bit_cast(uint16_t, b2) |
                        ((uint32_t)__builtin_bit_cast(uint16_t, b3) << 16);
    *reinterpret_cast<uint2*>(o) = make_uint2(w0, w1);
  } else {
    *reinterpret_cast<float4*>(reinterpret_cast<float*>(out) + at) = make_float4(o0, o1, o2, o3);
  }
}

template <int BITS, int OUT_BF16, int FMT, int NW, int S>
__global__ void __launch_bounds__(NW * S * 64, 8 / (NW * S))
attn_prefill_kernel(const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
                    const uint16_t* __restrict__ V, const int32_t* __restrict__ idx,
                    const int8_t* __restrict__ q_codes, const float* __restrict__ q_scale,
                    const uint8_t* __restrict__ k_codes, const float* __restrict__ k_scale,
                    const uint8_t* __restrict__ v_codes, const float* __restrict__ v_scale,
                    const int32_t* __restrict__ kq_pos, void* __restrict__ out, int Hq, int Hkv,
                    int nbj, int L, int P, int k, int nQ, int n_qblk, int n_kvblk,
                    float alpha_log2e, int band_w, int fold) {
  constexpr int NT = NW * 64;   // threads of a group
  __shared__ Smem sms[S];
  const int g = Hq / Hkv;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  // (written so that one group folds: its LDS base and tile steps are constants)
  const int grp = S == 1 ? 0 : wv / NW, w = S == 1 ? wv : wv % NW;
  Smem& sm = sms[grp];
  const int half = lane >> 5, col = lane & 31;

  // Work units of one KV head: (block rb of 32 rows, query head hh of the
  // group), ordered by rb; a workgroup takes NW consecutive units (with S = 2
  // both its groups take the same ones), longest first; kHalf (NW = 4, S = 1)
  // after `fold` workgroups of a head the rest shortest first.  (Where only
  // run time told which, the full-chip shape took 0.2 to 0.7% longer: 20000
  // rows, 32 heads, nearly every key in full precision 3767 us, 3719 so.)
  constexpr int kRows = 32;
  const int nrb = (L + kRows - 1) / kRows;
  const int units = g * nrb;
  const int wg_per_bj = (units + NW - 1) / NW;
  const int slot = (int)blockIdx.x / nbj;
  const bool up = NW == 4 && S == 1 && slot >= fold;
  const int wgi = up ? slot - fold : wg_per_bj - 1 - slot;
  const int bj = (int)blockIdx.x % nbj;
  const int u = wgi * NW + w;
  const bool active = u < units;
  const int uu = active ? u : units - 1;   // an idle wave mirrors the last unit, stores nothing
  const int rb = uu / g, hh = uu % g;
  const int u_last = min(wgi * NW + NW - 1, units - 1);
  const int t_last = min(L - 1, (u_last / g) * kRows + kRows - 1);   // workgroup
  const int b = bj / Hkv, j = bj % Hkv, h = j * g + hh;
  const size_t bh = (size_t)b * Hq + h;
  const int t0 = rb * kRows;
  const int tq = t0 + col;                 // this lane's query row
  const bool row_ok = active && tq < L;

  const uint16_t* Kh = K + (size_t)bj * L * kHeadDim;
  const uint16_t* Vh = V + (size_t)bj * L * kHeadDim;
  const int32_t* vl = idx + (size_t)bj * k;

  NState st;
  init_state(st);

  const KeyPlan pl = key_plan<BITS, FMT>(vl, v_scale + (size_t)bj * n_kvblk, k, P, nQ, n_kvblk,
                                         ((wgi * NW) / g) * kRows, t_last, band_w);
  const int shift = pl.shift, nq_tiles = pl.nq_tiles, fp_count = pl.fp_count;
  float vref = pl.vref;
  float inv_vref = 1.0f / vref;

  // ---------------- segment A: quantized keys ----------------
  if (nq_tiles > 0) {
    constexpr int kRow = BITS == 8 ? kHeadDim : kHeadDim / 2;
    constexpr int vRow = BITS == 8 ? kTile : kTile / 2;
    const size_t slots = (size_t)n_kvblk * kTile;
    SegA a;
    a.kc0 = k_codes + (size_t)bj * slots * kRow;
    a.vc0 = v_codes + (size_t)bj * n_kvblk * kHeadDim * vRow;
    a.kq0 = kq_pos + (size_t)bj * slots;
    a.ks0 = k_scale + (size_t)bj * n_kvblk;
    a.vs0 = v_scale + (size_t)bj * n_kvblk;
    a.n = nq_tiles;
    a.grp = grp;
    a.t0 = t0 - shift;   // rows t see quantized positions <= t - shift
    a.cq = alpha_log2e * q_scale[bh * n_qblk + t0 / kBlock];
    a.inv_vref = inv_vref;
    a.lane = lane;
    a.half = half;
    a.col = col;

    QFrag<FMT> qf;
    read_qfrag<FMT>(qf, q_codes + (bh * L + (row_ok ? tq : 0)) * kHeadDim, row_ok, half);

    // prologue: K(0), K(1) into LDS, K(2) and V(0) into registers, the
    // fragments of K(0) read; the V buffer that tile 0 multiplies by zero
    // weights is cleared (no stale NaNs)
    const int tid = group_tid<NT>(), steps = (nq_tiles + S - 1) / S;
    auto tile = [&](int i) { return min(i * S + grp, nq_tiles - 1); };
    StageRegs<BITS, NT> sr;
    stage_load<BITS, NT>(sr, a, tile(0), 0, tid);
    const VScale unit = make_vscale(1.0f);   // the V written here is cleared below
    stage_store<BITS, FMT, NT>(sm.q.kb[0], sm.q.vb[1], sr, tid, unit);
    stage_load<BITS, NT>(sr, a, tile(1), 0, tid);
    stage_store<BITS, FMT, NT>(sm.q.kb[1], sm.q.vb[1], sr, tid, unit);
    stage_load<BITS, NT>(sr, a, tile(2), tile(0), tid);
    __syncthreads();
    for (int i = tid; i < kVBytes / 16; i += NT)
      reinterpret_cast<v4u*>(sm.q.vb[1].v)[i] = v4u{0u, 0u, 0u, 0u};
    KFrag<FMT> kf;
    read_kfrag<FMT>(kf, sm.q.kb[0], col, half);
    __syncthreads();

    // the P V of tile c runs in iteration c+1, next to the softmax of c+1;
    // the weights alternate between two register sets
    v8h pa[4], pb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < 8; ++e) pa[i][e] = pb[i][e] = (_Float16)0.0f;
    int c = 0;
    for (; c + 3 < steps; c += 4) {
      segA_tile<BITS, FMT, NT, S, 0>(sm, a, c, qf, st, pa, pb, sr, kf);
      segA_tile<BITS, FMT, NT, S, 1>(sm, a, c + 1, qf, st, pb, pa, sr, kf);
      segA_tile<BITS, FMT, NT, S, 2>(sm, a, c + 2, qf, st, pa, pb, sr, kf);
      segA_tile<BITS, FMT, NT, S, 3>(sm, a, c + 3, qf, st, pb, pa, sr, kf);
    }
    if (c < steps) segA_tile<BITS, FMT, NT, S, 0>(sm, a, c, qf, st, pa, pb, sr, kf);
    if (c + 1 < steps) segA_tile<BITS, FMT, NT, S, 1>(sm, a, c + 1, qf, st, pb, pa, sr, kf);
    if (c + 2 < steps) segA_tile<BITS, FMT, NT, S, 2>(sm, a, c + 2, qf, st, pa, pb, sr, kf);
    // P V of the last tile
    const v8h (&plast)[4] = (steps & 1) ? pb : pa;
    const VBuf& lb = sm.q.vb[(steps - 1) & 1];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int dg = 0; dg < 4; ++dg) {
        const v8h va = *reinterpret_cast<const v8h*>(lb.v + (dg * 32 + col) * kVPitch + ks * 32 +
                                                     half * 16);
        st.acc[dg] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va, plast[ks], st.acc[dg], 0, 0, 0);
      }
    __syncthreads();   // the FP segment reuses the LDS
  }

  // ---------------- segments B and C: full-precision keys ----------------
  if constexpr (BITS == 16) {
    SegD a;
    a.k0 = reinterpret_cast<const uint8_t*>(Kh);
    a.v0 = reinterpret_cast<const uint8_t*>(Vh);
    a.n = (fp_count + kTile - 1) / kTile;
    a.grp = grp;
    a.rows = fp_count;
    a.t0 = t0;
    a.alpha_log2e = alpha_log2e;
    a.half = half;
    a.col = col;
    DRing& d = sm.d;
    const int tid = group_tid<NT>(), steps = (a.n + S - 1) / S;
    auto tile = [&](int i) { return min(i * S + grp, a.n - 1); };
    DenseRegs<NT> dr;
    dense_load_k<NT>(dr, a, tile(0));
    v8bf qb[8];
    const uint16_t* qrow = Q + (bh * L + (row_ok ? tq : 0)) * kHeadDim;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) qb[ks] = *reinterpret_cast<const v8bf*>(qrow + ks * 16 + half * 8);
    dense_store_k<NT>(d.k[0], dr);
    dense_load_k<NT>(dr, a, tile(1));
    dense_load_v<NT>(dr, a, tile(0));
    // the V buffer that tile 0 multiplies by zero weights is cleared (no stale NaNs)
    for (int i = tid; i < kVBytes / 16; i += NT)
      reinterpret_cast<v4u*>(d.vb[1].v)[i] = v4u{0u, 0u, 0u, 0u};
    if (tid == 0) d.ovf[0] = d.ovf[1] = -1;
    __syncthreads();
    v8h pa[4], pb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < 8; ++e) pa[i][e] = pb[i][e] = (_Float16)0.0f;
    int c = 0;
    for (; c + 1 < steps; c += 2) {
      segD_tile<NT, S, 0>(sms, a, c, qb, st, pa, pb, dr, vref, inv_vref);
      segD_tile<NT, S, 1>(sms, a, c + 1, qb, st, pb, pa, dr, vref, inv_vref);
    }
    if (c < steps) segD_tile<NT, S, 0>(sms, a, c, qb, st, pa, pb, dr, vref, inv_vref);
    dense_check_v<NT, S>(sms, a, steps - 1, st, vref, inv_vref);
    const v8h (&plast)[4] = (steps & 1) ? pb : pa;
    const VBuf& lb = d.vb[(steps - 1) & 1];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int dg = 0; dg < 4; ++dg) {
        const v8h va = *reinterpret_cast<const v8h*>(lb.v + (dg * 32 + col) * kVPitch + ks * 32 +
                                                     half * 16);
        st.acc[dg] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va, plast[ks], st.acc[dg], 0, 0, 0);
      }
    if (S > 1) __syncthreads();   // the merge reuses the LDS
  } else if (fp_count > 0) {
    v8bf qb[8];
    {
      const uint16_t* qrow = Q + (bh * L + (row_ok ? tq : 0)) * kHeadDim;
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) qb[ks] = *reinterpret_cast<const v8bf*>(qrow + ks * 16 + half * 8);
    }
    const int nft = (fp_count + kTile - 1) / kTile;
    const FpList fl = fp_list(pl, vl, kq_pos + (size_t)bj * n_kvblk * kTile, Kh);
    // prologue: tile 0 published, tile 1 in registers.  Tile f is computed
    // from sm.f[f % 2] while tile f+1 (loaded during tile f-1) is written to
    // the other buffer and the rows of tile f+2 (and the position words of
    // tile f+3) are loaded; one barrier per tile.  Tiles past the end are
    // staged as padding into the free buffer (no branch).
    if (group_tid<NT>() == 0) sm.f[0].ovf = sm.f[1].ovf = -1;
    FpRegs<NT> fr;
    fp_load_words<NT>(fr, fl, grp);
    fp_load<NT, S>(fr, fl, Kh, Vh, grp, L);
    __syncthreads();
    fp_store<NT>(sm.f[0], fr, inv_vref, grp, L);
    fp_load<NT, S>(fr, fl, Kh, Vh, S + grp, L);
    __syncthreads();
    for (int f = 0; f * S < nft; ++f) {   // the group's tile ft (all padding past the end)
      const int ft = f * S + grp;
      FBuf& cur = sm.f[f & 1];
      // without the band the list is ascending: a tile whose last position
      // is at or before the wave's first row is seen whole by every row
      const bool full = shift == 0 && cur.pos[kTile - 1] <= t0;
      uint32_t vis = ~0u;
      if (!full) vis = fp_vis_mask(cur, tq, half, shift > 0);
      {
        // V of this tile outside the f16 range at the current sVref: raise
        // sVref to 2^(E - 134) (every |V| / sVref of the tile below 2^8),
        // rescale the accumulator (exact), restage the tile's V.  The barrier
        // is for both groups, whichever has such a tile.
        const int ov = cur.ovf;
        const bool mine = (ov >> 8) == ft;
        const bool any = S > 1 &&
                         (mine || (sms[S - 1 - grp].f[f & 1].ovf >> 8) == f * S + (S - 1 - grp));
        if (mine) {
          const int ex = max(-100, (ov & 0xff) - 134);
          const float nv = fmaxf(vref, __builtin_ldexpf(1.0f, ex));
          const float c = vref / nv;
#pragma unroll
          for (int dg = 0; dg < 4; ++dg)
#pragma unroll
            for (int r = 0; r < 16; ++r) st.acc[dg][r] *= c;
          vref = nv;
          inv_vref = 1.0f / nv;
          fp_restage_v<NT>(cur, Vh, L, inv_vref);
          if (S == 1) __syncthreads();
        }
        if (any) __syncthreads();
      }
      v16f sf[2];
#pragma unroll
      for (int kh = 0; kh < 2; ++kh) {
#pragma unroll
        for (int r = 0; r < 16; ++r) sf[kh][r] = 0.0f;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
          const v8bf ka = *reinterpret_cast<const v8bf*>(cur.k + (kh * 32 + col) * kKPitchBf +
                                                         ks * 32 + half * 16);
          sf[kh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qb[ks], sf[kh], 0, 0, 0);
        }
      }
      fp_store<NT>(sm.f[(f + 1) & 1], fr, inv_vref, ft + S, L);
      fp_load<NT, S>(fr, fl, Kh, Vh, ft + 2 * S, L);
      if (!full) {
#pragma unroll
        for (int kh = 0; kh < 2; ++kh)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            sf[kh][r] = (vis >> (kh * 16 + r)) & 1 ? sf[kh][r] : -INFINITY;
      }
      // f16 weights against f16 V / sVref
      v8h p[4];
      fp_softmax(st, sf, alpha_log2e, p);
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int dg = 0; dg < 4; ++dg) {
          const v8h va = *reinterpret_cast<const v8h*>(cur.v + (dg * 32 + col) * kVPitch +
                                                       ks * 32 + half * 16);
          st.acc[dg] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va, p[ks], st.acc[dg], 0, 0, 0);
        }
      __syncthreads();
    }
  }

  if constexpr (S == 2) {
    // the second group's state joins the first's (same units, same lanes)
    struct Merge {
      float acc[NW][64][64], m[NT], l[NT], vref[NT];
    };
    static_assert(sizeof(Merge) <= sizeof(sms), "the states fit the tiles' LDS");
    Merge& mg = *reinterpret_cast<Merge*>(sms);
    const int tid = group_tid<NT>();
    if (grp == 1) {   // (every wave is past the last barrier of the tiles)
#pragma unroll
      for (int dg = 0; dg < 4; ++dg)
#pragma unroll
        for (int r = 0; r < 16; ++r) mg.acc[w][dg * 16 + r][lane] = st.acc[dg][r];
      mg.m[tid] = st.m;
      mg.l[tid] = st.l;
      mg.vref[tid] = vref;
    }
    __syncthreads();
    if (grp == 1) return;
    const float M = fmaxf(st.m, mg.m[tid]);
    const float f0 = __builtin_amdgcn_exp2f(st.m - M), f1 = __builtin_amdgcn_exp2f(mg.m[tid] - M);
    // the row sum first: each state is scaled by its weight's share of it and
    // never by sVref alone, so O * l (which may leave float32) is not formed
    // (sVref is a power of two: sVref * rl is sVref / l)
    const float rl = 1.0f / xhalf_sum(__builtin_fmaf(mg.l[tid], f1, st.l * f0));
    const float c0 = f0 * (vref * rl), c1 = f1 * (mg.vref[tid] * rl);
#pragma unroll
    for (int dg = 0; dg < 4; ++dg)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        st.acc[dg][r] = __builtin_fmaf(mg.acc[w][dg * 16 + r][lane], c1, st.acc[dg][r] * c0);
  }

  // ---------------- finalize: O = acc * sVref / l ----------------
  const float sc = S == 2 ? 1.0f : vref / xhalf_sum(st.l);
  if (!row_ok) return;
  const size_t obase = (bh * L + tq) * kHeadDim;
#pragma unroll
  for (int dg = 0; dg < 4; ++dg)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const int d = dg * 32 + r4 * 8 + half * 4;
      store_out4<OUT_BF16>(out, obase + d, st.acc[dg][r4 * 4 + 0] * sc, st.acc[dg][r4 * 4 + 1] * sc,
                           st.acc[dg][r4 * 4 + 2] * sc, st.acc[dg][r4 * 4 + 3] * sc);
    }
}

// ---------------------------------------------------------------------------
// Key-split variant for launches with too few work units to fill the chip:
// one workgroup per unit, its 8 waves taking every 8th quantized tile and
// every 8th full-precision tile, each with its own online-softmax state, and
// merging the 8 states in LDS at the end.  A unit then takes about an eighth
// of the serial steps.  The waves share no tile: K and V codes go from L2
// straight into MFMA registers, a tile ahead, and no barrier couples the
// waves; full-precision V tiles are transposed through a wave's own LDS.  The
// price is that every wave converts its own V codes (160 vector instructions
// a tile instead of 20), so full chips keep the shared-tile kernel.
//
// K rows are assigned to MFMA rows so that lane half h, register r of half-
// tile kh holds key kh*32 + h*16 + r: a lane's 16 keys are contiguous, hence
// its V operand is 16 contiguous codes of a channel.
// ---------------------------------------------------------------------------
constexpr int kSplitWaves = 8;
constexpr int kAccPitch = kHeadDim + 4;   // floats per merged row (+4: bank shift)
struct SplitTile {                        // a wave's full-precision tile
  alignas(16) uint8_t v[kVBytes];
  alignas(16) int32_t pos[kTile];
  alignas(16) int32_t hi[kTile];
};
struct SplitMerge {
  alignas(16) float acc[kSplitWaves][32 * kAccPitch];
  float m[kSplitWaves][32], l[kSplitWaves][32], vref[kSplitWaves];
};
union SplitSmem {
  SplitTile t[kSplitWaves];
  SplitMerge mg;
};

// Key (of a 32-key half-tile) of MFMA row m.
__device__ __forceinline__ int split_key(int m) {
  return ((m >> 2) & 1) * 16 + (m >> 3) * 4 + (m & 3);
}

// K and V codes of one tile in a wave's registers: the 16-byte chunks of K
// row kh*32 + split_key(col) that make up this lane half's fragments, and of
// V channel dg*32 + col the codes of keys kh*32 + half*16 .. +16.
template <int BITS>
struct SplitRaw {
  static constexpr int kK = BITS == 8 ? 4 : 2;
  v4u k[2][kK];
  std::conditional_t<BITS == 8, v4u, v2u> v[4][2];
};
template <int BITS, int FMT>
__device__ __forceinline__ void split_load_k(SplitRaw<BITS>& r, const uint8_t* kc, int col,
                                             int half) {
  constexpr int kRow = BITS == 8 ? kHeadDim : kHeadDim / 2;
#pragma unroll
  for (int kh = 0; kh < 2; ++kh) {
    const v4u* row = reinterpret_cast<const v4u*>(kc + (kh * 32 + split_key(col)) * kRow);
#pragma unroll
    for (int i = 0; i < SplitRaw<BITS>::kK; ++i)
      r.k[kh][i] = row[FMT == HYQ_FMT_FP8 ? (i >> 1) * 4 + half * 2 + (i & 1) : i * 2 + half];
  }
}
template <int BITS>
__device__ __forceinline__ void split_load_v(SplitRaw<BITS>& r, const uint8_t* vc, int col,
                                             int half) {
  constexpr int vRow = BITS == 8 ? kTile : kTile / 2;
#pragma unroll
  for (int dg = 0; dg < 4; ++dg)
#pragma unroll
    for (int kh = 0; kh < 2; ++kh) {
      using T = std::remove_reference_t<decltype(r.v[dg][kh])>;
      r.v[dg][kh] = *reinterpret_cast<const T*>(vc + (dg * 32 + col) * vRow + kh * (vRow / 2) +
                                                half * (vRow / 4));
    }
}

template <int BITS, int FMT>
__device__ __forceinline__ void split_kfrag(KFrag<FMT>& kf, const SplitRaw<BITS>& r) {
#pragma unroll
  for (int kh = 0; kh < 2; ++kh) {
    if constexpr (FMT == HYQ_FMT_FP8) {
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
        kf.f[kh][kk] = __builtin_shufflevector(__builtin_bit_cast(v4i, r.k[kh][2 * kk]),
                                               __builtin_bit_cast(v4i, r.k[kh][2 * kk + 1]), 0, 1,
                                               2, 3, 4, 5, 6, 7);
    } else if constexpr (kv_fp4(FMT) || BITS == 8) {
#pragma unroll
      for (int i = 0; i < SplitRaw<BITS>::kK; ++i) kf.f[kh][i] = __builtin_bit_cast(v4i, r.k[kh][i]);
    } else {   // a chunk of 32 int4 channels is two int8 fragments (16 * code)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        uint32_t o[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) i4x8_to_i8(r.k[kh][i][e], o[2 * e], o[2 * e + 1]);
        kf.f[kh][2 * i] = v4i{(int)o[0], (int)o[1], (int)o[2], (int)o[3]};
        kf.f[kh][2 * i + 1] = v4i{(int)o[4], (int)o[5], (int)o[6], (int)o[7]};
      }
    }
  }
}
// The Q fragments that go with split_kfrag: as read_qfrag, but int4 chunk i of
// lane half h covers channels 64i + 32h .. +32, the fragments 2i and 2i + 1.
template <int BITS, int FMT>
__device__ __forceinline__ void split_qfrag(QFrag<FMT>& qf, const int8_t* qrow, bool ok, int half) {
  if constexpr (BITS == 4 && FMT == HYQ_FMT_INT) {
#pragma unroll
    for (int k4 = 0; k4 < 4; ++k4)
      qf.f[k4] = ok ? *reinterpret_cast<const v4i*>(qrow + (k4 >> 1) * 64 + half * 32 + (k4 & 1) * 16)
                    : v4i{};
  } else {
    read_qfrag<FMT>(qf, qrow, ok, half);
  }
}

// V operand of channel group dg: keys kh*32 + half*16 + 8*e .. +8 as f16 * 2^ev.
template <int BITS, int FMT>
__device__ __forceinline__ void split_vfrag(v8h (&va)[2], const SplitRaw<BITS>& r, int dg, int kh,
                                            const VScale& vs) {
  uint32_t h[8];
  if constexpr (BITS == 8) {
#pragma unroll
    for (int e = 0; e < 4; ++e) codes4_to_h<FMT>(r.v[dg][kh][e], h[2 * e], h[2 * e + 1], vs);
  } else if constexpr (kv_fp4(FMT)) {
#pragma unroll
    for (int e = 0; e < 2; ++e)
      e2m1x8_to_h(r.v[dg][kh][e], *reinterpret_cast<uint32_t(*)[4]>(&h[4 * e]), vs.f32);
  } else {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      uint32_t b0, b1;
      i4x8_to_i8(r.v[dg][kh][e], b0, b1);
      i8x4_to_h(b0, h[4 * e], h[4 * e + 1], vs);
      i8x4_to_h(b1, h[4 * e + 2], h[4 * e + 3], vs);
    }
  }
  va[0] = __builtin_bit_cast(v8h, v4u{h[0], h[1], h[2], h[3]});
  va[1] = __builtin_bit_cast(v8h, v4u{h[4], h[5], h[6], h[7]});
}

__device__ __forceinline__ float lane_max(const float (&s)[2][16]) {
  float mx = -INFINITY;
#pragma unroll
  for (int kh = 0; kh < 2; ++kh)
#pragma unroll
    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kh][r]);
  return mx;
}
// Raise m to the tile maximum (of the lanes' maxima mx) when needed, then the
// f16 weights 2^(s * c + log2 fm - m) into p and their sum, divided by fm,
// into l (hidden keys are -inf; c > 0).
__device__ __forceinline__ void split_softmax(NState& st, const float (&s)[2][16], float mx, float c,
                                              float fm, v8h (&p)[4]) {
  lazy_max(st, xhalf_max(mx) * c);
  apply_corr(st);
  const float bias = __builtin_amdgcn_logf(fm) - st.m;
  const v2h one2 = {(_Float16)1.0f, (_Float16)1.0f};
  float ps = 0.0f;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int kh = i >> 3, r = (i & 7) * 2;
    v2f e;
    e[0] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[kh][r], c, bias));
    e[1] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[kh][r + 1], c, bias));
    const v2h pk = __builtin_convertvector(e, v2h);
    ps = __builtin_amdgcn_fdot2(pk, one2, ps, false);
    p[kh * 2 + (r >> 3)][r & 7] = pk[0];
    p[kh * 2 + (r >> 3)][(r & 7) + 1] = pk[1];
  }
  st.l = __builtin_fmaf(ps, __builtin_amdgcn_rcpf(fm), st.l);
}

template <int BITS, int OUT_BF16, int FMT>
__global__ void __launch_bounds__(kSplitWaves * 64, 1)
attn_prefill_split_kernel(const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
                          const uint16_t* __restrict__ V, const int32_t* __restrict__ idx,
                          const int8_t* __restrict__ q_codes, const float* __restrict__ q_scale,
                          const uint8_t* __restrict__ k_codes, const float* __restrict__ k_scale,
                          const uint8_t* __restrict__ v_codes, const float* __restrict__ v_scale,
                          const int32_t* __restrict__ kq_pos, void* __restrict__ out, int Hq,
                          int Hkv, int nbj, int L, int P, int k, int nQ, int n_qblk, int n_kvblk,
                          float alpha_log2e, int band_w) {
  __shared__ SplitSmem sm;
  const int g = Hq / Hkv;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int half = lane >> 5, col = lane & 31;
  // unit u = (32-row block u / g, head u % g of the group), longest first
  const int units = g * ((L + 31) / 32);
  const int u = units - 1 - (int)blockIdx.x / nbj, bj = (int)blockIdx.x % nbj;
  const int t0 = (u / g) * 32, t_last = min(L - 1, t0 + 31);
  const int b = bj / Hkv, h = (bj % Hkv) * g + u % g;
  const size_t bh = (size_t)b * Hq + h;
  const int tq = t0 + col;
  const bool row_ok = tq < L;
  const uint16_t* Kh = K + (size_t)bj * L * kHeadDim;
  const uint16_t* Vh = V + (size_t)bj * L * kHeadDim;
  const int32_t* vl = idx + (size_t)bj * k;
  const int32_t* kq0 = kq_pos + (size_t)bj * n_kvblk * kTile;

  NState st;
  init_state(st);
  constexpr int kQBits = BITS == 16 ? 8 : BITS;   // (the quantized part compiles to nothing at 16)
  constexpr size_t kTileK = (size_t)kTile * (kQBits == 8 ? kHeadDim : kHeadDim / 2);
  constexpr size_t kTileV = (size_t)kHeadDim * (kQBits == 8 ? kTile : kTile / 2);
  const uint8_t* kc0 = BITS == 16 ? nullptr : k_codes + (size_t)bj * n_kvblk * kTileK;
  const uint8_t* vc0 = BITS == 16 ? nullptr : v_codes + (size_t)bj * n_kvblk * kTileV;
  SplitRaw<kQBits> raw;
  QFrag<FMT> qf;
  if (BITS != 16 && n_kvblk > 0) {   // the first tile, in flight during the searches
    const int c = min(w, n_kvblk - 1);
    split_load_k<kQBits, FMT>(raw, kc0 + c * kTileK, col, half);
    split_qfrag<kQBits, FMT>(qf, q_codes + (bh * L + (row_ok ? tq : 0)) * kHeadDim, row_ok, half);
    split_load_v<kQBits>(raw, vc0 + c * kTileV, col, half);
  }
  const KeyPlan pl = key_plan<BITS, FMT>(vl, v_scale + (size_t)bj * n_kvblk, k, P, nQ, n_kvblk, t0,
                                         t_last, band_w);
  float vref = pl.vref, inv_vref = 1.0f / vref;

  // ---------------- quantized keys ----------------
  if (BITS != 16) {
    constexpr float kSub = (BITS == 8 || kv_fp4(FMT)) ? 1.0f : 0.0625f;
    const float* ks0 = k_scale + (size_t)bj * n_kvblk;
    const float* vs0 = v_scale + (size_t)bj * n_kvblk;
    const float cq = alpha_log2e * q_scale[bh * n_qblk + t0 / kBlock];
    const int last_seen = t0 - pl.shift;   // every row sees quantized positions up to here
    for (int c = w; c < pl.nq_tiles; c += kSplitWaves) {
      const int cn = min(c + kSplitWaves, pl.nq_tiles - 1);   // past the end: loaded, not used
      const float sv = vs0[c] * kSub;
      // (a zero K block has zero scores: the floor keeps -inf * c from a NaN)
      const float cqk = fmaxf(cq * (ks0[c] * kSub), 1e-30f);
      int ev;
      float fm = __builtin_frexpf(sv * inv_vref, &ev);
      if (!(sv > 0.0f)) {   // all-zero V block: its V codes are 0, fold nothing
        fm = 1.0f;
        ev = 0;
      }
      const VScale vs = make_vscale(__builtin_ldexpf(1.0f, ev));
      const bool diag = kq0[c * kTile + kTile - 1] > last_seen;
      SVec<FMT> s[2];
      {
        KFrag<FMT> kf;
        split_kfrag<kQBits, FMT>(kf, raw);
        qk_tile<FMT>(s, kf, qf);
      }
      split_load_k<kQBits, FMT>(raw, kc0 + cn * kTileK, col, half);
      float y[2][16];
#pragma unroll
      for (int kh = 0; kh < 2; ++kh)
#pragma unroll
        for (int r = 0; r < 16; ++r) y[kh][r] = (float)s[kh][r];
      // the maximum first: its reads of the MFMA results stay on the straight
      // path, where the compiler pads them with the wait states they need
      float mx = lane_max(y);
      asm volatile("" : "+v"(mx));   // (keeps it there)
      if (diag) {
        const int tv = tq - pl.shift;
#pragma unroll
        for (int kh = 0; kh < 2; ++kh)
#pragma unroll
          for (int r4 = 0; r4 < 4; ++r4) {
            const v4i p4 = *reinterpret_cast<const v4i*>(kq0 + c * kTile + kh * 32 + half * 16 + r4 * 4);
#pragma unroll
            for (int j = 0; j < 4; ++j)
              y[kh][r4 * 4 + j] = p4[j] <= tv ? y[kh][r4 * 4 + j] : -INFINITY;
          }
        mx = lane_max(y);
      }
      v8h p[4];
      split_softmax(st, y, mx, cqk, fm, p);
#pragma unroll
      for (int kh = 0; kh < 2; ++kh)
#pragma unroll
        for (int dg = 0; dg < 4; ++dg) {
          v8h va[2];
          split_vfrag<kQBits, FMT>(va, raw, dg, kh, vs);
#pragma unroll
          for (int e = 0; e < 2; ++e)
            st.acc[dg] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va[e], p[kh * 2 + e], st.acc[dg], 0,
                                                                0, 0);
        }
      split_load_v<kQBits>(raw, vc0 + cn * kTileV, col, half);
    }
  }

  // ---------------- full-precision keys ----------------
  const int nft = (pl.fp_count + kTile - 1) / kTile;
  if (w < nft) {
    SplitTile& T = sm.t[w];
    v8bf qb[8];
    const uint16_t* qrow = Q + (bh * L + (row_ok ? tq : 0)) * kHeadDim;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) qb[ks] = *reinterpret_cast<const v8bf*>(qrow + ks * 16 + half * 8);
    const FpList fl = fp_list(pl, vl, kq0, Kh);
    for (int ft = w; ft < nft; ft += kSplitWaves) {
      // K rows of this lane's two MFMA rows; V rows of key pair `col`
      int pk[2], hk[2], pv[2], hv[2];
#pragma unroll
      for (int kh = 0; kh < 2; ++kh) {
        const int e = ft * kTile + kh * 32 + split_key(col);
        fp_resolve(fl, e, *fp_src(fl, e), pk[kh], hk[kh]);
        const int ev = ft * kTile + 2 * col + kh;
        fp_resolve(fl, ev, *fp_src(fl, ev), pv[kh], hv[kh]);
      }
      v4u kr[2][8];
#pragma unroll
      for (int kh = 0; kh < 2; ++kh) {   // padding rows read row 0; they are hidden below
        const size_t row = (unsigned)pk[kh] < (unsigned)L ? (size_t)pk[kh] : 0;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks)
          kr[kh][ks] = reinterpret_cast<const v4u*>(Kh + row * kHeadDim)[ks * 2 + half];
      }
      if (half == 0) {
#pragma unroll
        for (int kh = 0; kh < 2; ++kh) {
          T.pos[kh * 32 + split_key(col)] = pk[kh];
          T.hi[kh * 32 + split_key(col)] = hk[kh];
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      v16f sf[2];
#pragma unroll
      for (int kh = 0; kh < 2; ++kh) {
#pragma unroll
        for (int r = 0; r < 16; ++r) sf[kh][r] = 0.0f;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks)
          sf[kh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, kr[kh][ks]), qb[ks],
                                                           sf[kh], 0, 0, 0);
      }
      // V: pair `col`, chunks 2i + half
      v4u vr[2][8];
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        const bool ok = (unsigned)pv[x] < (unsigned)L;
        const size_t row = ok ? (size_t)pv[x] : 0;
#pragma unroll
        for (int i = 0; i < 8; ++i)
          vr[x][i] = reinterpret_cast<const v4u*>(Vh + row * kHeadDim)[2 * i + half] &
                     (ok ? 0xffffffffu : 0u);
      }
      const bool full = pl.shift == 0 && T.pos[kTile - 1] <= t0;
      if (!full) {
#pragma unroll
        for (int kh = 0; kh < 2; ++kh)
#pragma unroll
          for (int r4 = 0; r4 < 4; ++r4) {
            const int e = kh * 32 + half * 16 + r4 * 4;
            const v4i p4 = *reinterpret_cast<const v4i*>(&T.pos[e]);
            const v4i h4 = *reinterpret_cast<const v4i*>(&T.hi[e]);
#pragma unroll
            for (int j = 0; j < 4; ++j)
              sf[kh][r4 * 4 + j] =
                  ((p4[j] <= tq) & (tq <= h4[j])) ? sf[kh][r4 * 4 + j] : -INFINITY;
          }
      }
      v8h p[4];
      fp_softmax(st, sf, alpha_log2e, p);
      float mx = 0.0f;
#pragma unroll
      for (int i = 0; i < 8; ++i)
        mx = fmaxf(mx, fp_store_vpair(T.v, vr[0][i], vr[1][i], 2 * col, 2 * i + half, inv_vref));
      if (__ballot(!(mx * inv_vref <= 65504.0f) && mx == mx)) {
        // V outside the f16 range at the current sVref: raise it to 2^(E - 134)
        // (every |V| / sVref of the tile below 2^8), rescale, store again
        int ex = (int)(__float_as_uint(mx) >> 23);
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) ex = max(ex, __shfl_xor(ex, o, 64));
        const float nv = fmaxf(vref, __builtin_ldexpf(1.0f, max(-100, ex - 134)));
        const float c = vref / nv;
#pragma unroll
        for (int dg = 0; dg < 4; ++dg)
#pragma unroll
          for (int r = 0; r < 16; ++r) st.acc[dg][r] *= c;
        vref = nv;
        inv_vref = 1.0f / nv;
#pragma unroll
        for (int i = 0; i < 8; ++i)
          fp_store_vpair(T.v, vr[0][i], vr[1][i], 2 * col, 2 * i + half, inv_vref);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int dg = 0; dg < 4; ++dg) {
          const v8h va = *reinterpret_cast<const v8h*>(T.v + (dg * 32 + col) * kVPitch +
                                                       (ks >> 1) * 64 + half * 32 + (ks & 1) * 16);
          st.acc[dg] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va, p[ks], st.acc[dg], 0, 0, 0);
        }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
  }

  // ---------------- merge of the 8 states ----------------
  const float lw = xhalf_sum(st.l);
  __syncthreads();   // the tiles' LDS is reused
  SplitMerge& mg = sm.mg;
#pragma unroll
  for (int dg = 0; dg < 4; ++dg)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4)
      *reinterpret_cast<float4*>(&mg.acc[w][col * kAccPitch + dg * 32 + r4 * 8 + half * 4]) =
          make_float4(st.acc[dg][r4 * 4], st.acc[dg][r4 * 4 + 1], st.acc[dg][r4 * 4 + 2],
                      st.acc[dg][r4 * 4 + 3]);
  if (half == 0) {
    mg.m[w][col] = st.m;
    mg.l[w][col] = lw;
  }
  if (lane == 0) mg.vref[w] = vref;
  __syncthreads();
  const int row = (int)threadIdx.x >> 4, d0 = ((int)threadIdx.x & 15) * 8;
  float M = mg.m[0][row];
#pragma unroll
  for (int v = 1; v < kSplitWaves; ++v) M = fmaxf(M, mg.m[v][row]);
  // the row sum before the accumulators, as in the kernel above
  float f[kSplitWaves], l = 0.0f, o[8];
#pragma unroll
  for (int v = 0; v < kSplitWaves; ++v) {
    f[v] = __builtin_amdgcn_exp2f(mg.m[v][row] - M);
    l = __builtin_fmaf(mg.l[v][row], f[v], l);
  }
  const float rl = 1.0f / l;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = 0.0f;
#pragma unroll
  for (int v = 0; v < kSplitWaves; ++v) {
    const float fv = f[v] * (mg.vref[v] * rl);
#pragma unroll
    for (int e4 = 0; e4 < 2; ++e4) {
      const float4 a = *reinterpret_cast<const float4*>(&mg.acc[v][row * kAccPitch + d0 + e4 * 4]);
      o[e4 * 4 + 0] = __builtin_fmaf(a.x, fv, o[e4 * 4 + 0]);
      o[e4 * 4 + 1] = __builtin_fmaf(a.y, fv, o[e4 * 4 + 1]);
      o[e4 * 4 + 2] = __builtin_fmaf(a.z, fv, o[e4 * 4 + 2]);
      o[e4 * 4 + 3] = __builtin_fmaf(a.w, fv, o[e4 * 4 + 3]);
    }
  }
  if (t0 + row >= L) return;
  const size_t at = (bh * L + t0 + row) * kHeadDim + d0;
  store_out4<OUT_BF16>(out, at, o[0], o[1], o[2], o[3]);
  store_out4<OUT_BF16>(out, at + 4, o[4], o[5], o[6], o[7]);
}

template <int BITS, int OB, int FMT>
hipError_t launch_t(const hyq_shape& s, const hyq_sizes& z, const uint16_t* Q,
                    const uint16_t* K, const uint16_t* V, const int32_t* idx,
                    const int8_t* q_codes, const float* q_scale, const uint8_t* k_codes,
                    const float* k_scale, const uint8_t* v_codes, const float* v_scale,
                    const int32_t* kq_pos, float softmax_scale, void* out, hipStream_t st) {
  const int units = s.Hq / s.Hkv * ((s.L + 31) / 32);   // per KV head
  const int nbj = s.B * s.Hkv;
  const int band_w = s.window_mode == HYQ_WIN_BAND ? s.window : 0;
#define HYQ_ARGS                                                                              \
  Q, K, V, idx, q_codes, q_scale, k_codes, k_scale, v_codes, v_scale, kq_pos, out, s.Hq, s.Hkv, \
      nbj, s.L, z.P, z.k, z.nQ, z.n_qblk, z.n_kvblk, softmax_scale * kLog2e, band_w
  const AttnKeys keys = attn_keys((int64_t)z.k + (s.window < s.L ? s.window : s.L), s.L, BITS == 16,
                                  band_w > 0);
  const AttnShape sh = choose_attn_shape(units, nbj, (s.L + kTile - 1) / kTile, keys, device_cus());
  const dim3 grid((unsigned)sh.grid);
  switch (sh.kind) {
    case AttnKind::kSplit8:
      attn_prefill_split_kernel<BITS, OB, FMT><<<grid, kSplitWaves * 64, 0, st>>>(HYQ_ARGS);
      break;
    case AttnKind::kSplit2:
      attn_prefill_kernel<BITS, OB, FMT, 4, 2><<<grid, 512, 0, st>>>(HYQ_ARGS, sh.fold);
      break;
    case AttnKind::kHalf:   // two resident workgroups per CU
      attn_prefill_kernel<BITS, OB, FMT, 4, 1><<<grid, 256, 0, st>>>(HYQ_ARGS, sh.fold);
      break;
    case AttnKind::kFull:
      attn_prefill_kernel<BITS, OB, FMT, 8, 1><<<grid, 512, 0, st>>>(HYQ_ARGS, sh.fold);
      break;
  }
#undef HYQ_ARGS
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_prefill(const hyq_shape& s, const hyq_sizes& z, const uint16_t* Q,
                               const uint16_t* K, const uint16_t* V, const int32_t* idx,
                               const int8_t* q_codes, const float* q_scale,
                               const uint8_t* k_codes, const float* k_scale,
                               const uint8_t* v_codes, const float* v_scale,
                               const int32_t* kq_pos, float softmax_scale, void* out,
                               int out_dtype, hipStream_t st) {
#define HYQ_LAUNCH(BITS, OB, FMT)                                                              \
  return launch_t<BITS, OB, FMT>(s, z, Q, K, V, idx, q_codes, q_scale, k_codes, k_scale,       \
                                 v_codes, v_scale, kq_pos, softmax_scale, out, st)
  if (s.bits_kv == 16) {
    if (out_dtype) HYQ_LAUNCH(16, 1, HYQ_FMT_INT);
    HYQ_LAUNCH(16, 0, HYQ_FMT_INT);
  } else if (s.bits_kv == 4 && s.kv_format == HYQ_FMT_FP4) {
    if (out_dtype) HYQ_LAUNCH(4, 1, HYQ_FMT_FP4);
    HYQ_LAUNCH(4, 0, HYQ_FMT_FP4);
  } else if (s.bits_kv == 4 && s.kv_format == HYQ_FMT_FP4Q6) {
    if (out_dtype) HYQ_LAUNCH(4, 1, HYQ_FMT_FP4Q6);
    HYQ_LAUNCH(4, 0, HYQ_FMT_FP4Q6);
  } else if (s.bits_kv == 8 && s.kv_format == HYQ_FMT_FP8) {
    if (out_dtype) HYQ_LAUNCH(8, 1, HYQ_FMT_FP8);
    HYQ_LAUNCH(8, 0, HYQ_FMT_FP8);
  } else if (s.bits_kv == 8) {
    if (out_dtype) HYQ_LAUNCH(8, 1, HYQ_FMT_INT);
    HYQ_LAUNCH(8, 0, HYQ_FMT_INT);
  } else {
    if (out_dtype) HYQ_LAUNCH(4, 1, HYQ_FMT_INT);
    HYQ_LAUNCH(4, 0, HYQ_FMT_INT);
  }
#undef HYQ_LAUNCH
}

}  // namespace hyq
