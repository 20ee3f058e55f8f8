// Vertical-line selection: Algorithm 1 (App. A.1, Vertical Token
// Identification) of HyQuant, GQA-native, one vertical set per KV head.
// (The exact column-mass score of eq. vl_score, HYQ_SEL_COLMASS, is computed
// in colmass.hip; the top-k below serves both.)
//
//   1. tail proxy   qsum[b][j] = sum over the g heads of the group and the
//                   last t = min(W, L) query rows (float32, pinned order);
//   2. scores       S[b][j][p] = qsum . K[b][j][p], p < P (pinned tree);
//   3. top-k        k largest S, ties to the lowest position, ascending.
//
// Every floating-point operation here is a separately rounded float32
// add or multiply in a fixed order, so the result is reproducible bit for
// bit; contraction into fused multiply-adds is disabled for this file.
//
// The top-k works on order keys (an order-preserving map of the float
// scores to uint32):
//   - while the scores are produced, every workgroup counts its keys by
//     their top 12 bits in LDS and adds the non-empty bins to a histogram of
//     its KV head in the workspace;
//   - classification: the bin holding the k-th largest key comes from that
//     histogram; a bitmap takes the positions in higher bins, a candidate
//     list the keys of that bin (about 1% of them);
//   - two 10-bit radix passes over the candidates resolve the remaining 20
//     bits of the threshold; the chosen positions are written in ascending
//     order (ordered compaction of the bitmaps; keys equal to the threshold
//     lowest position first).
// On short prefixes, and on longer ones of many heads (one_launch), one
// workgroup per head does all of that in one launch (topk_kernel); the others
// classify on many workgroups first (topk_classify_kernel, topk_final_kernel).
//
// A prefill's Q quantization needs nothing of the selection: its blocks ride
// along as extra workgroups of the tail-proxy launch, which alone is bound by
// latency (32k: 7.6 us, and 63 us for Q in a launch of its own; 62 to 65 us
// together).  Giving the top-k launch a share as well was slower: its 1024
// threads and 50 KB of LDS leave one quantizing workgroup per CU, whose waves
// all load and then all compute (8k prefill 522 us with every block here, 545
// / 550 / 576 with a quarter / half / all of them there).
#include "hyq_internal.h"
#include "quant_dev.h"

#pragma clang fp contract(off)

namespace hyq {
namespace {

// Per-head top-k scratch in the workspace: a 4-word header (the candidate
// count, then the bin of the k-th largest key and the keys still to take in
// it, as the classification finds them), the candidate list ((key, position) of the keys in the
// threshold's bin, at most P of them) and the bitmap of positions in higher
// bins (an even number of words).
__host__ __device__ __forceinline__ size_t topk_ws_words(int P) {
  return 4 + 2 * (size_t)P + (size_t)(P + 63) / 64 * 2;
}
struct TopkWs {
  uint32_t* ncand;   // header: [0] candidates, [1] bin, [2] keys of the bin to take
  uint2* cand;
  uint32_t* gt;
};
__device__ __forceinline__ TopkWs topk_ws(uint32_t* base, int bj, int P) {
  uint32_t* h = base + (size_t)bj * topk_ws_words(P);
  TopkWs w;
  w.ncand = h;
  w.cand = reinterpret_cast<uint2*>(h + 4);
  w.gt = h + 4 + 2 * (size_t)P;
  return w;
}

// One workgroup per (b, h, group of 16 channels), so that the short kernel
// spreads over the chip.  The head's t tail rows are staged through LDS
// kTailRows at a time (thread r loads the 32 bytes of row r); then lane d of
// the first wave adds the staged values of channel d in ascending row order,
// continuing from +0 over all t rows, which gives qpart[b][h][d].  The score
// kernel adds the g heads of a group in head order.  The first workgroup of
// each group also clears the key histogram and the top-k candidate count of
// its (b, j), which the next kernels fill.
constexpr int kTailRows = 256;
constexpr int kTailThreads = kTailRows;
constexpr int kTailCh = 16;   // channels per workgroup
constexpr int kTailGroups = kHeadDim / kTailCh;
// Workgroups from n_tail on quantize one Q block each instead.
template <int QFMT>
__global__ void __launch_bounds__(kTailThreads)
tail_proxy_kernel(const uint16_t* __restrict__ Q, float* __restrict__ qpart,
                  uint32_t* __restrict__ hist, uint32_t* __restrict__ tws, int BHq, int g, int L,
                  int t, int P, int n_tail, QuantQ qq) {
  __shared__ uint4 rows[kTailRows][kTailCh / 8];
  const int wg = (int)(blockIdx.y * gridDim.x + blockIdx.x);
  if (wg >= n_tail) {
    quant_q_block<QFMT>(qq, wg - n_tail, reinterpret_cast<float*>(&rows[0][0]));
    return;
  }
  const int bh = wg % BHq, cg = wg / BHq, c0 = cg * kTailCh;
  if (bh % g == 0 && cg == 0) {
    uint32_t* hj = hist + (size_t)(bh / g) * kSelHistBins;
    for (int i = threadIdx.x; i < kSelHistBins; i += kTailThreads) hj[i] = 0u;
    if (threadIdx.x < 4) tws[(size_t)(bh / g) * topk_ws_words(P) + threadIdx.x] = 0u;
  }
  const uint16_t* q = Q + ((size_t)bh * L + (L - t)) * kHeadDim + c0;
  const int d = threadIdx.x;   // channel c0 + d for the adding lanes
  float a = 0.0f;
  for (int r0 = 0; r0 < t; r0 += kTailRows) {
    const int n = min(kTailRows, t - r0);
    // rows past the tail re-read its last row (never added)
    const uint4* src = reinterpret_cast<const uint4*>(
        q + (size_t)min(r0 + (int)threadIdx.x, t - 1) * kHeadDim);
    const uint4 v0 = src[0], v1 = src[1];
    rows[threadIdx.x][0] = v0;
    rows[threadIdx.x][1] = v1;
    __syncthreads();
    if (d < kTailCh) {
      const uint16_t* col = reinterpret_cast<const uint16_t*>(&rows[0][0]) + d;
      for (int i0 = 0; i0 < n; i0 += 32) {   // 32 LDS reads in flight, then the adds in order
        uint16_t x[32];
#pragma unroll
        for (int i = 0; i < 32; ++i) x[i] = col[(size_t)min(i0 + i, kTailRows - 1) * kTailCh];
#pragma unroll
        for (int i = 0; i < 32; ++i)
          if (i0 + i < n) a = a + bf16_bits_to_f32(x[i]);
      }
    }
    __syncthreads();
  }
  if (d < kTailCh) qpart[(size_t)bh * kHeadDim + c0 + d] = a;
}

constexpr int kScoreThreads = 512;         // score_kernel: 64 keys per wave
constexpr int kScoreRows = kScoreThreads;  // keys per score workgroup

// Lane exchange within groups of four lanes (DPP quad permutations).
__device__ __forceinline__ float xor1(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xF, 0xF, true));
}
__device__ __forceinline__ float xor2(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x4E, 0xF, 0xF, true));
}

// Scores of 512 prefix keys per workgroup (two workgroups per CU, so that one
// computes while the other loads), 64 per wave.  A key row is read
// by 4 lanes: lane c (0..3) of the row's group loads the 16-byte chunks c,
// c+4, c+8, c+12 (channels 8c.., 32+8c.., 64+8c.., 96+8c.., eight each), so
// one load instruction covers 16 rows, 64 contiguous bytes each.  The pinned
// fold then runs as a butterfly: the halving steps l + 64 and l + 32 are
// in-lane, steps 16 and 8 pair lane c with lane c^2 and c^1 (the lower lane
// of a pair holds v[l], its partner v[l + h]; float addition is
// commutative, so both lanes get the bits of v[l] + v[l + h]), and steps
// 4, 2, 1 are in-lane again.
__global__ void __launch_bounds__(kScoreThreads, 2)
score_kernel(const uint16_t* __restrict__ K, const float* __restrict__ qpart,
             float* __restrict__ S, uint32_t* __restrict__ hist, int g, int L, int P) {
  __shared__ uint32_t lh[kSelHistBins];
  __shared__ float4 qs[kHeadDim / 4];
  const int bj = blockIdx.x;   // consecutive workgroups take consecutive heads (see the launch)
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int c = lane & 3, rsub = lane >> 2;
  const int base = blockIdx.y * kScoreRows + w * 64;
  const uint4* Kb = reinterpret_cast<const uint4*>(K + (size_t)bj * L * kHeadDim);
  uint4 kr[4][4];   // [iteration][quarter q]: chunk c + 4q of row base + 16*it + rsub
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    // rows past P load row P-1 (unconditional loads stay in flight together);
    // their scores are never stored
    const uint4* rp = Kb + (size_t)min(base + it * 16 + rsub, P - 1) * (kHeadDim / 8);
#pragma unroll
    for (int q = 0; q < 4; ++q) kr[it][q] = rp[c + 4 * q];
  }
  hist_clear(lh);
  if (threadIdx.x < kHeadDim) {   // qsum = the g head partials added in head order
    const float* pp = qpart + (size_t)bj * g * kHeadDim + threadIdx.x;
    float part[8];   // g <= 8; unconditional loads, all in flight
#pragma unroll
    for (int r = 0; r < 8; ++r) part[r] = pp[(size_t)min(r, g - 1) * kHeadDim];
    float a = part[0];
#pragma unroll
    for (int r = 1; r < 8; ++r)
      if (r < g) a = a + part[r];
    reinterpret_cast<float*>(qs)[threadIdx.x] = a;
  }
  __syncthreads();
  // qv[q][e] = qsum[32q + 8c + e]
  float qv[4][8];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float4 a = qs[8 * q + 2 * c], b = qs[8 * q + 2 * c + 1];
    qv[q][0] = a.x; qv[q][1] = a.y; qv[q][2] = a.z; qv[q][3] = a.w;
    qv[q][4] = b.x; qv[q][5] = b.y; qv[q][6] = b.z; qv[q][7] = b.w;
  }

  float sv[4];
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    float pr[4][8];   // products of channel 32q + 8c + e
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t wq[4] = {kr[it][q].x, kr[it][q].y, kr[it][q].z, kr[it][q].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        pr[q][2 * e] = qv[q][2 * e] * bf16_lo(wq[e]);
        pr[q][2 * e + 1] = qv[q][2 * e + 1] * bf16_hi(wq[e]);
      }
    }
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float a = pr[0][e] + pr[2][e];   // step 64: l = 8c+e,    l + 64
      const float b = pr[1][e] + pr[3][e];   //          l = 32+8c+e, l + 64
      v[e] = a + b;                          // step 32: l = 8c+e,    l + 32
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = v[e] + xor2(v[e]);   // step 16
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = v[e] + xor1(v[e]);   // step 8
#pragma unroll
    for (int h = 4; h >= 1; h >>= 1)
#pragma unroll
      for (int e = 0; e < h; ++e) v[e] = v[e] + v[e + h];
    sv[it] = v[0];
  }
  // lane l takes the score of row base + l: iteration l/16, row group l%16
  float s = 0.0f;
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const float x = __shfl(sv[it], 4 * (lane & 15), 64);
    if ((lane >> 4) == it) s = x;
  }
  const int p = base + lane;
  if (p < P) {
    S[(size_t)bj * P + p] = s;
    atomicAdd(&lh[order_key(s) >> kHistShift], 1u);
  }
  __syncthreads();
  hist_flush(lh, hist + (size_t)bj * kSelHistBins);
}

constexpr int kTopkThreads = 1024;
constexpr int kTopkWaves = kTopkThreads / 64;
constexpr int kDigitBits = 10;
constexpr int kDigitBins = 1 << kDigitBits;
static_assert(kSelHistBits + 2 * kDigitBits == 32, "bin + two digits cover the key");
static_assert(kSelHistBins == 4 * kTopkThreads, "four histogram bins per thread");
static_assert(kDigitBins == kTopkThreads, "one digit bin per thread");

struct TopkShared {
  uint32_t dig[kDigitBins];
  uint32_t wtot[2][kTopkWaves];   // wave totals of a block scan (scans alternate)
  uint32_t sel_bin;
  int sel_rem;
};

// Inclusive prefix sum over the 16 lanes of a DPP row, and over the wave.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_add(uint32_t x) {   // lanes without a source add 0
  return x + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ uint32_t row_prefix(uint32_t x) {
  x = dpp_add<0x111, 0xF>(x);   // row_shr:1, 2, 4, 8
  x = dpp_add<0x112, 0xF>(x);
  x = dpp_add<0x114, 0xF>(x);
  return dpp_add<0x118, 0xF>(x);
}
__device__ __forceinline__ uint32_t wave_prefix(uint32_t x) {
  x = row_prefix(x);
  x = dpp_add<0x142, 0xA>(x);      // row_bcast:15 into rows 1 and 3
  return dpp_add<0x143, 0xC>(x);   // row_bcast:31 into rows 2 and 3
}

// Exclusive prefix sum over the workgroup's threads in thread order; the sum
// over all threads goes to `total`.  One barrier: a scan writes the wave
// totals the last one did not (slot alternates from call to call), so they
// are overwritten only after another scan's barrier.
__device__ __forceinline__ uint32_t block_prefix_excl(uint32_t x, TopkShared& sh, int slot,
                                                      uint32_t& total) {
  static_assert(kTopkWaves == 16, "the wave totals fill one DPP row");
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const uint32_t incl = wave_prefix(x);
  if (lane == 63) sh.wtot[slot][w] = incl;
  __syncthreads();
  const uint32_t t = row_prefix(sh.wtot[slot][lane & 15]);
  total = (uint32_t)__builtin_amdgcn_readlane((int)t, 15);
  const uint32_t before = w ? (uint32_t)__builtin_amdgcn_readlane((int)t, w - 1) : 0u;
  return before + incl - x;
}

// Thread t owns the N bins c[0..N) = bins N*t .. N*t+N-1 of an ascending
// histogram.  Finds the bin holding the need-th largest key and how many
// keys of that bin are still to take; the owning thread publishes both.
template <int N>
__device__ __forceinline__ void find_bin(const uint32_t (&c)[N], int need, TopkShared& sh,
                                         int slot) {
  uint32_t mine = 0;
#pragma unroll
  for (int e = 0; e < N; ++e) mine += c[e];
  uint32_t total;
  const uint32_t before = block_prefix_excl(mine, sh, slot, total);
  const uint32_t above = total - before - mine;   // keys in the bins of later threads
  if (above < (uint32_t)need && (uint32_t)need <= above + mine) {
    uint32_t acc = above;
#pragma unroll
    for (int e = N - 1; e >= 0; --e) {
      if (acc + c[e] >= (uint32_t)need) {
        sh.sel_bin = (uint32_t)(N * threadIdx.x + e);
        sh.sel_rem = need - (int)acc;
        break;
      }
      acc += c[e];
    }
  }
  __syncthreads();
}

// The bin of the k-th largest key of head bj from its histogram.
__device__ __forceinline__ void hist_bin(const uint32_t* __restrict__ hist, int bj, int k,
                                         TopkShared& sh) {
  const uint4 h4 = reinterpret_cast<const uint4*>(hist + (size_t)bj * kSelHistBins)[threadIdx.x];
  const uint32_t hc[4] = {h4.x, h4.y, h4.z, h4.w};
  find_bin<4>(hc, k, sh, 0);
}

// Classification, 1024 keys per workgroup (grid: head fastest, then key
// chunk; one key per thread, coalesced): every workgroup finds the bin of
// the k-th largest key from the histogram; a ballot per wave gives the 64
// positions' bits "in a higher bin" as two bitmap words; the keys of that
// bin are appended to the head's candidate list (one atomic reservation per
// wave).
__global__ void __launch_bounds__(kTopkThreads)
topk_classify_kernel(const float* __restrict__ S, const uint32_t* __restrict__ hist,
                     uint32_t* __restrict__ tws, int P, int k) {
  __shared__ TopkShared sh;
  const int bj = blockIdx.x;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int p = blockIdx.y * kTopkThreads + (int)threadIdx.x;
  const bool in = p < P;
  const uint32_t u = order_key(S[(size_t)bj * P + min(p, P - 1)]);   // in flight meanwhile
  hist_bin(hist, bj, k, sh);
  const uint32_t bin = sh.sel_bin;
  const TopkWs f = topk_ws(tws, bj, P);
  if (blockIdx.y == 0 && threadIdx.x == 0) {
    f.ncand[1] = bin;
    f.ncand[2] = (uint32_t)sh.sel_rem;
  }
  const uint32_t b = u >> kHistShift;
  const uint64_t mg = __ballot(in && b > bin);
  const uint64_t mc = __ballot(in && b == bin);
  const int x = (blockIdx.y * kTopkThreads + w * 64) / 32;   // word of this wave's first position
  if (lane == 0 && x * 32 < P)
    *reinterpret_cast<uint2*>(&f.gt[x]) = make_uint2((uint32_t)mg, (uint32_t)(mg >> 32));
  if (mc) {
    uint32_t base = 0;
    if (lane == 0) base = atomicAdd(f.ncand, (uint32_t)__popcll(mc));
    base = __shfl(base, 0, 64);
    const uint32_t r = __builtin_amdgcn_mbcnt_hi((uint32_t)(mc >> 32),
                                                 __builtin_amdgcn_mbcnt_lo((uint32_t)mc, 0u));
    if (in && b == bin && base + r < (uint32_t)P) f.cand[base + r] = make_uint2(u, (uint32_t)p);
  }
}

// The candidates of a head are kept as lists of which each wave owns one: the
// first kLdsCap entries in LDS, the rest (crowded or tied bins) in the
// workspace.  A wave appends to and reads only its own list.
constexpr int kLdsCap = 128;
struct Cands {
  uint2* lds;
  uint2* ws;
  int n;
};
__device__ __forceinline__ uint2 cand_at(const Cands& cs, int c) {
  return c < kLdsCap ? cs.lds[c] : cs.ws[c];
}

// Radix pass over the candidates whose bits above `shift + kDigitBits`
// equal `prefix`: histogram of the next 10-bit digit, then the digit holding
// the need-th largest of them.
__device__ __forceinline__ void cand_digit_pass(const Cands& cs, uint32_t prefix, int shift,
                                                int need, TopkShared& sh, int slot) {
  sh.dig[threadIdx.x] = 0u;
  __syncthreads();
  const int top = shift + kDigitBits;
  for (int c = threadIdx.x & 63; c < cs.n; c += 64) {
    const uint32_t key = cand_at(cs, c).x;
    if ((key >> top) == prefix) atomicAdd(&sh.dig[(key >> shift) & (kDigitBins - 1)], 1u);
  }
  __syncthreads();
  const uint32_t c1[1] = {sh.dig[threadIdx.x]};
  find_bin<1>(c1, need, sh, slot);
}

// The threshold key T from the candidates of bin `bin`, and how many keys
// equal to T to take (lowest positions first).
__device__ __forceinline__ uint32_t cand_threshold(const Cands& cs, uint32_t bin, int need,
                                                   TopkShared& sh, int& need_eq) {
  cand_digit_pass(cs, bin, kDigitBits, need, sh, 1);
  const uint32_t d1 = sh.sel_bin;
  cand_digit_pass(cs, (bin << kDigitBits) | d1, 0, sh.sel_rem, sh, 0);
  need_eq = sh.sel_rem;
  return (bin << (2 * kDigitBits)) | (d1 << kDigitBits) | sh.sel_bin;
}

// Chosen positions of kTopkThreads bitmap words, one per thread: every
// position of `g` plus the lowest positions of `e` while need_eq lasts,
// written ascending from out[o_base] on.  Advances o_base and eq_base.
__device__ __forceinline__ void emit_words(uint32_t g, uint32_t e, int x, int need_eq, int k,
                                           int32_t* __restrict__ out, uint32_t& o_base,
                                           uint32_t& eq_base, TopkShared& sh) {
  const int ne = __popc(e);
  uint32_t eq_tot;
  const int eq_before = (int)(eq_base + block_prefix_excl((uint32_t)ne, sh, 1, eq_tot));
  int keep = max(0, min(ne, need_eq - eq_before));
  uint32_t kept = 0;
  for (; keep > 0; --keep) {   // the lowest `keep` positions equal to T
    const uint32_t low = e & (0u - e);
    kept |= low;
    e ^= low;
  }
  uint32_t sel = g | kept, sel_tot;
  uint32_t o = o_base + block_prefix_excl((uint32_t)__popc(sel), sh, 0, sel_tot);
  while (sel) {
    const int b = __builtin_ctz(sel);
    if (o < (uint32_t)k) out[o] = x * 32 + b;   // never more than k
    ++o;
    sel &= sel - 1u;
  }
  o_base += sel_tot;
  eq_base += eq_tot;
}

constexpr int kMapWords = 4096;                // bitmap words held in LDS (131072 positions)
constexpr int kWholeKeys = kMapWords * 32;     // longest prefix of topk_kernel
constexpr int kKeyBatch = 8;                   // keys per thread loaded together

// The whole top-k of one (b, j) per workgroup.  One workgroup reads a head's
// scores at about one CU's L2 rate (a microsecond per 4096 keys), which on
// short prefixes, or with enough heads to occupy the chip, costs less than a
// second launch and the round trip of bitmap and candidates through memory
// (one_launch; 1k, one head: classification 3.0 us + final 3.9 us, here 4.7).
// Short prefixes are bound by the chain of barriers, so the block scans use
// DPP within the waves and one barrier each.
__global__ void __launch_bounds__(kTopkThreads)
topk_kernel(const float* __restrict__ S, const uint32_t* __restrict__ hist,
            uint32_t* __restrict__ tws, int32_t* __restrict__ idx, int P, int k) {
  __shared__ TopkShared sh;
  __shared__ uint2 lcand[kTopkWaves * kLdsCap];
  __shared__ __attribute__((aligned(8))) uint32_t xgt[kMapWords], xeq[kMapWords];
  const int bj = blockIdx.x;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const float* Sj = S + (size_t)bj * P;
  float f[kKeyBatch];
#pragma unroll
  for (int i = 0; i < kKeyBatch; ++i)   // the first batch, in flight during the bin search
    f[i] = Sj[min(i * kTopkThreads + (int)threadIdx.x, P - 1)];
  const int W = (P + 31) / 32;
  for (int x = threadIdx.x; x < W; x += kTopkThreads) xeq[x] = 0u;
  hist_bin(hist, bj, k, sh);
  const uint32_t bin = sh.sel_bin;
  const int need = sh.sel_rem;
  // the wave's list: at most one entry per key it classifies, so the waves'
  // shares of the workspace (P entries in all) never meet
  Cands cs;
  cs.lds = lcand + w * kLdsCap;
  cs.ws = topk_ws(tws, bj, P).cand + (size_t)(P / kTopkThreads) * 64 * w + min(64 * w, P % kTopkThreads);
  cs.n = 0;
  // order keys of the bin: [k_lo, k_hi)  (k_hi wraps to 0 for the last bin)
  const uint32_t k_lo = bin << kHistShift, k_last = k_lo | ((1u << kHistShift) - 1u);
  for (int p0 = 0; p0 < P; p0 += kKeyBatch * kTopkThreads) {
    uint32_t u[kKeyBatch];
#pragma unroll
    for (int i = 0; i < kKeyBatch; ++i) u[i] = order_key(f[i]);
    if (p0 + kKeyBatch * kTopkThreads < P) {
#pragma unroll
      for (int i = 0; i < kKeyBatch; ++i)
        f[i] = Sj[min(p0 + (kKeyBatch + i) * kTopkThreads + (int)threadIdx.x, P - 1)];
    }
    uint32_t bits_lo = 0u, bits_hi = 0u;   // lane i: batch i's "in a higher bin" bits
#pragma unroll
    for (int i = 0; i < kKeyBatch; ++i) {
      const int pw = p0 + i * kTopkThreads + w * 64;   // the wave's first position
      if (pw >= P) break;
      const uint64_t in = P - pw >= 64 ? ~0ull : (1ull << (P - pw)) - 1ull;
      const uint64_t mg = __ballot(u[i] > k_last) & in;
      const uint64_t mc = __ballot(u[i] >= k_lo && u[i] <= k_last) & in;
      bits_lo = lane == i ? (uint32_t)mg : bits_lo;
      bits_hi = lane == i ? (uint32_t)(mg >> 32) : bits_hi;
      if (mc) {
        if ((mc >> lane) & 1ull) {
          const int r = cs.n + (int)__builtin_amdgcn_mbcnt_hi(
                                   (uint32_t)(mc >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)mc, 0u));
          const uint2 e = make_uint2(u[i], (uint32_t)(pw + lane));
          if (r < kLdsCap) cs.lds[r] = e;
          else cs.ws[r] = e;
        }
        cs.n += (int)__popcll(mc);
      }
    }
    const int pl = p0 + lane * kTopkThreads + w * 64;   // lane i writes batch i's two words
    if (lane < kKeyBatch && pl < P)
      *reinterpret_cast<uint2*>(&xgt[pl / 32]) = make_uint2(bits_lo, bits_hi);
  }
  __threadfence_block();   // list entries are read by other lanes of the wave
  __syncthreads();
  int need_eq;
  const uint32_t T = cand_threshold(cs, bin, need, sh, need_eq);
  for (int c = lane; c < cs.n; c += 64) {
    const uint2 e = cand_at(cs, c);
    const uint32_t bit = 1u << (e.y & 31);
    if (e.x > T) atomicOr(&xgt[e.y >> 5], bit);
    else if (e.x == T) atomicOr(&xeq[e.y >> 5], bit);
  }
  __syncthreads();
  uint32_t o_base = 0, eq_base = 0;
  for (int x0 = 0; x0 < W; x0 += kTopkThreads) {
    const int x = x0 + (int)threadIdx.x;
    const bool ok = x < W;
    emit_words(ok ? xgt[x] : 0u, ok ? xeq[x] : 0u, x, need_eq, k, idx + (size_t)bj * k, o_base,
               eq_base, sh);
  }
}

// Final top-k after the classification, one workgroup per (b, j):
//  1. the bin of the k-th largest key (from the classification) and the
//     candidates, of which each wave takes a contiguous share (its first
//     kLdsCap into LDS);
//  2. two digit passes over the candidates give T and how many keys equal
//     to T to take;
//  3. per window of kMapWords bitmap words: candidates above T and equal to
//     T are marked in two LDS bitmaps; then, one word (32 positions) per
//     thread and round, the positions in higher bins plus the marked ones
//     above T plus the lowest positions equal to T are written in ascending
//     order.
__global__ void __launch_bounds__(kTopkThreads)
topk_final_kernel(uint32_t* __restrict__ tws, int32_t* __restrict__ idx, int P, int k) {
  __shared__ TopkShared sh;
  __shared__ uint2 lcand[kTopkWaves * kLdsCap];
  __shared__ uint32_t xgt[kMapWords], xeq[kMapWords];
  const int bj = blockIdx.x;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const TopkWs f = topk_ws(tws, bj, P);
  const uint4 hdr = *reinterpret_cast<const uint4*>(f.ncand);
  const uint32_t bin = hdr.y;
  const int need = (int)hdr.z;
  Cands cs;
  const int nc = (int)min(hdr.x, (uint32_t)P), share = (nc + kTopkWaves - 1) / kTopkWaves;
  const int c0 = min(nc, w * share);
  cs.lds = lcand + w * kLdsCap;
  cs.ws = f.cand + c0;
  cs.n = min(nc, c0 + share) - c0;
  for (int c = lane; c < min(cs.n, kLdsCap); c += 64) cs.lds[c] = cs.ws[c];
  __syncthreads();
  int need_eq;
  const uint32_t T = cand_threshold(cs, bin, need, sh, need_eq);

  int32_t* out = idx + (size_t)bj * k;
  uint32_t o_base = 0, eq_base = 0;
  const int W = (P + 31) / 32;
  for (int m0 = 0; m0 < W; m0 += kMapWords) {
    const int m1 = min(W, m0 + kMapWords);
    for (int x = threadIdx.x; x < kMapWords; x += kTopkThreads) xgt[x] = xeq[x] = 0u;
    __syncthreads();
    for (int c = lane; c < cs.n; c += 64) {
      const uint2 e = cand_at(cs, c);
      const int x = (int)(e.y >> 5);
      if (x < m0 || x >= m1) continue;
      const uint32_t bit = 1u << (e.y & 31);
      if (e.x > T) atomicOr(&xgt[x - m0], bit);
      else if (e.x == T) atomicOr(&xeq[x - m0], bit);
    }
    __syncthreads();
    for (int x0 = m0; x0 < m1; x0 += kTopkThreads) {
      const int x = x0 + (int)threadIdx.x;
      const bool ok = x < m1;
      emit_words(ok ? f.gt[x] | xgt[x - m0] : 0u, ok ? xeq[x - m0] : 0u, x, need_eq, k, out, o_base,
                 eq_base, sh);
    }
    __syncthreads();   // the window's bitmaps are read before the next window clears them
  }
}

}  // namespace

// Whether topk_kernel takes a prefix of P keys of each of `heads` KV heads.
// The whole selection in microseconds, one launch / classification and final:
//   heads    16k            24k            32k            48k            64k            128k
//     1   17.6 /  17.6   20.0 /  19.9   22.0 /  20.1   27.2 /  23.0   31.8 /  26.3   48.8 /  33.4
//     8   19.0 /  19.8   25.8 /  25.9   29.6 /  29.5   39.4 /  36.9   47.4 /  43.9   84.8 /  75.6
//    16   28.0 /  28.9   34.8 /  34.9   41.8 /  41.5   55.1 /  54.0   70.1 /  67.8    143 /   136
//    24                  41.0 /  42.2   50.3 /  50.9   70.0 /  70.0    103 /  99.4    194 /   193
//    32   38.9 /  40.9   47.4 /  48.7   60.8 /  61.7    101 /   101    125 /   124    253 /   250
//    64   57.3 /  61.7   95.3 /  98.2    118 /   121    174 /   179    231 /   235    465 /   472
//   128    116 /   125    168 /   177    220 /   231    323 /   340    425 /   445
// The lines cross at about 24k keys up to 16 heads, then at 1536 per head; from
// 48 heads on (98k: 259.5 / 259.2, 128k: 353.3 / 353.3) they do not cross.
static bool one_launch(int heads, int P) {
  return P <= kWholeKeys && (P <= 24576 || heads >= 48 || P <= heads * 1536);
}

bool prefill_fuses(const hyq_shape& s, const QuantQ& qq) {
  return ((int64_t)s.B * s.Hq * kTailGroups + qq.count) * kTailThreads < (int64_t)1 << 32;
}

size_t select_topk_ws_bytes(int BH, int P) { return (size_t)BH * topk_ws_words(P) * 4; }

namespace {

template <int QFMT>
void launch_tail_proxy(const hyq_shape& s, const uint16_t* Q, float* qsum, uint32_t* hist,
                       uint32_t* tws, int t, int P, const QuantQ& qq, hipStream_t st) {
  const int BHq = s.B * s.Hq, n_tail = BHq * kTailGroups;
  static_assert(kTailThreads == kQuantThreads, "both kinds of workgroup share the launch");
  // a dimension of a launch holds fewer than 2^32 threads (prefill_fuses keeps
  // the two kinds together below that)
  const dim3 grid = qq.count ? dim3(n_tail + qq.count) : dim3(BHq, kTailGroups);
  tail_proxy_kernel<QFMT><<<grid, kTailThreads, 0, st>>>(Q, qsum, hist, tws, BHq, s.Hq / s.Hkv, s.L,
                                                         t, P, n_tail, qq);
}

template <int QFMT>
hipError_t launch_select_t(const hyq_shape& s, const hyq_sizes& z, const uint16_t* Q,
                           const uint16_t* K, int32_t* idx, float* scores, float* qsum,
                           uint32_t* hist, uint32_t* tws, float* cm_ws, const QuantQ& qq,
                           hipStream_t st) {
  const int g = s.Hq / s.Hkv;
  const int t = s.window < s.L ? s.window : s.L;
  const int BH = s.B * s.Hkv;
  // (KV head, key chunk) with the head index fastest: workgroups are spread
  // over the XCDs round-robin, so with B*Hkv a multiple of 8 every chunk of a
  // head (and its top-k workgroup) runs on one XCD and shares that XCD's L2.
  if (s.selector == HYQ_SEL_COLMASS) {
    const hipError_t e = launch_colmass_scores(s, z, Q, K, scores, hist, tws, topk_ws_words(z.P),
                                               cm_ws, st);
    if (e != hipSuccess) return e;
    launch_quant_q(qq, st);
  } else {
    launch_tail_proxy<QFMT>(s, Q, qsum, hist, tws, t, z.P, qq, st);
    score_kernel<<<dim3(BH, (z.P + kScoreRows - 1) / kScoreRows), kScoreThreads, 0, st>>>(
        K, qsum, scores, hist, g, s.L, z.P);
  }
  if (one_launch(BH, z.P)) {
    topk_kernel<<<BH, kTopkThreads, 0, st>>>(scores, hist, tws, idx, z.P, z.k);
  } else {
    const dim3 cg(BH, (z.P + kTopkThreads - 1) / kTopkThreads);
    topk_classify_kernel<<<cg, kTopkThreads, 0, st>>>(scores, hist, tws, z.P, z.k);
    topk_final_kernel<<<BH, kTopkThreads, 0, st>>>(tws, idx, z.P, z.k);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_select(const hyq_shape& s, const hyq_sizes& z, const uint16_t* Q,
                         const uint16_t* K, int32_t* idx, float* scores, float* qsum,
                         uint32_t* hist, uint32_t* tws, float* cm_ws, const QuantQ* qq,
                         hipStream_t st) {
  if (z.k == 0) return hipSuccess;
  const QuantQ q = qq ? *qq : QuantQ{};   // none: no blocks
#define HYQ_SELECT(F) \
  launch_select_t<F>(s, z, Q, K, idx, scores, qsum, hist, tws, cm_ws, q, st)
  return q.fmt == HYQ_FMT_FP4Q6 ? HYQ_SELECT(HYQ_FMT_FP4Q6)
         : q.fmt == HYQ_FMT_INT ? HYQ_SELECT(HYQ_FMT_INT)
                                : HYQ_SELECT(HYQ_FMT_FP8);
#undef HYQ_SELECT
}

}  // namespace hyq
