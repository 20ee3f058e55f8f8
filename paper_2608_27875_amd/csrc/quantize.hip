// Partition and per-block symmetric quantization: Algorithm 2, Stages 1-2
// (App. A.2) of HyQuant.
//
//   kq_pos  = [0, P) minus the vertical positions, ascending (the K_Q set of
//             the partition of Section 4.1);
//   Q       : blocks of 64 query rows per head;
//   K, V    : blocks of 64 consecutive entries of the compacted K_Q sequence
//             (rows gathered through kq_pos);
//   s = fl32(max|x| / c), code = clamp(rint(fl32(x / s)), -c, c), s = 0 ->
//   codes 0 (c = 127 for 8-bit, 7 for 4-bit);
//   FP8 codes (c = 448): the OCP E4M3 value nearest to fl32(x / s), ties to
//   even, saturating at +-448, zero keeping the sign (the hardware
//   float32 -> E4M3 conversion, which rounds to nearest even).
//
// Every quotient is the IEEE correctly rounded float32 quotient (for bf16
// inputs by the block's reciprocal and a residual correction, see
// recip_quotient) and rint rounds half to even, so codes match the definition
// bit for bit.  HBM-bound: each input row is read once, 16 bytes a load, and
// each code written once (Q 8 bytes a store, K and V 16).
#include "hyq_internal.h"
#include "quant_dev.h"

#pragma clang fp contract(off)

namespace hyq {
namespace {

typedef unsigned v4u __attribute__((ext_vector_type(4)));

// Number of the ascending a[0, n) with a[i] - i <= x: the vertical positions
// that precede the x-th (from 0) non-vertical one.
__device__ __forceinline__ int verticals_before(const int32_t* __restrict__ a, int n, int x) {
  return wave_search(n, [=](int i) { return a[i] - i <= x; });
}

// Positions of the 64 slots [n0, n0 + 64) of a head (the n-th non-vertical
// prefix position, n < nQ), one per row of the workgroup's block; -1 from nQ
// on.  kSpan entries of the vertical list are staged in LDS: those around
// where an evenly spread list would have the block's first slot, which is one
// dependent read; if they do not hold all the block needs, those that follow
// the first slot by search, and a row whose entries lie beyond them searches
// the list itself.  This replaces a launch of its own that wrote kq_pos for
// this kernel to read back.
constexpr int kSpan = kQuantThreads;
__device__ __forceinline__ int slot_position(const int32_t* __restrict__ idx, int k, int nQ,
                                             int n0, int row, int32_t* span) {
  const int n = n0 + row;
  if (k == 0) return n < nQ ? n : -1;
  int c0 = (int)min((int64_t)max(k - kSpan, 0),
                    max((int64_t)n0 * k / nQ - kSpan / 2, (int64_t)0));
  auto stage = [&] {
    const int i = c0 + (int)threadIdx.x;
    span[threadIdx.x] = i < k ? idx[i] - i : INT32_MAX;
    __syncthreads();
  };
  stage();
  // every entry before c0 must count for the first slot, none after the span for the last
  if (!((c0 == 0 || span[0] <= n0) && span[kSpan - 1] > n0 + kBlock - 1)) {
    c0 = verticals_before(idx, k, n0 - 1);
    __syncthreads();
    stage();
  }
  if (n >= nQ) return -1;
  int lo = 0, hi = kSpan;   // entries of the span with idx[i] - i <= n
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (span[mid] <= n) lo = mid + 1; else hi = mid;
  }
  int c = c0 + lo;
  if (lo == kSpan) {   // the span ends before the row's position: search the rest
    int l2 = c, h2 = k;
    while (l2 < h2) {
      const int mid = (l2 + h2) >> 1;
      if (idx[mid] - mid <= n) l2 = mid + 1; else h2 = mid;
    }
    c = l2;
  }
  return n + c;
}

// The Q blocks of a call that no other launch carries, one per workgroup.
template <int FMT>
__global__ void __launch_bounds__(kQuantThreads)
quant_q_kernel(QuantQ q) {
  __shared__ float red[kQuantThreads / 64];
  quant_q_block<FMT>(q, (int)(blockIdx.y * gridDim.x + blockIdx.x), red);
}

// The codes of a thread's 32 values of a block with scale s.
template <int FMT>
__device__ __forceinline__ void block_codes(const float (&x)[32], float s, float c, int (&o)[32]) {
  if (recip_ok(s)) {
    const float r = 1.0f / s;
#pragma unroll
    for (int e = 0; e < 32; ++e) o[e] = code_of<FMT>(quot<FMT>(x[e], s, r), c);
  } else if (s > 0.0f) {
#pragma unroll
    for (int e = 0; e < 32; ++e) o[e] = quant_code<FMT>(x[e], s, c);
  } else {
#pragma unroll
    for (int e = 0; e < 32; ++e) o[e] = 0;
  }
}

// Freeze's bf16 rows (64 cache rows per workgroup): the vertical-line rows
// (padded with zero rows to vl_rows) and the window, K row-major and V
// channel-major through an LDS tile; every other row is zeroed.
struct Gather {
  const int32_t* idx;
  uint16_t* fk;
  uint16_t* fv;
  int W, k, vl_rows, nfp;
};
typedef uint16_t GatherTile[kBlock][kHeadDim + 2];
__device__ __forceinline__ void gather_rows(const Gather& ga, const uint16_t* __restrict__ K,
                                            const uint16_t* __restrict__ V, int L, int bj, int blk,
                                            GatherTile& tile) {
  const int row = threadIdx.x >> 2, c0 = (threadIdx.x & 3) * 32;
  const int i = blk * kBlock + row;
  int src = -1;
  if (i < ga.k) src = ga.idx[(size_t)bj * ga.k + i];
  else if (i >= ga.vl_rows && i - ga.vl_rows < ga.W) src = L - ga.W + (i - ga.vl_rows);
  v4u kw[4], vw[4];
  if (src >= 0) {
    const v4u* kp = reinterpret_cast<const v4u*>(K + ((size_t)bj * L + src) * kHeadDim + c0);
    const v4u* vp = reinterpret_cast<const v4u*>(V + ((size_t)bj * L + src) * kHeadDim + c0);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      kw[u] = kp[u];
      vw[u] = vp[u];
    }
  } else {
#pragma unroll
    for (int u = 0; u < 4; ++u) kw[u] = vw[u] = v4u{0u, 0u, 0u, 0u};
  }
  v4u* kd = reinterpret_cast<v4u*>(ga.fk + ((size_t)bj * ga.nfp + i) * kHeadDim + c0);
#pragma unroll
  for (int u = 0; u < 4; ++u) kd[u] = kw[u];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      tile[row][c0 + u * 8 + 2 * e] = (uint16_t)(vw[u][e] & 0xffffu);
      tile[row][c0 + u * 8 + 2 * e + 1] = (uint16_t)(vw[u][e] >> 16);
    }
  }
  __syncthreads();
  // transposed write: thread -> (channel d, 32 rows)
  const int d = threadIdx.x >> 1, r0 = (threadIdx.x & 1) * 32;
  v4u o[4];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      o[u][e] = (uint32_t)tile[r0 + u * 8 + 2 * e][d] |
                ((uint32_t)tile[r0 + u * 8 + 2 * e + 1][d] << 16);
  v4u* vd = reinterpret_cast<v4u*>(ga.fv + ((size_t)bj * kHeadDim + d) * ga.nfp +
                                   (size_t)blk * kBlock + r0);
#pragma unroll
  for (int u = 0; u < 4; ++u) vd[u] = o[u];
}

// One workgroup per (b, j, compacted block).  Writes the block's kq_pos slots,
// K codes row-major, V codes channel-major (the block transposed) through an
// LDS tile.  cap_blocks is the number of blocks each (b, j) owns in the
// outputs; workgroups from n_blocks on gather Freeze's bf16 rows, then mark
// the slots of the blocks the cache still has free (neither in a prefill).
template <int BITS, int FMT>
__global__ void __launch_bounds__(kQuantThreads)
quant_kv_kernel(const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
                const int32_t* __restrict__ idx, int32_t* __restrict__ kq_pos,
                uint8_t* __restrict__ kc, float* __restrict__ ks, uint8_t* __restrict__ vc,
                float* __restrict__ vs, int L, int k, int nQ, int cap_blocks, int n_blocks,
                Gather ga) {
  static_assert((FMT != HYQ_FMT_FP8 || BITS == 8) && (FMT != HYQ_FMT_FP4 || BITS == 4),
                "FP8 codes are 8-bit, FP4 codes 4-bit");
  constexpr float C = code_bound<BITS, FMT>();
  constexpr int kRow = BITS == 8 ? kHeadDim : kHeadDim / 2;   // bytes per K code row
  constexpr int vRow = BITS == 8 ? kBlock : kBlock / 2;        // bytes per V code row (one channel)
  __shared__ float red[kQuantThreads / 64];
  typedef int8_t CodeTile[kBlock][kHeadDim + 4];                // V codes, [key][channel]
  __shared__ __attribute__((aligned(16))) uint8_t lds[sizeof(GatherTile)];
  static_assert(sizeof(CodeTile) <= sizeof(GatherTile), "one LDS tile serves both");
  __shared__ int32_t span[kSpan];
  const int bj = blockIdx.y, blk = blockIdx.x;
  const size_t slots = (size_t)cap_blocks * kBlock;
  if (blk >= n_blocks) {
    const int e = blk - n_blocks, n_gather = ga.nfp / kBlock;
    if (e < n_gather) {
      gather_rows(ga, K, V, L, bj, e, reinterpret_cast<GatherTile&>(lds));
    } else {
      const int n = n_blocks * kBlock + (e - n_gather) * kQuantThreads + (int)threadIdx.x;
      if ((size_t)n < slots) kq_pos[(size_t)bj * slots + n] = HYQ_KQ_POS_PAD;
    }
    return;
  }
  CodeTile& vt = reinterpret_cast<CodeTile&>(lds);
  const int row = threadIdx.x >> 2, c0 = (threadIdx.x & 3) * 32;
  const int n = blk * kBlock + row;
  float xk[32], xv[32];
  const int pos = slot_position(idx + (size_t)bj * k, k, nQ, blk * kBlock, row, span);
  if ((threadIdx.x & 3) == 0) kq_pos[(size_t)bj * slots + n] = pos < 0 ? HYQ_KQ_POS_PAD : pos;
  if ((unsigned)pos < (unsigned)L) {
    load32(K + ((size_t)bj * L + pos) * kHeadDim + c0, xk);
    load32(V + ((size_t)bj * L + pos) * kHeadDim + c0, xv);
  } else {
#pragma unroll
    for (int e = 0; e < 32; ++e) xk[e] = xv[e] = 0.0f;
  }
  float mk = 0.0f, mv = 0.0f;
#pragma unroll
  for (int e = 0; e < 32; ++e) {
    mk = fmaxf(mk, fabsf(xk[e]));
    mv = fmaxf(mv, fabsf(xv[e]));
  }
  const float sk = block_max(mk, red) / C;
  const float sv = block_max(mv, red) / C;
  if (threadIdx.x == 0) {
    ks[(size_t)bj * cap_blocks + blk] = sk;
    vs[(size_t)bj * cap_blocks + blk] = sv;
  }
  int ck[32], cv[32];
  block_codes<FMT>(xk, sk, C, ck);
  block_codes<FMT>(xv, sv, C, cv);
  // K: row-major codes
  uint8_t* kdst = kc + ((size_t)bj * slots + n) * kRow;
  if (BITS == 8) {
    uint32_t w[8];
#pragma unroll
    for (int e = 0; e < 8; ++e)
      w[e] = (uint32_t)(ck[4 * e] & 0xff) | ((uint32_t)(ck[4 * e + 1] & 0xff) << 8) |
             ((uint32_t)(ck[4 * e + 2] & 0xff) << 16) | ((uint32_t)(ck[4 * e + 3] & 0xff) << 24);
    uint4* d4 = reinterpret_cast<uint4*>(kdst + c0);
    d4[0] = make_uint4(w[0], w[1], w[2], w[3]);
    d4[1] = make_uint4(w[4], w[5], w[6], w[7]);
  } else {
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      uint32_t a = 0;
#pragma unroll
      for (int b = 0; b < 8; ++b) a |= (uint32_t)(ck[8 * e + b] & 0xf) << (4 * b);
      w[e] = a;
    }
    *reinterpret_cast<uint4*>(kdst + c0 / 2) = make_uint4(w[0], w[1], w[2], w[3]);
  }
  // V: stage codes, then write channel-major
#pragma unroll
  for (int e = 0; e < 32; ++e) vt[row][c0 + e] = (int8_t)cv[e];
  __syncthreads();
  {
    const int d = threadIdx.x >> 1, k0 = (threadIdx.x & 1) * 32;
    uint8_t* vdst = vc + (((size_t)bj * cap_blocks + blk) * kHeadDim + d) * vRow;
    if (BITS == 8) {
      uint32_t w[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        uint32_t a = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) a |= (uint32_t)(uint8_t)vt[k0 + 4 * e + b][d] << (8 * b);
        w[e] = a;
      }
      uint4* d4 = reinterpret_cast<uint4*>(vdst + k0);
      d4[0] = make_uint4(w[0], w[1], w[2], w[3]);
      d4[1] = make_uint4(w[4], w[5], w[6], w[7]);
    } else {
      uint32_t w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        uint32_t a = 0;
#pragma unroll
        for (int b = 0; b < 8; ++b) a |= (uint32_t)(vt[k0 + 8 * e + b][d] & 0xf) << (4 * b);
        w[e] = a;
      }
      *reinterpret_cast<uint4*>(vdst + k0 / 2) = make_uint4(w[0], w[1], w[2], w[3]);
    }
  }
}

}  // namespace

QuantQ quant_q_all(const hyq_shape& s, const hyq_sizes& z, const uint16_t* Q, int8_t* q_codes,
                   float* q_scale) {
  QuantQ q;
  q.Q = Q;
  q.qc = q_codes;
  q.qs = q_scale;
  q.L = s.L;
  q.n_qblk = z.n_qblk;
  // E4M3 queries for FP8 and FP4
  q.fmt = s.kv_format == HYQ_FMT_INT || s.kv_format == HYQ_FMT_FP4Q6 ? s.kv_format : HYQ_FMT_FP8;
  q.count = s.B * s.Hq * z.n_qblk;
  return q;
}

void launch_quant_q(const QuantQ& q, hipStream_t st) {
  if (q.count <= 0) return;
  const dim3 grid(q.n_qblk, q.count / q.n_qblk);
  if (q.fmt == HYQ_FMT_FP4Q6) quant_q_kernel<HYQ_FMT_FP4Q6><<<grid, kQuantThreads, 0, st>>>(q);
  else if (q.fmt == HYQ_FMT_FP8) quant_q_kernel<HYQ_FMT_FP8><<<grid, kQuantThreads, 0, st>>>(q);
  else quant_q_kernel<HYQ_FMT_INT><<<grid, kQuantThreads, 0, st>>>(q);
}

static void launch_kv(int bits, int fmt, const uint16_t* K, const uint16_t* V, const int32_t* idx,
                      int32_t* kq_pos, uint8_t* k_codes, float* k_scale, uint8_t* v_codes,
                      float* v_scale, int L, int k, int nQ, int n_blocks, int cap_blocks, int BHkv,
                      const Gather& ga, hipStream_t st) {
  const int n_pad = ((cap_blocks - n_blocks) * kBlock + kQuantThreads - 1) / kQuantThreads;
  const dim3 kg(n_blocks + ga.nfp / kBlock + n_pad, BHkv);
  if (kg.x == 0) return;
#define HYQ_KV(BITS, FMT)                                                                        \
  quant_kv_kernel<BITS, FMT><<<kg, kQuantThreads, 0, st>>>(K, V, idx, kq_pos, k_codes, k_scale,   \
                                                           v_codes, v_scale, L, k, nQ,            \
                                                           cap_blocks, n_blocks, ga)
  if (fmt == HYQ_FMT_FP4 || fmt == HYQ_FMT_FP4Q6) HYQ_KV(4, HYQ_FMT_FP4);   // the same E2M1 codes
  else if (fmt == HYQ_FMT_FP8) HYQ_KV(8, HYQ_FMT_FP8);
  else if (bits == 8) HYQ_KV(8, HYQ_FMT_INT);
  else HYQ_KV(4, HYQ_FMT_INT);
#undef HYQ_KV
}

void launch_quant_kv(const hyq_shape& s, const hyq_sizes& z, const uint16_t* K, const uint16_t* V,
                     const int32_t* idx, int32_t* kq_pos, uint8_t* k_codes, float* k_scale,
                     uint8_t* v_codes, float* v_scale, hipStream_t st) {
  launch_kv(s.bits_kv, s.kv_format, K, V, idx, kq_pos, k_codes, k_scale, v_codes, v_scale, s.L, z.k,
            z.nQ, z.n_kvblk, z.n_kvblk, s.B * s.Hkv, Gather{}, st);
}

hipError_t launch_freeze_kv(const hyq_dcache& c, const hyq_sizes& z, int N, const uint16_t* K,
                            const uint16_t* V, hipStream_t st) {
  Gather ga;
  ga.idx = c.vl_pos;
  ga.fk = static_cast<uint16_t*>(c.fp_k);
  ga.fv = static_cast<uint16_t*>(c.fp_v);
  ga.W = c.window;
  ga.k = c.n_vl;
  ga.vl_rows = c.vl_rows;
  ga.nfp = c.vl_rows + c.ring_rows;
  launch_kv(c.bits_kv, c.kv_format, K, V, c.vl_pos, c.q_pos, static_cast<uint8_t*>(c.k_codes),
            c.k_scale, static_cast<uint8_t*>(c.v_codes), c.v_scale, N, z.k, z.nQ, z.n_kvblk,
            c.cap_blocks, c.B * c.Hkv, ga, st);
  return hipGetLastError();
}

hipError_t launch_quantize(const hyq_shape& s, const hyq_sizes& z, const uint16_t* Q,
                           const uint16_t* K, const uint16_t* V, const int32_t* idx,
                           int8_t* q_codes, float* q_scale, uint8_t* k_codes, float* k_scale,
                           uint8_t* v_codes, float* v_scale, int32_t* kq_pos, hipStream_t st) {
  if (s.bits_kv == 16) return hipSuccess;
  launch_quant_q(quant_q_all(s, z, Q, q_codes, q_scale), st);
  launch_quant_kv(s, z, K, V, idx, kq_pos, k_codes, k_scale, v_codes, v_scale, st);
  return hipGetLastError();
}

}  // namespace hyq
