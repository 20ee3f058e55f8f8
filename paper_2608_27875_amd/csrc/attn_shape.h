// Host-side choice of the prefill attention's launch shape.  Plain C++ (no
// HIP), so that the policy can be checked on any host.
//
// A work unit is 32 query rows of one head, one wave's work.  The full-chip
// shape takes 8 units per workgroup, one workgroup per CU, every K/V tile
// staged once for all 8; it is the cheapest per tile but a workgroup's time
// is its longest unit's serial scan, so it needs many workgroups per CU.
// Measured on 256 CUs (int8, microseconds; U units in all, T key tiles):
//
//      U     T     kFull  kHalf  kSplit2  kSplit8
//     32    16      43.7   33.4     33.2     19.5
//    256    16      41.0   33.4     33.6     20.9
//    500    63      97.4   77.3     67.2     51.7
//    512     8      32.3   27.1     28.2     32.2
//   1000    63     102.3   79.3     70.9     95.4
//   1376   172     237.4  179.8    156.7    253.0
//   1504    24      50.3   43.5     59.4    100.3
//   2000   125     183.0  150.1    150.1    264.2
//   2000   250     349.1  275.4    259.4    436.7
//   2016    32      64.8   54.9     71.6    141.6
//   2520    32      69.5   72.0     98.8    175.6
//   4000    63     142.3  144.0    186.5    360.6
//   8192   128     484      508      595     1080
//
// kSplit8 wins while the units fit the CUs about twice, unless a unit is so
// short that its fixed work (about 16 us) is all there is; kSplit2 while its
// workgroups of 4 units fit the CUs once (or twice, when the scans are long,
// or everything is full precision, where the shared staging weighs more than
// kHalf's overlap of two workgroups: kHalf 38.6, 54.9, 70.5, 151.6, 117.4
// against kSplit2 32.6, 46.8, 68.3, 118.8, 105.3 at U, T = 1120, 18; 1504, 24;
// 2016, 32; 1376, 86; 2000, 63); kHalf while its workgroups of 4 units
// are all resident, two per CU.
#pragma once

#include <cstdint>

namespace hyq {

enum class AttnKind {
  kFull,     // 8 units per workgroup, one workgroup per CU
  kHalf,     // 4 units per workgroup, two workgroups per CU
  kSplit2,   // 4 units per workgroup, keys split over two groups of 4 waves
  kSplit8,   // 1 unit per workgroup, keys split over 8 waves
};

struct AttnShape {
  AttnKind kind;
  int64_t grid;   // workgroups, a multiple of the KV heads
  int fold;       // kHalf: workgroups per KV head that come longest first (the rest come
                  // shortest first, so that the two on a CU are long and short)
};

// units per KV head, `heads` KV heads (B * Hkv) in the launch, `tiles` =
// ceil(L / 64), bf16 = nothing quantized, n_cu compute units.
inline AttnShape choose_attn_shape(int64_t units, int64_t heads, int64_t tiles, bool bf16,
                                   int64_t n_cu) {
  const int64_t n4 = (units + 3) / 4, n8 = (units + 7) / 8;
  const int64_t all = units * heads, wg4 = n4 * heads;
  if (all <= n_cu || (all <= 2 * n_cu && tiles >= 16))
    return {AttnKind::kSplit8, all, 0};
  if (wg4 <= n_cu || (wg4 <= 2 * n_cu && (bf16 || tiles >= 128)))
    return {AttnKind::kSplit2, wg4, 0};
  if (wg4 <= 2 * n_cu) return {AttnKind::kHalf, wg4, (int)(n_cu / heads)};
  return {AttnKind::kFull, n8 * heads, 0};
}

}  // namespace hyq
