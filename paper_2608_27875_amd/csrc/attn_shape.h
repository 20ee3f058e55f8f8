// Host-side choice of the prefill attention's launch shape.  Plain C++ (no
// HIP), so that the policy can be checked on any host.
//
// A work unit is 32 query rows of one head, one wave's work.  The full-chip
// shape takes 8 units per workgroup, one workgroup per CU, every K/V tile
// staged once for all 8; it is the cheapest per tile but a workgroup's time
// is its longest unit's serial scan, so it needs many workgroups per CU.
//
// Measured on 256 CUs (microseconds; U units in all, T key tiles of 64):
//
//     U     T     kFull  kHalf  kSplit2  kSplit8
//   int8 codes, window 128, 2% vertical lines
//   1280     2     21.8   22.7
//    256     4     25.4   21.9     21.7     18.7
//    320     8     32.1   27.5     28.6     30.4
//   1024     8     34.1   29.4     31.0     60.9
//    384    16     41.7   34.6     34.3     32.8
//    512    16     41.8   34.4     34.6     35.1
//   1024    16     43.1   36.2     36.5     64.7
//    512    32     60.6   48.8     46.8     41.7
//    640    32     62.2   49.8     47.7     55.4
//   1280    32     62.1   52.2     58.1     92.9
//   1280    64      102   81.8     74.3      123
//   1536    64      102   83.2     84.0      144   (FP8 76.0, 78.9; int4 90.2, 85.3)
//   2048    64      106   89.6     98.5      186
//   2048   128      187    155      154      273
//   2304    32     66.1   73.7     93.3      166
//   int8 codes, half of the keys in full precision
//    264    12     42.7   38.4     35.9     31.4
//   1280    32     78.5   74.1     61.8      116
//   1536    48      108    103     82.5      167
//   int8 codes, three quarters
//   1024     4     26.9   24.2     27.9     64.4
//   1284     6     32.5   35.0
//   1536    12     45.9   44.6     53.3      114
//   1536    16     54.1   52.6     56.6      127
//   2016    48      127    128      119      310
//   int8 codes, all of them (a window as long as the prompt)
//    512    16     49.5   50.8     39.3     45.5
//    512    64      161    171      119      116
//   1024     4     22.4   21.6     21.1     47.0
//   1280     8     32.8   33.6     34.3     73.8
//   2048    16     52.3   54.7     54.6      161
//   2048    32     91.4   96.1     82.3      246
//   per-query window, nine tenths of the prompt
//   1152     9     38.4   38.2     33.5
//   1344     7     37.8   39.5     35.5            (last workgroups not full)
//   2016    14     63.6   65.6     66.2            (FP8, 288 kFull workgroups)
//   per-query window, all of the prompt
//    512     2     13.4   14.3     14.6            (4 units a head)
//   1152     9     37.4   40.1     33.0
//   1440    18     65.9   70.4     51.0
//   1536    48      163    171      114
//   2016    14     54.9   58.0     59.1
//   2016    18     67.1   71.1     66.8
//   nothing quantized
//    256     4     16.7   14.2     15.8     14.4
//    320     4     17.0   14.5     16.0     20.1
//    256     8     22.9   20.8     19.9     20.7
//   1024     8     25.1   22.9     22.5     54.1
//   1280     8     25.4   25.0     27.7     66.0
//    256    16     35.5   33.6     28.7     29.6
//    512    16     35.9   34.2     29.5     40.8
//   1280    16     37.4   37.1     33.6     92.4
//   2048    16     39.9   39.8     43.8      143
//   2048    32     65.9   65.9     62.9      214
//   2304    32     67.5   71.4     80.2      248
//
// kSplit8 wins while the units fit the CUs once, and with longer scans twice
// (int4 and FP4 codes, whose loads are half, about three times from T = 64
// on: 640 units 59 us against 74 with kSplit2; the line is the other formats').
// With nothing quantized it has only its own key-list stage to set against
// the others' dense pipeline and leads on the shortest scans alone.  kSplit2
// holds 4 units, so its staging is shared by fewer waves, and pays as the
// scans get longer: from `once` tiles on while its workgroups fit the CUs
// once, from `half_more` up to one and a half times, from `twice` up to twice.
// Below those kHalf, whose two workgroups per CU cover each other's waits,
// except (`half_many`) where there are two and the scan is a few tiles (a tile
// more where the last workgroup of a head is not full); the key-list stage of
// full-precision keys leaves them nothing to cover, so where that is most of
// the work kFull is at least as good, unless its workgroups (8 units each, the
// last of a head not full) are more than the CUs and the scan is short (2044
// units of 73 heads, 7 tiles: kFull 51.3, kHalf 36.0; 2016 of 72, 14 tiles:
// 43.3, 48.1).  With a per-query window the smaller workgroups also list fewer
// keys (1536 units, 3 tiles, FP4: kFull 32.1, kHalf 27.4; 516 units, 6 tiles:
// kHalf 33.4, kSplit2 30.4), the less so the more of the prompt the window is;
// a window of all of it is one more scan of listed keys.
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

// How the keys of a row are read: coded for the most part, all of them as
// dense rows, a mixed or a mostly listed (full-precision) scan, or a per-query
// window, whose key list grows with the rows of a workgroup until the window
// is most of the prompt, or all of it.
enum class AttnKeys { kCoded, kDense, kMixed, kListed, kBanded, kBandedWide, kBandedAll };

// `full` of the L keys of the last row are vertical lines or in its window;
// dense = nothing is quantized, band = the window is per query.  kHalf against
// kFull with 12 or 14 tiles and 1280 units: 0.96 to 0.98 of the time at a share
// of 0.4, 0.97 to 1.01 at 0.5, 0.98 to 1.03 at 0.65, 1.00 to 1.05 at 0.75, 1.04
// to 1.09 at 0.9.
inline AttnKeys attn_keys(int64_t full, int64_t L, bool dense, bool band) {
  if (dense) return AttnKeys::kDense;
  if (band)
    return 100 * full >= 97 * L ? AttnKeys::kBandedAll
           : 4 * full >= 3 * L ? AttnKeys::kBandedWide : AttnKeys::kBanded;
  return 50 * full >= 31 * L ? AttnKeys::kListed
         : 5 * full >= 2 * L ? AttnKeys::kMixed : AttnKeys::kCoded;
}

// units per KV head, `heads` KV heads (B * Hkv) in the launch, `tiles` =
// ceil(L / 64), n_cu compute units.
inline AttnShape choose_attn_shape(int64_t units, int64_t heads, int64_t tiles, AttnKeys keys,
                                   int64_t n_cu) {
  struct Lines {   // tiles from which ...
    int64_t once, half_more, twice;   // kSplit2, see above
    int64_t half_many;                // kHalf takes more workgroups than CUs
  };
  constexpr int64_t kNever = (int64_t)1 << 40, kSplit8Twice = 16, kDenseSplit8 = 12,
                    kSecondTurn = 12;
  static constexpr Lines kLines[] = {
      {12, 96, 128, 3},        // kCoded
      {8, 12, 24, 4},          // kDense
      {12, 24, 48, 3},         // kMixed
      {5, 20, 32, kNever},     // kListed
      {5, 96, 128, 0},         // kBanded
      {5, 9, 14, 0},           // kBandedWide
      {5, 9, 18, kNever},      // kBandedAll
  };
  const Lines& t = kLines[(int)keys];
  const int64_t n4 = (units + 3) / 4, n8 = (units + 7) / 8;
  const int64_t all = units * heads, wg4 = n4 * heads;
  if (keys == AttnKeys::kDense ? all <= n_cu && tiles < kDenseSplit8
                               : all <= n_cu || (all <= 2 * n_cu && tiles >= kSplit8Twice))
    return {AttnKind::kSplit8, all, 0};
  if ((wg4 <= n_cu && tiles >= t.once) || (2 * wg4 <= 3 * n_cu && tiles >= t.half_more) ||
      (wg4 <= 2 * n_cu && tiles >= t.twice))
    return {AttnKind::kSplit2, wg4, 0};
  // Whether kHalf's workgroups cover each other's waits.  Where not, they must
  // spread a head over more CUs, or spare kFull a second turn of short scans.
  const bool covers = t.half_many != kNever;
  if (wg4 <= n_cu ? covers || n4 > n8
                  : wg4 <= 2 * n_cu && (tiles >= t.half_many + (units % 4 != 0) ||
                                        (n8 * heads > n_cu && (covers || tiles < kSecondTurn))))
    return {AttnKind::kHalf, wg4, (int)(n_cu / heads)};
  return {AttnKind::kFull, n8 * heads, 0};
}

}  // namespace hyq
