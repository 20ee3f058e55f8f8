// Prints the prefill attention's launch shape for each case read from stdin:
// "units heads L full mode n_cu" per line (full: keys of the last row in full
// precision; mode: 1 nothing quantized, 2 per-query window, 0 neither) ->
// "kind grid fold keys".
#include <cstdio>

#include "attn_shape.h"

int main() {
  long long units, heads, L, full, n_cu;
  int mode;
  while (std::scanf("%lld %lld %lld %lld %d %lld", &units, &heads, &L, &full, &mode, &n_cu) == 6) {
    const hyq::AttnKeys keys = hyq::attn_keys(full, L, mode == 1, mode == 2);
    const hyq::AttnShape s = hyq::choose_attn_shape(units, heads, (L + 63) / 64, keys, n_cu);
    std::printf("%d %lld %d %d\n", (int)s.kind, (long long)s.grid, s.fold, (int)keys);
  }
  return 0;
}
