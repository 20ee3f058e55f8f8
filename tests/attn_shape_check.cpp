// Prints the prefill attention's launch shape for each case read from stdin:
// "units heads tiles bf16 n_cu" per line -> "kind grid fold".
#include <cstdio>

#include "attn_shape.h"

int main() {
  long long units, heads, tiles, n_cu;
  int bf16;
  while (std::scanf("%lld %lld %lld %d %lld", &units, &heads, &tiles, &bf16, &n_cu) == 5) {
    const hyq::AttnShape s = hyq::choose_attn_shape(units, heads, tiles, bf16 != 0, n_cu);
    std::printf("%d %lld %d\n", (int)s.kind, (long long)s.grid, s.fold);
  }
  return 0;
}
