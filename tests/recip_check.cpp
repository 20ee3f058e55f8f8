// Exhaustive check of recip_quotient: for each bound c, every amax mantissa,
// every x mantissa and every exponent difference down to quotients that round
// to code 0 in every format.  Scaling amax and x by a power of two scales
// every step alike, so one binade of amax stands for all that recip_ok
// admits; its ends are checked too.  Prints the number of pairs and of
// mismatches.
#include <cmath>
#include <cstdio>
#include <initializer_list>

#include "recip_quotient.h"

int main() {
  long pairs = 0, bad = 0;
  for (float c : {127.0f, 7.0f, 448.0f, 6.0f, 7.5f})
    for (int scale : {0, -60, -57, 119})   // s near 1 and near both ends of the range
      for (int ma = 128; ma < 256; ++ma) {
        const float amax = std::ldexp((float)ma, scale);
        const float s = amax / c, r = 1.0f / s;
        if (!hyq::recip_ok(s)) continue;
        for (int d = 0; d <= 22; ++d)
          for (int mx = 128; mx < 256; ++mx) {
            const float x = std::ldexp((float)mx, scale - d);
            if (x > amax) continue;
            for (float v : {x, -x}) {
              ++pairs;
              bad += hyq::recip_quotient(v, s, r) != v / s;
            }
          }
      }
  std::printf("%ld %ld\n", pairs, bad);
  return bad != 0;
}
