// Checks on the host that a start which the scatter lets into a segment's
// buckets (start_in_range) is looked for in the same bucket later
// (bucket_index), also past the range that the geometry was made from: a
// sampled range need not hold every start.
#define __host__
#define __device__
#include <cstdio>
#include <random>

#include "hpop_geom.h"

using namespace hpop;

int main() {
  std::mt19937_64 rng(99);
  long long in = 0, past = 0;
  for (int nb : {1, 2, 3, 100, 46342, 1 << 17, 1 << 20, (1 << 24) - 1, 1 << 24}) {
    for (int bits : {1, 20, 30, 31, 32, 40, 55, 61}) {
      for (int rep = 0; rep < 64; ++rep) {
        // spans up to and just below a power of two: 31 bits of it are the bucket index's numerator
        const unsigned long long top = 1ull << bits;
        const unsigned long long span = rep % 4 == 0 ? top - 1 : rep % 4 == 1 ? top - 1 - rng() % (top / 2 + 1) / 1024
                                                                              : top / 2 + rng() % (top / 2 + 1);
        const unsigned long long min_s = 1000 + rng() % (1ull << 61);
        const Geom g = make_geom(SegStats{min_s, min_s + span, 0, 0}, SegDesc{0, nb, 2});
        const unsigned long long end = (unsigned long long)nb * g.wx << g.s0;  // of the last bucket
        for (int i = 0; i < 64; ++i) {
          // around the range's end, the last bucket's and 2^31 units, and anywhere
          const unsigned long long at[] = {span, end, 1ull << (31 + g.s0), span + rng() % (end - span + 1), rng() % (end + 1)};
          const unsigned long long rel = at[i % 5] + rng() % 5 - (at[i % 5] >= 2 ? 2 : 0);
          const long long s = (long long)(min_s + rel);
          if (rel <= span && !start_in_range(g, s)) return std::printf("FAIL refused nb=%d span=%llu rel=%llu\n", nb, span, rel), 1;
          if (!start_in_range(g, s)) continue;
          ++in;
          past += rel > span;
          const long long b = bucket_of_start(g, s), lo = bucket_lo(g, b);
          if (b < 0 || b >= nb || lo > s || (unsigned long long)(s - lo) >= (unsigned long long)g.wx << g.s0)
            return std::printf("FAIL outside its bucket nb=%d span=%llu rel=%llu\n", nb, span, rel), 1;
          if (bucket_index(g, rel) != b)
            return std::printf("FAIL looked for in bucket %lld, put into %lld: nb=%d span=%llu rel=%llu\n",
                               (long long)bucket_index(g, rel), b, nb, span, rel), 1;
        }
        for (long long d : {1ll, 2ll, 1000ll})
          if (start_in_range(g, (long long)min_s - d)) return std::printf("FAIL before the range\n"), 1;
      }
    }
  }
  std::printf("ok %lld starts, %lld past the range\n", in, past);
  return 0;
}
