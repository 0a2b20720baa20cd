// Checks when start ranges are sampled again after a miss (hpop_range.h).
#include <cstdio>

#include "hpop_range.h"

using hpop::RangeChoice;

// builds of `n` sets of records, of which those with odd(i) miss: returns the builds made
template <class Odd>
static int builds(RangeChoice& c, int n, Odd odd) {
  int made = 0;
  for (int i = 0; i < n; ++i) {
    if (i) c.new_records();
    for (int again = 0; again < 3; ++again) {  // the same records three times
      ++made;
      if (c.exact) continue;
      if (odd(i)) {
        c.missed();
        ++made;
        if (!c.exact) return -1;
      } else {
        c.held();
      }
    }
  }
  return made;
}

int main() {
  RangeChoice one;
  // one odd set: its own second build, and the next set is sampled again
  if (builds(one, 10, [](int i) { return i == 3; }) != 31 || one.exact) return std::printf("FAIL one\n"), 1;
  RangeChoice all;
  const int extra = builds(all, 64 * 64, [](int) { return true; }) - 3 * 64 * 64;
  if (extra > 64 + 6 || extra < 60) return std::printf("FAIL all: %d\n", extra), 1;
  // a row of misses is forgotten once a sample held
  for (int i = 0; i < 200; ++i) all.new_records();
  if (all.exact) return std::printf("FAIL still exact\n"), 1;
  all.held();
  all.missed();
  all.new_records();
  if (all.exact) return std::printf("FAIL after held\n"), 1;
  std::printf("ok\n");
  return 0;
}
