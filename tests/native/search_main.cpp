// Checks the search in merged intervals (hpop_search.h) on the host: against a
// linear scan for random lists of up to 700 components, and against the
// closed form for lists of up to 2^33 (a rule in place of their memory).
#define __host__
#define __device__
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>

#include "hpop_search.h"

using namespace hpop;

template <int PROBES, class N, class T>
static bool same_as_scan(std::mt19937_64& rng, int n, T width) {
  std::vector<T> cs(n);
  std::vector<long long> pl(n);
  for (int i = 0; i < n; ++i) cs[i] = (T)(rng() % (unsigned long long)width);
  std::sort(cs.begin(), cs.end());
  n = (int)(std::unique(cs.begin(), cs.end()) - cs.begin());
  for (int i = 0; i < n; ++i) pl[i] = i ? pl[i - 1] + 1 + (long long)(rng() % 9) : (long long)(rng() % 5);
  const long long bs = n ? pl[n - 1] + 7 : 3;
  for (int q = 0; q < 40; ++q) {
    T x = q % 4 == 0 && n ? cs[rng() % n] : (T)(rng() % (2ull * (unsigned long long)width));
    if (q % 8 == 1) x = x + 1;
    int want = -1;
    while (want + 1 < n && cs[want + 1] < x) ++want;
    T c;
    long long p, next;
    bool inside = true;
    const bool any = find_comp<PROBES>(
        [&](N k, T& s, long long& m) {
          inside = inside && k >= 0 && k < n;
          if (!inside) return;
          s = cs[(size_t)k];
          m = pl[(size_t)k];
        },
        (N)n, x, width, bs, c, p, next);
    if (!inside || any != (want >= 0) || next != (want + 1 < n ? pl[want + 1] : bs)) return false;
    if (any && (c != cs[want] || p != pl[want])) return false;
  }
  return true;
}

int main() {
  std::mt19937_64 rng(3);
  for (int rep = 0; rep < 3000; ++rep) {
    const int n = (int)(rng() % (rep % 3 ? 40 : 700));
    if (!same_as_scan<3, int, unsigned int>(rng, n, 1 + (unsigned int)(rng() % (1u << 30))) ||
        !same_as_scan<5, long long, long long>(rng, n, 1 + (long long)(rng() % (1ull << 50))))
      return std::printf("FAIL list %d of %d\n", rep, n), 1;
  }
  // entry k: starts at 1000 k + k % 700, measure 300 k
  for (long long n : {1ll << 20, (1ll << 31) - 1, 1ll << 31, (1ll << 31) + 5, 1ll << 32, 1ll << 33}) {
    auto start = [](long long k) { return 1000 * k + k % 700; };
    for (int q = 0; q < 2000; ++q) {
      const long long want = q < 4 ? n - 1 - q : (long long)(rng() % (unsigned long long)n);
      const long long x = start(want) + 1 + (long long)(rng() % 300);
      long long c, p, next;
      bool inside = true;
      const bool any = find_comp<5>(
          [&](long long k, long long& s, long long& m) {
            inside = inside && k >= 0 && k < n;
            s = start(k);
            m = 300 * k;
          },
          n, x, start(n - 1) + 1, 300 * n, c, p, next);
      if (!inside || !any || c != start(want) || p != 300 * want || next != 300 * (want + 1))
        return std::printf("FAIL %lld of %lld\n", want, n), 1;
    }
  }
  std::printf("ok\n");
  return 0;
}
