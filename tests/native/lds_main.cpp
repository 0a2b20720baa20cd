// Checks the LDS layout of k_merge_rest on the host: whichever of its two
// areas each wave of a workgroup uses, no two waves' bytes overlap, and the
// workgroups that its launch bounds ask for fit a CU's 160 KB.
#include <cstdio>

#include "hpop_lds.h"

using namespace hpop;

template <class A, class B>
static bool apart(const A& a, const B& b) {
  const char *a0 = (const char*)&a, *a1 = (const char*)(&a + 1), *b0 = (const char*)&b, *b1 = (const char*)(&b + 1);
  return a1 <= b0 || b1 <= a0;
}

template <int THREADS, int CAP>
static int check(int per_cu) {
  static RestSmem<THREADS, CAP> u;
  constexpr int NW = THREADS / 64;
  for (int i = 0; i < NW; ++i) {
    if ((size_t)((const char*)&u.wave[i].w - (const char*)&u) % 16) return std::printf("FAIL alignment of wave %d\n", i), 1;
    if (apart(u.wave[i].w, u.block) || apart(u.wave[i].one, u.block)) return std::printf("FAIL wave %d outside\n", i), 1;
    for (int j = 0; j < NW; ++j) {
      if (i == j) continue;
      if (!apart(u.wave[i].w, u.wave[j].w) || !apart(u.wave[i].w, u.wave[j].one) ||
          !apart(u.wave[i].one, u.wave[j].w) || !apart(u.wave[i].one, u.wave[j].one))
        return std::printf("FAIL waves %d and %d share LDS\n", i, j), 1;
    }
  }
  if (sizeof u != sizeof u.block) return std::printf("FAIL size %zu\n", sizeof u), 1;
  if (per_cu * sizeof u > 160 * 1024) return std::printf("FAIL %d workgroups of %zu B\n", per_cu, sizeof u), 1;
  return 0;
}

int main() {
  if (check<256, 2048>(3) || check<256, 4096>(1)) return 1;
  std::printf("ok\n");
  return 0;
}
