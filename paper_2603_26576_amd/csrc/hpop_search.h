// Search in a sorted list of merged intervals: the same code on the device
// (kernels) and the host (CPU tests).
#pragma once

namespace hpop {

// The last of cnt components that starts before x (both relative to the first
// time of what holds them, width long): its start and measure and the next
// one's measure (bs after the last). False: none starts before x, and next is
// the first one's measure.
//
// A query is a chain of dependent loads, one cache miss each, so what counts
// is the number of probes. Starts spread about evenly over their bucket:
// each probe takes the place that the starts known so far on both sides of x
// suggest and reads two neighbours, which mostly ends after three or four
// probes where halving took nine (a 350-record bucket) and then read the
// result's words in two more. Buckets with their starts in a few places get
// halving after PROBES of them. Against halving alone the region stage of a
// batch of 128 traces (512 regions) takes 32 us instead of 39, that of 256
// devices with their streams 17.6 instead of 20, the mid trace's the same.
// N counts the components: a bucket's fit an int, a serving list may hold more
// than 2^31 of 16 B in 288 GB.
template <int PROBES = 3, class N, class T, class Load>
__host__ __device__ inline __attribute__((always_inline)) bool find_comp(Load load, N cnt, T x, T width, long long bs,
                                                                         T& cs, long long& pl, long long& next) {
  N L = -1, H = cnt;
  T csL = 0, csH = width;
  long long plL = 0, plH = bs;
  for (int it = 0; H - L > 1; ++it) {
    N k = (L + H) >> 1;
    if (it < PROBES) {
      const float f = x >= csH ? 1.0f : (float)(x - csL) / (float)(csH - csL);
      k = L + (N)(f * (float)(H - L - 1) + 0.5f);
      k = k <= L ? L + 1 : (k >= H ? H - 1 : k);
    }
    const bool two = k + 1 < H;
    T c0, c1;
    long long p0, p1;
    load(k, c0, p0);
    load(two ? k + 1 : k, c1, p1);
    if (c0 >= x) {
      H = k;
      csH = c0;
      plH = p0;
    } else {
      L = k;
      csL = c0;
      plL = p0;
      if (two) {
        if (c1 >= x) {
          H = k + 1;
          csH = c1;
          plH = p1;
        } else {
          L = k + 1;
          csL = c1;
          plL = p1;
        }
      }
    }
  }
  cs = csL;
  pl = plL;
  next = plH;
  return L >= 0;
}

}  // namespace hpop
