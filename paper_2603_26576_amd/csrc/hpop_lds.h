// LDS layouts of the merge kernels (plain C++: the CPU tests read them too).
#pragma once
#include <stdint.h>

#include "hpop_internal.h"

namespace hpop {

constexpr int kWaveCap = 512;   // records one wave sorts and flattens on its own
constexpr int kWaveBins = 512;  // sub-bins of the wave path's counting sort (at most)

// The wave path's area.
struct alignas(16) WaveSmem {
  unsigned int key[kWaveCap];        // sorted keys (then, with end[], the components of one level)
  unsigned int end[kWaveCap];        // ends of the sorted records
  unsigned int bins[kWaveBins / 2];  // two 16-bit counters (then sub-bin starts) per word
};

// Of the groups that sort records with 64-bit keys (one bucket or one list tile at a time).
template <int THREADS, int CAP>
struct alignas(16) SortSmem {
  static constexpr int NW = THREADS / 64;
  Elem E[CAP];
  unsigned short ordA[CAP];
  unsigned short ordB[CAP];
  unsigned int whist[THREADS < 256 ? 1 : NW * 256];  // the radix passes' (a thread per digit)
  unsigned int dstart[THREADS < 256 ? 1 : 256];
  unsigned int dcount[THREADS < 256 ? 1 : 256];
  long long lds_scan[NW * 6];
  unsigned long long red[2][NW];
};

// k_merge_rest: first a bucket for the whole workgroup, then, with no barrier
// between them, a bucket for each wave, which goes through `w`, `one` or both.
// A wave's two areas share its own place and no other wave's.
template <int THREADS, int CAP>
union RestSmem {
  SortSmem<THREADS, CAP> block;
  union Wave {
    WaveSmem w;
    SortSmem<64, kWaveCap> one;
  } wave[THREADS / 64];
};

}  // namespace hpop
