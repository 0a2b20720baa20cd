// Device building blocks shared by the trace-reduction and serving kernels.
#pragma once
#include <hip/hip_runtime.h>

#include <climits>

#include "hpop_geom.h"
#include "hpop_internal.h"
#include "hpop_lds.h"
#include "hpop_search.h"

namespace hpop {

// ----------------------------------------------------------------------------
// small device helpers
// ----------------------------------------------------------------------------

__device__ __forceinline__ int bitlen64(unsigned long long x) { return x ? 64 - __clzll((long long)x) : 0; }

__device__ __forceinline__ bool rec_valid(long long s, long long e) {
  // 0 <= s <= e < 2^62: a negative one is above every other as an unsigned word
  return (unsigned long long)s <= (unsigned long long)e && (unsigned long long)e < (unsigned long long)kTimeLimit;
}

__device__ __forceinline__ Geom seg_geom(const Plan& p, long long seg) { return p.geom[seg]; }

// The components of one bucket at one level, in either storage form.
struct CompView {
  const Comp* wide;     // wide segments
  const CompN* narrow;  // narrow segments: relative to lo
  long long lo;
  __device__ __forceinline__ long long cs(long long k) const {
    return narrow ? lo + (long long)narrow[k].cs : wide[k].cs;
  }
  __device__ __forceinline__ long long pl(long long k) const {
    return narrow ? (long long)narrow[k].pl : wide[k].pl;
  }
};

__device__ __forceinline__ CompView comp_view(const Plan& p, const Geom& g, long long bucket_begin, long long gb,
                                              int l) {
  CompView v;
  const long long off = (long long)p.offsets[gb];
  if (seg_narrow(g)) {
    v.wide = nullptr;
    v.narrow = p.compn[l] + off;
    v.lo = bucket_lo(g, gb - bucket_begin);
  } else {
    v.wide = p.comp[l] + off;
    v.narrow = nullptr;
    v.lo = 0;
  }
  return v;
}

// The records of one bucket: n8 in the 8 B form, n16 in the 16 B form.
struct BucketRecs {
  const uint2* narrow;
  const Elem* wide;
  int n8, n16;
  bool overflow;  // more records than fixed slots: the build is redone with exact offsets
};

__device__ __forceinline__ BucketRecs bucket_recs(const Plan& p, long long gb) {
  BucketRecs r;
  const unsigned long long cu = p.cursor[gb];
  r.n8 = (int)(unsigned int)cu;
  r.n16 = (int)(cu >> 32);
  long long ub, ucap;
  if (p.slot_cap) {
    ub = 2 * gb * (long long)p.slot_cap;
    ucap = 2 * (long long)p.slot_cap;
    r.overflow = (long long)r.n8 + r.n16 > (long long)p.slot_cap;
  } else {
    ub = 2 * (long long)p.offsets[gb];
    ucap = 2 * ((long long)r.n8 + r.n16);
    r.overflow = false;
  }
  const uint2* u = (const uint2*)p.elems;
  r.narrow = u + ub;
  r.wide = (const Elem*)(u + ub + ucap) - r.n16;
  return r;
}

// The 16 B form of an 8 B record of the bucket starting at lo. A clamped end
// (field 0xFFFFFFFF) becomes the largest end of the bucket's records of the
// same rank (maxend: per rank): every clamped record of a rank reaches past
// lo + 2^32 - 2 and starts before lo + 2^30, so they all overlap, and giving
// each the largest of their ends leaves the union of every level unchanged.
__device__ __forceinline__ Elem widen(uint2 x, long long lo, const unsigned long long* maxend) {
  Elem el;
  const unsigned int slot = x.x & 3u;
  el.s = lo + (long long)(x.x >> 2);
  const long long e = x.y == 0xFFFFFFFFu ? (long long)maxend[slot] : lo + (long long)x.y - 1;
  el.e_slot = (long long)((unsigned long long)e | ((unsigned long long)slot << kSlotShift));
  return el;
}

// bucket of a valid record start inside its segment (min_s <= start <= max_s)
__device__ __forceinline__ int bucket_of(long long s, const Geom& g) { return bucket_of_start(g, s); }

__device__ __forceinline__ long long wave_red_min(long long v) {
  for (int d = 32; d >= 1; d >>= 1) { long long o = __shfl_xor(v, d, 64); v = o < v ? o : v; }
  return v;
}
__device__ __forceinline__ unsigned long long wave_red_minu(unsigned long long v) {
  for (int d = 32; d >= 1; d >>= 1) { unsigned long long o = __shfl_xor(v, d, 64); v = o < v ? o : v; }
  return v;
}
__device__ __forceinline__ unsigned long long wave_red_maxu(unsigned long long v) {
  for (int d = 32; d >= 1; d >>= 1) { unsigned long long o = __shfl_xor(v, d, 64); v = o > v ? o : v; }
  return v;
}

struct OpMax {
  __device__ static long long apply(long long a, long long b) { return a > b ? a : b; }
};
struct OpSum {
  __device__ static long long apply(long long a, long long b) { return a + b; }
};

// ----------------------------------------------------------------------------
// wave-level scans with DPP lane shifts (no LDS round trips)
// ----------------------------------------------------------------------------

// DPP controls of the gfx9 family: row_shr:n, row_bcast:15 / :31, wave_shr:1
constexpr int kDppRowShr1 = 0x111, kDppRowShr2 = 0x112, kDppRowShr4 = 0x114, kDppRowShr8 = 0x118;
constexpr int kDppRowBcast15 = 0x142, kDppRowBcast31 = 0x143, kDppWaveShr1 = 0x138;

// v from the lane selected by CTRL, or `old` where that lane is outside the
// row/bank masks or has no source lane
template <int CTRL, int ROW_MASK, int BANK_MASK>
__device__ __forceinline__ long long dpp64(long long old, long long v) {
  const int lo = __builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, ROW_MASK, BANK_MASK, false);
  const int hi = __builtin_amdgcn_update_dpp((int)(old >> 32), (int)(v >> 32), CTRL, ROW_MASK, BANK_MASK, false);
  return (long long)(((unsigned long long)(unsigned int)hi << 32) | (unsigned long long)(unsigned int)lo);
}

// lanes of m below this one
__device__ __forceinline__ unsigned int lanes_below(unsigned long long m) {
  return __builtin_amdgcn_mbcnt_hi((unsigned int)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)m, 0u));
}

__device__ __forceinline__ long long readlane64(long long v, int lane) {
  const int lo = __builtin_amdgcn_readlane((int)v, lane);
  const int hi = __builtin_amdgcn_readlane((int)(v >> 32), lane);
  return (long long)(((unsigned long long)(unsigned int)hi << 32) | (unsigned long long)(unsigned int)lo);
}

// Exclusive scan over the 64 lanes (lane order) with identity `id`, and the total.
template <class Op>
__device__ __forceinline__ long long wave_excl_scan_dpp(long long x, long long id, long long& total) {
  x = Op::apply(x, dpp64<kDppRowShr1, 0xf, 0xf>(id, x));
  x = Op::apply(x, dpp64<kDppRowShr2, 0xf, 0xf>(id, x));
  x = Op::apply(x, dpp64<kDppRowShr4, 0xf, 0xf>(id, x));
  x = Op::apply(x, dpp64<kDppRowShr8, 0xf, 0xf>(id, x));
  x = Op::apply(x, dpp64<kDppRowBcast15, 0xa, 0xf>(id, x));
  x = Op::apply(x, dpp64<kDppRowBcast31, 0xc, 0xf>(id, x));
  total = readlane64(x, 63);
  return dpp64<kDppWaveShr1, 0xf, 0xf>(id, x);
}

struct OpMaxU {
  __device__ static unsigned int apply(unsigned int a, unsigned int b) { return a > b ? a : b; }
};
struct OpSumU {
  __device__ static unsigned int apply(unsigned int a, unsigned int b) { return a + b; }
};

template <int CTRL, int ROW_MASK, int BANK_MASK>
__device__ __forceinline__ unsigned int dpp32(unsigned int old, unsigned int v) {
  return (unsigned int)__builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, ROW_MASK, BANK_MASK, false);
}

// Exclusive scan over the 64 lanes (lane order) with identity `id`, and the total.
template <class Op>
__device__ __forceinline__ unsigned int wave_excl_scan_u32(unsigned int x, unsigned int id, unsigned int& total) {
  x = Op::apply(x, dpp32<kDppRowShr1, 0xf, 0xf>(id, x));
  x = Op::apply(x, dpp32<kDppRowShr2, 0xf, 0xf>(id, x));
  x = Op::apply(x, dpp32<kDppRowShr4, 0xf, 0xf>(id, x));
  x = Op::apply(x, dpp32<kDppRowShr8, 0xf, 0xf>(id, x));
  x = Op::apply(x, dpp32<kDppRowBcast15, 0xa, 0xf>(id, x));
  x = Op::apply(x, dpp32<kDppRowBcast31, 0xc, 0xf>(id, x));
  total = (unsigned int)__builtin_amdgcn_readlane((int)x, 63);
  return dpp32<kDppWaveShr1, 0xf, 0xf>(id, x);
}

struct OpMinI {
  __device__ static int apply(int a, int b) { return a < b ? a : b; }
};
struct OpMaxI {
  __device__ static int apply(int a, int b) { return a > b ? a : b; }
};
struct OpMaxU32 {  // unsigned maximum on int lanes
  __device__ static int apply(int a, int b) { return (unsigned int)a > (unsigned int)b ? a : b; }
};
struct OpOrI {
  __device__ static int apply(int a, int b) { return a | b; }
};

// Reduction over the 64 lanes with DPP row shifts (no LDS round trips); every
// lane receives the result.
template <class Op>
__device__ __forceinline__ int wave_reduce_i32(int x, int id) {
  x = Op::apply(x, __builtin_amdgcn_update_dpp(id, x, kDppRowShr1, 0xf, 0xf, false));
  x = Op::apply(x, __builtin_amdgcn_update_dpp(id, x, kDppRowShr2, 0xf, 0xf, false));
  x = Op::apply(x, __builtin_amdgcn_update_dpp(id, x, kDppRowShr4, 0xf, 0xf, false));
  x = Op::apply(x, __builtin_amdgcn_update_dpp(id, x, kDppRowShr8, 0xf, 0xf, false));
  x = Op::apply(x, __builtin_amdgcn_update_dpp(id, x, kDppRowBcast15, 0xa, 0xf, false));
  x = Op::apply(x, __builtin_amdgcn_update_dpp(id, x, kDppRowBcast31, 0xc, 0xf, false));
  return __builtin_amdgcn_readlane(x, 63);
}

template <class Op>
__device__ __forceinline__ long long wave_reduce_i64(long long x, long long id) {
  long long total;
  (void)wave_excl_scan_dpp<Op>(x, id, total);
  return total;
}

// The code below runs on groups of THREADS threads: a workgroup, or with 64 one
// wave of any workgroup (its waves then work apart from one another).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
template <int THREADS>
__device__ __forceinline__ int group_thread() {
  return THREADS == 64 ? (int)(threadIdx.x & 63) : (int)threadIdx.x;
}
template <int THREADS>
__device__ __forceinline__ int group_wave() {
  return THREADS == 64 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
}
template <int THREADS>
__device__ __forceinline__ void group_sync() {
  if (THREADS == 64) wave_sync();
  else __syncthreads();
}
template <int THREADS>
__device__ __forceinline__ bool group_any(bool x) {
  if (THREADS == 64) {
    wave_sync();
    return __ballot(x) != 0;
  }
  return __syncthreads_or(x);
}

// Group-wide exclusive scan of K int64 lanes per thread (thread order), with totals.
// `lds` holds NW*K int64. Contains barriers: call from uniform control flow.
template <int THREADS, int K, class Op>
__device__ __forceinline__ void block_excl_scan(const long long (&v)[K], long long (&excl)[K],
                                                long long (&total)[K], long long ident, long long* lds) {
  constexpr int NW = THREADS / 64;
  static_assert(NW <= 16, "the waves' totals are scanned within a row of 16 lanes");
  const int lane = threadIdx.x & 63, wave = group_wave<THREADS>();
  long long ex[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    long long tot;
    ex[k] = wave_excl_scan_dpp<Op>(v[k], ident, tot);
    if constexpr (NW == 1) {
      excl[k] = ex[k];
      total[k] = tot;
    } else if (lane == 0) {
      lds[wave * K + k] = tot;
    }
  }
  if constexpr (NW == 1) return;
  group_sync<THREADS>();
#pragma unroll
  for (int k = 0; k < K; ++k) {
    // lane w holds wave w's total: scanned across lanes, as reading all of them
    // in every thread takes 2 NW K registers (and spills)
    long long t = lane < NW ? lds[lane * K + k] : ident;
    if (NW > 1) t = Op::apply(t, dpp64<kDppRowShr1, 0xf, 0xf>(ident, t));
    if (NW > 2) t = Op::apply(t, dpp64<kDppRowShr2, 0xf, 0xf>(ident, t));
    if (NW > 4) t = Op::apply(t, dpp64<kDppRowShr4, 0xf, 0xf>(ident, t));
    if (NW > 8) t = Op::apply(t, dpp64<kDppRowShr8, 0xf, 0xf>(ident, t));
    const long long pre = wave > 0 ? readlane64(t, wave - 1) : ident;
    excl[k] = Op::apply(pre, ex[k]);
    total[k] = readlane64(t, NW - 1);
  }
  group_sync<THREADS>();
}

// One stable LSD pass on 8 bits of (start - lo) >> sh over the positions
// in[0..n): out[] receives the element indices in the new order, dstart[d] the
// first output position of digit d. Waves own contiguous position ranges;
// lanes with equal digits are matched with ballots, so the pass is stable.
template <int THREADS, int MAXR>
__device__ __forceinline__ void radix_pass(const Elem* E, const unsigned short* in, unsigned short* out, int n,
                                           long long lo, int sh, unsigned int* whist, unsigned int* dstart,
                                           long long* lds_scan) {
  constexpr int NW = THREADS / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int span = (((n + NW - 1) / NW) + 63) & ~63;
  const unsigned long long lt = (1ull << lane) - 1ull;
  for (int i = threadIdx.x; i < NW * 256; i += THREADS) whist[i] = 0;
  __syncthreads();
  unsigned int loc[MAXR];
  unsigned char dig[MAXR];
  unsigned short idx[MAXR];
#pragma unroll
  for (int r = 0; r < MAXR; ++r) {
    loc[r] = 0;
    dig[r] = 0;
    idx[r] = 0;
    if (r * 64 < span) {  // wave-uniform
      const int pos = wave * span + r * 64 + lane;
      const bool act = pos < n;
      const unsigned short i = act ? (in ? in[pos] : (unsigned short)pos) : (unsigned short)0;
      const unsigned int d = act ? (unsigned int)(((unsigned long long)(E[i].s - lo) >> sh) & 255ull) : 0u;
      unsigned long long peers = __ballot(act);
#pragma unroll
      for (int bit = 0; bit < 8; ++bit) {
        const bool b = (d >> bit) & 1u;
        const unsigned long long m = __ballot(b);
        peers &= b ? m : ~m;
      }
      if (act) {
        unsigned int* h = &whist[wave * 256 + d];
        const unsigned int before = *h;
        loc[r] = before + (unsigned int)__popcll(peers & lt);
        dig[r] = (unsigned char)d;
        idx[r] = i;
        if ((peers & lt) == 0) *h = before + (unsigned int)__popcll(peers);
      }
    }
  }
  __syncthreads();
  // digit-major exclusive prefix over (digit, wave)
  {
    long long tot = 0;
    unsigned int h[NW];
    if (threadIdx.x < 256) {
#pragma unroll
      for (int w = 0; w < NW; ++w) { h[w] = whist[w * 256 + threadIdx.x]; tot += h[w]; }
    }
    long long v[1] = {threadIdx.x < 256 ? tot : 0}, ex[1], all[1];
    block_excl_scan<THREADS, 1, OpSum>(v, ex, all, 0, lds_scan);
    if (threadIdx.x < 256) {
      unsigned int run = (unsigned int)ex[0];
      dstart[threadIdx.x] = run;
#pragma unroll
      for (int w = 0; w < NW; ++w) { whist[w * 256 + threadIdx.x] = run; run += h[w]; }
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < MAXR; ++r) {
    if (r * 64 < span) {
      const int pos = wave * span + r * 64 + lane;
      if (pos < n) out[whist[wave * 256 + dig[r]] + loc[r]] = idx[r];
    }
  }
  __syncthreads();
}

struct FlatState {
  long long M[3];  // running max end (with the carry)
  long long P[3];  // measure accumulated in this bucket
  long long R[3];  // components written in this bucket
};

// Flatten the NLEV levels of one sorted tile of n <= THREADS * MAXI records:
// positions 0..n-1 in order ord (or identity). Writes components of each level
// at comp[l][R], or in the narrow form relative to `nlo` at compn[l][R] when
// compn is given; advances `st`. A thread's records are read once, into
// registers, and the levels' break counts (at most 2^12 each) share one scan:
// a wave's 64-bit scans are most of its instructions.
template <int THREADS, int MAXI, int NLEV>
__device__ __forceinline__ void flatten_tile(const Elem* E, const unsigned short* ord, int n, Comp* const* comp,
                                             CompN* const* compn, long long nlo, FlatState& st, long long* lds_scan) {
  static_assert(THREADS * MAXI <= 1 << 12 && NLEV <= 3, "break counts take 20 bits per level");
  const int ipt = (n + THREADS - 1) / THREADS;
  const int p0 = group_thread<THREADS>() * ipt;
  constexpr long long EMASK = (1ll << kSlotShift) - 1;
  // past the tile: a record of no level
  long long s[MAXI], e[MAXI];
  int slot[MAXI];
#pragma unroll
  for (int j = 0; j < MAXI; ++j) {
    const int q = p0 + j;
    const bool in = j < ipt && q < n;
    const Elem el = E[in ? (ord ? (int)ord[q] : q) : 0];
    s[j] = el.s;
    e[j] = el.e_slot & EMASK;
    slot[j] = in ? (int)((unsigned long long)el.e_slot >> kSlotShift) : 3;
  }
  // phase A: exclusive max-scan of ends per level
  long long tmax[NLEV];
#pragma unroll
  for (int l = 0; l < NLEV; ++l) {
    tmax[l] = LLONG_MIN;
#pragma unroll
    for (int j = 0; j < MAXI; ++j)
      if (slot[j] <= l && e[j] > tmax[l]) tmax[l] = e[j];
  }
  long long M[NLEV], totm[NLEV];
  block_excl_scan<THREADS, NLEV, OpMax>(tmax, M, totm, LLONG_MIN, lds_scan);
  // phase B: per-thread measure per level, and break counts in fields of 20 bits
  long long acc[NLEV + 1];
  acc[NLEV] = 0;
#pragma unroll
  for (int l = 0; l < NLEV; ++l) {
    M[l] = M[l] > st.M[l] ? M[l] : st.M[l];
    long long Mb = M[l], a = 0;
    int breaks = 0;
#pragma unroll
    for (int j = 0; j < MAXI; ++j) {
      if (slot[j] <= l) {
        const long long lo = s[j] > Mb ? s[j] : Mb;
        if (e[j] > lo) a += e[j] - lo;
        if (s[j] > Mb) ++breaks;
        if (e[j] > Mb) Mb = e[j];
      }
    }
    acc[l] = a;
    acc[NLEV] |= (long long)breaks << (20 * l);
  }
  long long exa[NLEV + 1], tota[NLEV + 1];
  block_excl_scan<THREADS, NLEV + 1, OpSum>(acc, exa, tota, 0, lds_scan);
  // phase C: write components
#pragma unroll
  for (int l = 0; l < NLEV; ++l) {
    long long P = st.P[l] + exa[l], R = st.R[l] + ((exa[NLEV] >> (20 * l)) & 0xFFFFF), Ml = M[l];
#pragma unroll
    for (int j = 0; j < MAXI; ++j) {
      if (slot[j] <= l) {
        if (s[j] > Ml) {
          if (compn) {
            CompN c;
            c.cs = (uint32_t)(s[j] - nlo);
            c.pl = (uint32_t)P;
            compn[l][R] = c;
          } else {
            Comp c;
            c.cs = s[j];
            c.pl = P;
            comp[l][R] = c;
          }
          R += 1;
        }
        const long long lo = s[j] > Ml ? s[j] : Ml;
        if (e[j] > lo) P += e[j] - lo;
        if (e[j] > Ml) Ml = e[j];
      }
    }
    st.M[l] = totm[l] > st.M[l] ? totm[l] : st.M[l];
    st.P[l] += tota[l];
    st.R[l] += (tota[NLEV] >> (20 * l)) & 0xFFFFF;
  }
}

__device__ __forceinline__ double ratio(long long num, long long den, int bit, unsigned int& mask) {
  if (den == 0) {
    mask |= 1u << bit;
    return 1.0;
  }
  return (double)num / (double)den;
}


// Block-wide OR and AND of per-thread key accumulators: the bits in which keys differ.
template <int THREADS>
__device__ __forceinline__ unsigned long long block_vary(unsigned long long kor, unsigned long long kand,
                                                         unsigned long long (*red)[THREADS / 64]) {
  constexpr int NW = THREADS / 64;
  for (int d = 32; d >= 1; d >>= 1) {
    kor |= __shfl_xor(kor, d, 64);
    kand &= __shfl_xor(kand, d, 64);
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) {
    red[0][wave] = kor;
    red[1][wave] = kand;
  }
  __syncthreads();
  kor = 0;
  kand = ~0ull;
  for (int w = 0; w < NW; ++w) {
    kor |= red[0][w];
    kand &= red[1][w];
  }
  __syncthreads();
  return kor ^ kand;
}

// Group-wide minimum and maximum of per-thread keys.
template <int THREADS>
__device__ __forceinline__ void block_range(unsigned long long& mn, unsigned long long& mx,
                                            unsigned long long (*red)[THREADS / 64]) {
  constexpr int NW = THREADS / 64;
  mn = wave_red_minu(mn);
  mx = wave_red_maxu(mx);
  const int lane = threadIdx.x & 63, wave = group_wave<THREADS>();
  if (lane == 0) {
    red[0][wave] = mn;
    red[1][wave] = mx;
  }
  group_sync<THREADS>();
  for (int w = 0; w < NW; ++w) {
    mn = red[0][w] < mn ? red[0][w] : mn;
    mx = red[1][w] > mx ? red[1][w] : mx;
  }
}

// The place of a key inside its sub-bin of 2^sh keys, as a fraction of 2^32.
__device__ __forceinline__ unsigned int bin_fraction(unsigned long long key, int sh) {
  const unsigned long long low = key & ((1ull << sh) - 1ull);
  return sh >= 32 ? (unsigned int)(low >> (sh - 32)) : (unsigned int)(low << (32 - sh));
}

// Order of sm.E[0..n) (n <= CAP, already in LDS and visible to the group) by
// start - lo, in ord: nullptr where E is already in an acceptable order (all
// starts equal). False, with nothing in ord: a sub-bin is crowded.
//
// A counting sort over about one sub-bin per record, between the smallest and
// the largest start, then an insertion sort in each sub-bin of two or more.
// Where starts lie in a few places (a sub-bin of more than kBinRefine
// records) a second count first splits every sub-bin into as many parts as it
// holds records. A sub-bin that is crowded even then (many equal starts) is
// left to the radix sort of sort_lds, which alone took five passes of eight
// barriers for a wide bucket.
constexpr unsigned int kBinRefine = 8, kBinCrowd = 32;

template <int THREADS, int CAP>
__device__ __forceinline__ bool sort_bins(SortSmem<THREADS, CAP>& sm, int n, long long lo, const unsigned short*& ord) {
  constexpr int MAXR = CAP / THREADS;
  const int tid = group_thread<THREADS>();
  ord = nullptr;
  unsigned long long mn = ~0ull, mx = 0;
  for (int i = tid; i < n; i += THREADS) {
    const unsigned long long k = (unsigned long long)(sm.E[i].s - lo);
    mn = k < mn ? k : mn;
    mx = k > mx ? k : mx;
  }
  block_range<THREADS>(mn, mx, sm.red);
  if (mn == mx) return true;
  // 2 THREADS sub-bins at least (a thread scans one word or more), CAP at most
  int bits = bitlen64(2 * THREADS - 1);
  while ((1 << bits) < n) ++bits;
  const int words = 1 << (bits - 1);  // two 16-bit counters (then sub-bin starts) per word
  const int hb = bitlen64(mx - mn), sh = hb > bits ? hb - bits : 0;
  unsigned int* bins = (unsigned int*)sm.ordB;
  auto start_of = [&](unsigned int d) { return (bins[d >> 1] >> (16u * (d & 1u))) & 0xFFFFu; };
  auto stop_of = [&](unsigned int d) { return (d + 1) >> 1 < (unsigned int)words ? start_of(d + 1) : (unsigned int)n; };
  unsigned int bin[MAXR], rk[MAXR];
#pragma unroll
  for (int r = 0; r < MAXR; ++r) {
    const int i = tid + r * THREADS;
    bin[r] = i < n ? (unsigned int)(((unsigned long long)(sm.E[i].s - lo) - mn) >> sh) : 0u;
    rk[r] = 0;
  }
  // ranks within the sub-bins bin[], and the sub-bins' starts; true if one holds more than `most`
  auto count = [&](unsigned int most) -> bool {
    for (int w = tid; w < words; w += THREADS) bins[w] = 0;
    group_sync<THREADS>();
    bool over = false;
#pragma unroll
    for (int r = 0; r < MAXR; ++r) {
      if (tid + r * THREADS < n) {
        const unsigned int half = 16u * (bin[r] & 1u);
        rk[r] = (atomicAdd(&bins[bin[r] >> 1], 1u << half) >> half) & 0xFFFFu;
        over |= rk[r] >= most;
      }
    }
    group_sync<THREADS>();
    const int per = words / THREADS, w0 = tid * per;
    long long v[1] = {0}, ex[1], all[1];
    for (int j = 0; j < per; ++j) v[0] += (bins[w0 + j] & 0xFFFFu) + (bins[w0 + j] >> 16);
    block_excl_scan<THREADS, 1, OpSum>(v, ex, all, 0, sm.lds_scan);
    unsigned int run = (unsigned int)ex[0];
    for (int j = 0; j < per; ++j) {
      const unsigned int c = bins[w0 + j], mid = run + (c & 0xFFFFu);
      bins[w0 + j] = run | (mid << 16);
      run = mid + (c >> 16);
    }
    return group_any<THREADS>(over);
  };
  if (count(kBinRefine) && sh > 0) {
#pragma unroll
    for (int r = 0; r < MAXR; ++r) {
      const int i = tid + r * THREADS;
      if (i < n) {
        const unsigned int st = start_of(bin[r]), c = stop_of(bin[r]) - st;
        bin[r] = st + __umulhi(bin_fraction((unsigned long long)(sm.E[i].s - lo) - mn, sh), c);
      }
    }
    group_sync<THREADS>();
    (void)count(kBinRefine);
  }
#pragma unroll
  for (int r = 0; r < MAXR; ++r) {
    const int i = tid + r * THREADS;
    if (i < n) sm.ordA[start_of(bin[r]) + rk[r]] = (unsigned short)i;
  }
  group_sync<THREADS>();
  bool crowded = false;
  if (sh > 0) {
    // the thread that placed a sub-bin's second record puts it in order; a
    // larger one needs no order where its starts are all equal
#pragma unroll
    for (int r = 0; r < MAXR; ++r) {
      const int i = tid + r * THREADS;
      if (i < n && rk[r] >= 1) {
        const unsigned int st = start_of(bin[r]), c = stop_of(bin[r]) - st;
        if (c > kBinCrowd) {
          crowded |= sm.E[i].s != sm.E[sm.ordA[st]].s;
          continue;
        }
        if (rk[r] > 1) continue;
        unsigned short* o = sm.ordA + st;
        for (int a = 1; a < (int)c; ++a) {
          const unsigned short x = o[a];
          const long long s = sm.E[x].s;
          int b = a - 1;
          while (b >= 0 && sm.E[o[b]].s > s) {
            o[b + 1] = o[b];
            --b;
          }
          o[b + 1] = x;
        }
      }
    }
  }
  if (group_any<THREADS>(crowded)) return false;
  ord = sm.ordA;
  return true;
}

// The same order for every case. Where a sub-bin is crowded: an LSD radix sort
// of 8 of the varying bits per pass, or by one wave a bitonic sort.
template <int THREADS, int CAP>
__device__ __forceinline__ const unsigned short* sort_lds(SortSmem<THREADS, CAP>& sm, int n, long long lo) {
  const unsigned short* ord;
  if (sort_bins<THREADS, CAP>(sm, n, lo, ord)) return ord;
  if constexpr (THREADS < 256) {
    // places past the records hold the largest key: none of them moves before one
    const int tid = group_thread<THREADS>();
    int size = 2;
    while (size < n) size <<= 1;
    for (int i = tid; i < size; i += THREADS) sm.ordA[i] = (unsigned short)i;
    group_sync<THREADS>();
    auto key = [&](int i) { return i < n ? sm.E[i].s : LLONG_MAX; };
    for (int k = 2; k <= size; k <<= 1) {
      for (int j = k >> 1; j > 0; j >>= 1) {
        for (int i = tid; i < size / 2; i += THREADS) {
          const int a = ((i & ~(j - 1)) << 1) | (i & (j - 1)), b = a | j;
          const unsigned short x = sm.ordA[a], y = sm.ordA[b];
          if ((key(x) > key(y)) == ((a & k) == 0)) {
            sm.ordA[a] = y;
            sm.ordA[b] = x;
          }
        }
        group_sync<THREADS>();
      }
    }
    return sm.ordA;
  } else {
    constexpr int MAXR = CAP / THREADS;
    unsigned long long kor = 0, kand = ~0ull;
    for (int i = threadIdx.x; i < n; i += THREADS) {
      const unsigned long long k = (unsigned long long)(sm.E[i].s - lo);
      kor |= k;
      kand &= k;
    }
    const unsigned long long vary = block_vary<THREADS>(kor, kand, sm.red);
    const int lb = __ffsll((long long)vary) - 1;
    const int passes = (bitlen64(vary) - lb + 7) >> 3;
    const unsigned short* in = nullptr;  // identity for the first pass
    for (int ps = 0; ps < passes; ++ps) {
      unsigned short* out = (ps & 1) ? sm.ordB : sm.ordA;
      radix_pass<THREADS, MAXR>(sm.E, in, out, n, lo, lb + 8 * ps, sm.whist, sm.dstart, sm.lds_scan);
      in = out;
    }
    return in;
  }
}

// Stable LSD sort of n records in global memory by start - lo, CAP records of
// LDS at a time; dst is scratch of the same size. Returns the buffer that
// holds the sorted records (src or dst).
template <int THREADS, int CAP>
__device__ Elem* sort_global(SortSmem<THREADS, CAP>& sm, Elem* src, Elem* dst, long long n, long long lo) {
  constexpr int MAXR = CAP / THREADS;
  unsigned long long kor = 0, kand = ~0ull;
  for (long long i = threadIdx.x; i < n; i += THREADS) {
    const unsigned long long k = (unsigned long long)(src[i].s - lo);
    kor |= k;
    kand &= k;
  }
  const unsigned long long vary = block_vary<THREADS>(kor, kand, sm.red);
  if (!vary) return src;
  const int lb = __ffsll((long long)vary) - 1;
  const int hb = bitlen64(vary);
  const int passes = (hb - lb + 7) >> 3;
  for (int ps = 0; ps < passes; ++ps) {
    const int sh = lb + 8 * ps;
    // digit histogram of all records -> running output base per digit
    for (int i = threadIdx.x; i < 256; i += THREADS) sm.dcount[i] = 0;
    __syncthreads();
    for (long long i = threadIdx.x; i < n; i += THREADS)
      atomicAdd(&sm.dcount[((unsigned long long)(src[i].s - lo) >> sh) & 255ull], 1u);
    __syncthreads();
    {
      long long v[1] = {threadIdx.x < 256 ? (long long)sm.dcount[threadIdx.x] : 0}, ex[1], all[1];
      block_excl_scan<THREADS, 1, OpSum>(v, ex, all, 0, sm.lds_scan);
      if (threadIdx.x < 256) sm.dcount[threadIdx.x] = (unsigned int)ex[0];
    }
    __syncthreads();
    for (long long t0 = 0; t0 < n; t0 += CAP) {
      const int cnt = (int)min((long long)CAP, n - t0);
      for (int i = threadIdx.x; i < cnt; i += THREADS) sm.E[i] = src[t0 + i];
      __syncthreads();
      radix_pass<THREADS, MAXR>(sm.E, nullptr, sm.ordA, cnt, lo, sh, sm.whist, sm.dstart, sm.lds_scan);
      for (int q = threadIdx.x; q < cnt; q += THREADS) {
        const unsigned short i = sm.ordA[q];
        const unsigned int d = (unsigned int)(((unsigned long long)(sm.E[i].s - lo) >> sh) & 255ull);
        dst[sm.dcount[d] + (q - sm.dstart[d])] = sm.E[i];
      }
      __syncthreads();
      if (threadIdx.x < 256) {
        const unsigned int d = threadIdx.x;
        const unsigned int next = d < 255 ? sm.dstart[d + 1] : (unsigned int)cnt;
        sm.dcount[d] += next - sm.dstart[d];
      }
      __syncthreads();
    }
    Elem* t = src;
    src = dst;
    dst = t;
  }
  return src;
}

// Ratios of one region's metric trees from exact integer aggregates.
// v: sumU, sumW, sumMPI, sumOther, sumK, sumM, maxUW, maxK, maxKM
__device__ __forceinline__ Tree make_tree(long long E, int n_hosts, int n_devices, const long long (&v)[9]) {
  Tree t;
  t.E = E;
  t.n = n_hosts;
  t.m = n_devices;
  const long long U = v[0], W = v[1], UW = v[0] + v[1];
  t.sum[0] = U;
  t.sum[1] = W;
  t.sum[2] = v[2];
  t.sum[3] = v[3];
  t.sum[4] = UW;
  t.sum[5] = v[6];
  t.sum[6] = v[4];
  t.sum[7] = v[5];
  t.sum[8] = v[7];
  t.sum[9] = v[8];
  unsigned int mask = 0;
  const long long n = n_hosts, m = n_devices;
  t.ratio[0] = ratio(U, n * E, 0, mask);        // eq. 6
  t.ratio[1] = ratio(UW, n * E, 1, mask);       // eq. 7
  t.ratio[2] = ratio(UW, n * v[6], 2, mask);    // eq. 4, U+W useful
  t.ratio[3] = ratio(v[6], E, 3, mask);         // eq. 5, U+W useful
  t.ratio[4] = ratio(U, UW, 4, mask);           // eq. 8
  t.ratio[5] = ratio(v[4], m * E, 5, mask);     // eq. 9
  t.ratio[6] = ratio(v[4], m * v[7], 6, mask);  // eq. 10
  t.ratio[7] = ratio(v[7], v[8], 7, mask);      // eq. 11
  t.ratio[8] = ratio(v[8], E, 8, mask);         // eq. 12
  t.undefined_mask = mask;
  t.reserved = 0;
  return t;
}

// State times of resource r of region rd from its levels' measures D inside
// it, written to `times` and added to v (sums U, W, MPI, Other, K, M; maxima
// U+W, K, K+M).
__device__ __forceinline__ void add_times(bool host, const long long (&D)[3], long long E, long long* out,
                                          long long (&v)[9]) {
  if (host) {
    const long long u = D[0], w = D[1] - D[0], mpi = D[2] - D[1], o = E - D[2];
    out[0] = u; out[1] = w; out[2] = mpi; out[3] = o;
    v[0] += u; v[1] += w; v[2] += mpi; v[3] += o;
    v[6] = u + w > v[6] ? u + w : v[6];
  } else {
    const long long k = D[0], mm = D[1] - D[0], idle = E - D[1];
    out[0] = k; out[1] = mm; out[2] = idle; out[3] = 0;
    v[4] += k; v[5] += mm;
    v[7] = k > v[7] ? k : v[7];
    v[8] = k + mm > v[8] ? k + mm : v[8];
  }
}

// Eight neighbouring lanes hold one resource's measures (lane 2 l + end, level
// l): the first of them gets the levels' measures inside the region.
__device__ __forceinline__ void group_levels(long long M, long long (&D)[3]) {
#pragma unroll
  for (int l = 0; l < 3; ++l) D[l] = __shfl(M, 2 * l + 1, 8) - __shfl(M, 2 * l, 8);
}

// The finished trees of a workgroup's n consecutive regions go out as whole
// words, neighbouring lanes to neighbouring words: the results lie in host
// memory, where every store is a bus transfer.
__device__ __forceinline__ void put_trees(const Tree* lds, int n, Tree* out) {
  constexpr int kWords = sizeof(Tree) / 8;
  const unsigned long long* src = (const unsigned long long*)lds;
  for (int i = threadIdx.x; i < n * kWords; i += blockDim.x) ((unsigned long long*)out)[i] = src[i];
}

// Block reduction of per-thread resource state times (thread 0 receives it).
// Per thread: host rows add U, W, MPI, Other; device rows K, M. `lds` holds 10
// int64 per wave; ends with a barrier.
__device__ __forceinline__ void block_tree(long long (&v)[9], long long* lds) {
#pragma unroll
  for (int i = 0; i < 6; ++i) v[i] = wave_reduce_i64<OpSum>(v[i], 0);
#pragma unroll
  for (int i = 6; i < 9; ++i) v[i] = wave_reduce_i64<OpMax>(v[i], 0);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = (int)blockDim.x >> 6;
  if (lane == 0)
    for (int i = 0; i < 9; ++i) lds[wave * 10 + i] = v[i];
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < nw; ++w) {
      for (int i = 0; i < 6; ++i) v[i] += lds[w * 10 + i];
      for (int i = 6; i < 9; ++i) v[i] = lds[w * 10 + i] > v[i] ? lds[w * 10 + i] : v[i];
    }
  }
  __syncthreads();
}

}  // namespace hpop
