// HIP kernels of the trace reduction, written for CDNA4 (gfx950, wave64).
//
// All passes are memory-bound integer work: no MFMA (there is no dense
// contraction), loads and stores are coalesced, the fine-grained sort runs in
// LDS (160 KB per workgroup on gfx950), and cross-workgroup communication is
// limited to atomics on per-bucket counters plus one decoupled look-back scan
// over bucket counts.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>

#include "hpop_device.h"
#include "hpop_internal.h"
#include "hpop_kernels.h"

namespace hpop {

// ----------------------------------------------------------------------------
// gather: the chunks of one add call into the record arena
// ----------------------------------------------------------------------------

// Up to kGatherChunks chunks of a launch, in the kernel's arguments (no table
// to upload): chunk i covers workgroups [first[i], first[i + 1]), each of
// kGatherPiece records of both arrays. A few hundred copies of some ten
// thousand bytes are bound by what enqueueing each costs the host (about 4 us
// per copy, two copies per chunk); one launch per 80 chunks took the add and
// build of 264 chunks (9e5 records) from 1049 to 232 us. Pieces of 1024 records:
// 80 chunks of 8191 take 6.0 us, 7.9 with pieces of 2048 and 11.4 with 4096,
// which left most CUs without a workgroup.
constexpr int kGatherChunks = 80;
constexpr int kGatherPiece = 1024;
struct GatherArgs {
  CopyChunk c[kGatherChunks];
  unsigned int first[kGatherChunks + 1];
  int n;
};
static_assert(sizeof(GatherArgs) <= 4000, "kernel arguments");

// n words from src to dst (256 B aligned) by the workgroup: pairs of words
// when src is 16 B aligned, with all of a thread's loads in flight.
__device__ __forceinline__ void copy_words(const int64_t* src, int64_t* dst, int n) {
  if ((((uintptr_t)src) & 15) == 0 && n == kGatherPiece) {
    const longlong2* a = (const longlong2*)src;
    longlong2* b = (longlong2*)dst;
    static_assert(kGatherPiece == 4 * 256, "two pairs per thread");
    const longlong2 x0 = a[threadIdx.x], x1 = a[threadIdx.x + 256];
    b[threadIdx.x] = x0;
    b[threadIdx.x + 256] = x1;
  } else {
    for (int i = threadIdx.x; i < n; i += 256) dst[i] = src[i];
  }
}

__global__ __launch_bounds__(256) void k_gather(GatherArgs g) {
  int lo = 0, hi = g.n - 1;  // the last chunk whose first workgroup is at or before this one
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (g.first[mid] <= blockIdx.x) lo = mid; else hi = mid - 1;
  }
  const CopyChunk c = g.c[lo];
  const long long at = (long long)(blockIdx.x - g.first[lo]) * kGatherPiece;
  const int n = (int)min((long long)kGatherPiece, c.count - at);
  copy_words(c.s + at, c.dst_s + at, n);
  copy_words(c.e + at, c.dst_e + at, n);
}

// ----------------------------------------------------------------------------
// reset: per-build counters to their identities
// ----------------------------------------------------------------------------

__device__ __forceinline__ void reset_counters(const Plan& p) {
  const long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long i = tid; i < p.n_buckets; i += stride) {
    p.counts[i] = 0;
    p.cursor[i] = 0;
  }
  for (long long i = tid; i < 3 * p.n_buckets; i += stride) p.maxend[i] = 0;
  const long long nscan = (p.n_buckets + kScanTile - 1) / kScanTile + 1;
  for (long long i = tid; i < nscan; i += stride) p.scan_state[i] = 0;
  if (tid == 0) {
    p.err[0] = ULLONG_MAX;
    p.oversized[0] = 0;
    p.oversized[1] = 0;
  }
  if (tid < 4) p.ticket[tid] = 0;
  for (long long i = tid; i < 2 * kQueues * kQueuePad; i += stride) p.qlen[i] = 0;
  if (tid == 0 && p.ts) p.ts[kTsBuild] = __builtin_amdgcn_s_memrealtime();
  for (long long i = tid; i < p.n_owners; i += stride) p.owner_err[i] = 0;
  for (long long i = tid; i < kRaccWords * p.n_racc; i += stride) p.racc[i] = 0;
}

__global__ void k_reset(Plan p) {
  reset_counters(p);
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < p.n_segs; i += stride) {
    p.stats[i].min_s = ULLONG_MAX;
    p.stats[i].max_s = 0;
    p.stats[i].max_e = 0;
    p.stats[i].far_e = 0;
  }
}

// ----------------------------------------------------------------------------
// shared tiles: chunks of fewer than half a tile of records, several per tile.
// The same passes as for a tile of one chunk, with the chunk (and so the
// segment, kind and bucket geometry) looked up per record and buckets indexed
// globally. They run in the same launches as the other tiles (the blocks past
// n_own_tiles), reusing those kernels' LDS arrays where the layouts agree.
// ----------------------------------------------------------------------------

// One 8 B word stored past the caches: a record in the bucketed form (the
// regrouped records, 1 GB for 1.25e8, are read back only by the merge, after
// the scatter has finished), or a merged interval of the wave merge.
__device__ __forceinline__ void put_rec8(uint2* dst, unsigned int key, unsigned int end) {
  __builtin_nontemporal_store((unsigned long long)key | ((unsigned long long)end << 32), (unsigned long long*)dst);
}

// Two 8 B words loaded past the caches: the start-range pass reads every
// start once, and the scatter after it reads them again from HBM anyway.
__device__ __forceinline__ ulonglong2 get_pair_nt(const ulonglong2* src) {
  typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
  const u64x2 t = __builtin_nontemporal_load((const u64x2*)src);
  return make_ulonglong2(t.x, t.y);
}

// The chunks of one shared tile, staged in LDS.
struct ShTile {
  const int64_t* s[kTileChunks];
  const int64_t* e[kTileChunks];
  long long bucket_begin[kTileChunks];
  Geom g[kTileChunks];
  int off[kTileChunks + 1];  // off[j]: the tile's index of chunk j's first record; off[n]: records in the tile
  int seg[kTileChunks];
  int slot[kTileChunks];
  int n;                     // chunks in the tile
  int first;                 // index of the first one in the chunk table
};

// Stages the chunks of shared tile `tile` (every thread calls; ends with a
// barrier). They are the chunks up to the tile's last one whose first tile is
// `tile`: thread j takes the j-th from the end and files it at its place. The
// geometry exists only after the start-range pass.
template <bool kGeom>
__device__ __forceinline__ void sh_load(const Plan& p, long long tile, ShTile& T) {
  const int last = p.tile_chunk[tile];
  for (int j = threadIdx.x; j < kTileChunks && j <= last; j += blockDim.x) {
    const ChunkDesc cd = p.chunks[last - j];
    if (cd.tile_begin != tile) continue;
    const int q = cd.tile_pos;
    T.s[q] = cd.s;
    T.e[q] = cd.e;
    T.off[q] = cd.tile_off;
    T.seg[q] = cd.seg;
    T.slot[q] = cd.slot;
    if (kGeom) {
      T.bucket_begin[q] = p.segs[cd.seg].bucket_begin;
      T.g[q] = p.geom[cd.seg];
    }
    if (j == 0) {
      T.off[q + 1] = cd.tile_off + (int)cd.count;
      T.n = q + 1;
      T.first = last - q;
    }
  }
  __syncthreads();
}

// The chunk of tile record x < off[n]: the largest j < n with off[j] <= x.
__device__ __forceinline__ int sh_find(const ShTile& T, int x) {
  int j = 0;
#pragma unroll
  for (int step = kTileChunks / 2; step > 0; step >>= 1) {
    const int m = j + step;
    if (m < T.n && T.off[m] <= x) j = m;
  }
  return j;
}

struct ShStatsSmem {
  ShTile T;
  unsigned long long mn[kTileChunks], mx[kTileChunks];  // start range per chunk of the tile
};

// Start range of the records of shared tile `tile`, per chunk, into the segment statistics.
template <int THREADS>
__device__ __forceinline__ void stats_shared(const Plan& p, long long tile, ShStatsSmem& S) {
  for (int j = threadIdx.x; j < kTileChunks; j += THREADS) {
    S.mn[j] = ULLONG_MAX;
    S.mx[j] = 0;
  }
  sh_load<false>(p, tile, S.T);
  const int n = S.T.off[S.T.n];
  for (int x = threadIdx.x; x < n; x += THREADS) {
    const int j = sh_find(S.T, x);
    const unsigned long long v = (unsigned long long)S.T.s[j][x - S.T.off[j]];
    if (v < (unsigned long long)kTimeLimit) {  // invalid starts stay out of the range
      atomicMin(&S.mn[j], v);
      atomicMax(&S.mx[j], v);
    }
  }
  __syncthreads();
  for (int j = threadIdx.x; j < S.T.n; j += THREADS) {
    if (S.mn[j] != ULLONG_MAX) {
      atomicMin(&p.stats[S.T.seg[j]].min_s, S.mn[j]);
      atomicMax(&p.stats[S.T.seg[j]].max_s, S.mx[j]);
    }
  }
}

// Per record of a shared tile: its chunk, and its start and end, loaded for
// all rounds first from positions clamped into the tile (n >= 1).
template <int THREADS, int IPT>
__device__ __forceinline__ void sh_records(const ShTile& T, int n, int (&jj)[IPT], long long (&svs)[IPT],
                                           long long (&evs)[IPT]) {
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const int x = threadIdx.x + k * THREADS;
    const int xc = x < n ? x : n - 1;
    jj[k] = sh_find(T, xc);
  }
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const int x = threadIdx.x + k * THREADS;
    const int i = (x < n ? x : n - 1) - T.off[jj[k]];
    svs[k] = T.s[jj[k]][i];
    evs[k] = T.e[jj[k]][i];
  }
}

// Bucket counts of shared tile `tile` (s_rng and hist: the count kernel's LDS arrays).
template <int THREADS, int IPT>
__device__ __forceinline__ void hist_shared(const Plan& p, long long tile, ShTile& T, int (*s_rng)[THREADS / 64],
                                            unsigned int* hist) {
  constexpr int NW = THREADS / 64;
  constexpr int HW = THREADS * IPT <= kHistWin ? THREADS * IPT / 4 : kHistWin;
  for (int i = threadIdx.x; i < HW; i += THREADS) hist[i] = 0;
  sh_load<true>(p, tile, T);
  const int n = T.off[T.n];
  int jj[IPT], gbk[IPT];
  long long svs[IPT], evs[IPT];
  sh_records<THREADS, IPT>(T, n, jj, svs, evs);
  int bmin = INT_MAX, bmax = -1;
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    gbk[k] = -1;
    if ((int)threadIdx.x + k * THREADS < n && rec_valid(svs[k], evs[k]) && svs[k] < evs[k]) {
      const int j = jj[k];
      gbk[k] = (int)(T.bucket_begin[j] + bucket_of(svs[k], T.g[j]));
      bmin = min(bmin, gbk[k]);
      bmax = max(bmax, gbk[k]);
    }
  }
  bmin = wave_reduce_i32<OpMinI>(bmin, INT_MAX);
  bmax = wave_reduce_i32<OpMaxI>(bmax, -1);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) { s_rng[0][wave] = bmin; s_rng[1][wave] = bmax; }
  __syncthreads();
  bmin = INT_MAX; bmax = -1;
  for (int w = 0; w < NW; ++w) { bmin = min(bmin, s_rng[0][w]); bmax = max(bmax, s_rng[1][w]); }
  if (bmax < 0) return;  // uniform: no valid record in this tile
  if (bmax - bmin < HW) {
#pragma unroll
    for (int k = 0; k < IPT; ++k) {
      unsigned long long todo = __ballot(gbk[k] >= 0);
      while (todo) {
        const int leader = __ffsll((long long)todo) - 1;
        const int lb = __builtin_amdgcn_readlane(gbk[k], leader);
        const unsigned long long m = __ballot(gbk[k] == lb);
        if (lane == leader) atomicAdd(&hist[lb - bmin], (unsigned int)__popcll(m));
        todo &= ~m;
      }
    }
    __syncthreads();
    for (int i = threadIdx.x; i <= bmax - bmin; i += THREADS)
      if (hist[i]) atomicAdd(&p.counts[bmin + i], hist[i]);
  } else {
#pragma unroll
    for (int k = 0; k < IPT; ++k)
      if (gbk[k] >= 0) atomicAdd(&p.counts[gbk[k]], 1u);
  }
}

// Scatter of shared tile `tile` (its chunks have fewer than half a tile of
// records, so a sampled range holds all of them). s_rng, hist, bbase and bunit are the
// scatter kernel's LDS arrays; the largest ends are kept per bucket and kind
// slot: slot 0 in the kernel's bmaxe, slots 1 and 2 in bmaxe12 (2 x HW).
template <int THREADS, int IPT>
__device__ __forceinline__ void scatter_shared(const Plan& p, long long tile, ShTile& T, int (*s_rng)[THREADS / 64],
                                               unsigned long long* hist, unsigned long long* bbase,
                                               unsigned long long* bmaxe0, unsigned long long* bmaxe12,
                                               long long* bunit) {
  constexpr int NW = THREADS / 64;
  constexpr int HW = THREADS * IPT <= kHistWin ? THREADS * IPT / 4 : kHistWin;
  auto bmaxe = [&](int w, int sl) -> unsigned long long& { return sl == 0 ? bmaxe0[w] : bmaxe12[(sl - 1) * HW + w]; };
  for (int i = threadIdx.x; i < HW; i += THREADS) {
    hist[i] = 0;
    bmaxe0[i] = 0;
    bmaxe12[i] = 0;
    bmaxe12[HW + i] = 0;
  }
  sh_load<true>(p, tile, T);
  const int n = T.off[T.n];
  int jj[IPT], gbk[IPT];
  bool nr[IPT];
  unsigned int kx[IPT], ex[IPT];
  {
    long long svs[IPT], evs[IPT];
    sh_records<THREADS, IPT>(T, n, jj, svs, evs);
#pragma unroll
    for (int k = 0; k < IPT; ++k) {
      const int x = threadIdx.x + k * THREADS;
      gbk[k] = -1;
      nr[k] = false;
      kx[k] = 0;
      ex[k] = 0;
      if (x < n) {
        const int j = jj[k];
        const long long sv = svs[k], ev = evs[k];
        if (!rec_valid(sv, ev)) {
          // first bad record of the build: chunk << 40 | index (rare path)
          const ChunkDesc& cd = p.chunks[T.first + j];
          atomicMin(p.err, ((unsigned long long)cd.chunk_id << 40) | (unsigned long long)(x - T.off[j]));
          p.owner_err[cd.owner] = 1u;
        } else if (sv < ev) {
          const Geom& g = T.g[j];
          const int b = bucket_of(sv, g);
          const long long lo = bucket_lo(g, b);
          gbk[k] = (int)(T.bucket_begin[j] + b);
          nr[k] = seg_narrow(g);
          kx[k] = ((unsigned int)(sv - lo) << 2) | (unsigned int)T.slot[j];
          ex[k] = ev - lo < 0xFFFFFFFFll ? (unsigned int)(ev - lo + 1) : 0xFFFFFFFFu;  // far ends clamped
        }
      }
    }
  }
  int bmin = INT_MAX, bmax = -1;
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    if (gbk[k] >= 0) {
      bmin = min(bmin, gbk[k]);
      bmax = max(bmax, gbk[k]);
    }
  }
  bmin = wave_reduce_i32<OpMinI>(bmin, INT_MAX);
  bmax = wave_reduce_i32<OpMaxI>(bmax, -1);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) { s_rng[0][wave] = bmin; s_rng[1][wave] = bmax; }
  __syncthreads();
  bmin = INT_MAX; bmax = -1;
  for (int w = 0; w < NW; ++w) { bmin = min(bmin, s_rng[0][w]); bmax = max(bmax, s_rng[1][w]); }
  if (bmax < 0) return;  // uniform: no valid record in this tile
  const long long scap = p.slot_cap;
  unsigned long long* gmax = p.maxend;
  uint2* units = (uint2*)p.elems;
  auto region = [&](long long gb, long long& ub, long long& ucap) {
    if (scap) {
      ub = 2 * gb * scap;
      ucap = 2 * scap;
    } else {
      ub = 2 * (long long)p.offsets[gb];
      ucap = 2 * (long long)p.counts[gb];
    }
  };
  // a record in the 16 B form, read again from its chunk (rare)
  auto put_wide = [&](int k, long long ub, long long ucap, unsigned long long rank) {
    if (2 * ((long long)rank + 1) <= ucap) {
      const int j = jj[k];
      const int i = (int)threadIdx.x + k * THREADS - T.off[j];
      Elem el;
      el.s = T.s[j][i];
      el.e_slot = (long long)((unsigned long long)T.e[j][i] | ((unsigned long long)T.slot[j] << kSlotShift));
      *(Elem*)(units + ub + ucap - 2 * ((long long)rank + 1)) = el;
    }
  };
  auto end_of = [&](int k) { return T.e[jj[k]][(int)threadIdx.x + k * THREADS - T.off[jj[k]]]; };
  if (bmax - bmin < HW) {
    unsigned int rk[IPT];
    const unsigned long long lt = (1ull << lane) - 1ull;
#pragma unroll
    for (int k = 0; k < IPT; ++k) {
      // lanes of one bucket and kind share one LDS atomic: the leader reserves
      // their ranks (per form) and folds their largest end in
      rk[k] = 0;
      const int sl = gbk[k] >= 0 ? T.slot[jj[k]] : 0;
      unsigned long long todo = __ballot(gbk[k] >= 0);
      while (todo) {
        const int leader = __ffsll((long long)todo) - 1;
        const int lb = __builtin_amdgcn_readlane(gbk[k], leader);
        const int ls = __builtin_amdgcn_readlane(sl, leader);
        const bool in = gbk[k] == lb && sl == ls;
        const unsigned long long m = __ballot(in);
        const unsigned long long mn = __ballot(in && nr[k]);
        long long emax;
        unsigned int e32 = 0;
        if (mn == m) e32 = (unsigned int)wave_reduce_i32<OpMaxU32>((int)(in ? ex[k] : 0u), 0);
        if (mn == m && e32 != 0xFFFFFFFFu) {
          // all 8 B records, none clamped: the largest end in 32 bits, relative to the bucket
          const int jl = __builtin_amdgcn_readlane(jj[k], leader);
          emax = bucket_lo(T.g[jl], lb - T.bucket_begin[jl]) + (long long)e32 - 1;
        } else {
          emax = wave_reduce_i64<OpMax>(in ? end_of(k) : 0ll, 0ll);
        }
        unsigned long long b = 0;
        if (lane == leader) {
          const unsigned long long c8 = (unsigned long long)__popcll(mn), c16 = (unsigned long long)__popcll(m & ~mn);
          b = atomicAdd(&hist[lb - bmin], c8 | (c16 << 32));
          atomicMax(&bmaxe(lb - bmin, ls), (unsigned long long)emax);
        }
        b = (unsigned long long)readlane64((long long)b, leader);
        if (in) rk[k] = nr[k] ? (unsigned int)b + (unsigned int)__popcll(mn & lt)
                              : (unsigned int)(b >> 32) + (unsigned int)__popcll(m & ~mn & lt);
        todo &= ~m;
      }
    }
    __syncthreads();
    for (int i = threadIdx.x; i <= bmax - bmin; i += THREADS) {
      const unsigned long long h = hist[i];
      if (h) {
        const long long gb = (long long)bmin + i;
        const unsigned long long old = atomicAdd(&p.cursor[gb], h);
        bbase[i] = old;
        long long ub, ucap;
        region(gb, ub, ucap);
        bunit[i] = ub;
        for (int sl = 0; sl < 3; ++sl)
          if (bmaxe(i, sl)) atomicMax(&gmax[gb * 3 + sl], bmaxe(i, sl));
        const unsigned long long tot = (old & 0xFFFFFFFFull) + (old >> 32) + (h & 0xFFFFFFFFull) + (h >> 32);
        if (scap && tot > (unsigned long long)scap && tot - (h & 0xFFFFFFFFull) - (h >> 32) <= (unsigned long long)scap)
          atomicAdd(&p.oversized[1], 1ull);  // slot overflow: the build is redone with exact offsets
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < IPT; ++k) {
      if (gbk[k] >= 0) {
        const int w = gbk[k] - bmin;
        const unsigned long long bb = bbase[w];
        const long long ub = bunit[w];
        long long ub2, ucap;
        region(gbk[k], ub2, ucap);
        if (nr[k]) {
          const unsigned long long rank = (bb & 0xFFFFFFFFull) + rk[k];
          // non-temporal: written once here and read once by the merge, never cached in between
          if ((long long)rank < ucap) put_rec8(units + ub + (long long)rank, kx[k], ex[k]);
        } else {
          put_wide(k, ub, ucap, (bb >> 32) + rk[k]);
        }
      }
    }
  } else {
#pragma unroll
    for (int k = 0; k < IPT; ++k) {
      if (gbk[k] >= 0) {
        const long long gb = gbk[k];
        const unsigned long long old = atomicAdd(&p.cursor[gb], nr[k] ? 1ull : (1ull << 32));
        atomicMax(&gmax[gb * 3 + T.slot[jj[k]]], (unsigned long long)end_of(k));
        if (scap && (old & 0xFFFFFFFFull) + (old >> 32) == (unsigned long long)scap)
          atomicAdd(&p.oversized[1], 1ull);
        long long ub, ucap;
        region(gb, ub, ucap);
        if (nr[k]) {
          if ((long long)(old & 0xFFFFFFFFull) < ucap) units[ub + (long long)(old & 0xFFFFFFFFull)] = make_uint2(kx[k], ex[k]);
        } else {
          put_wide(k, ub, ucap, old >> 32);
        }
      }
    }
  }
}

// ----------------------------------------------------------------------------
// stats: validate records, per-segment min/max start and max end
// ----------------------------------------------------------------------------

template <int THREADS, bool kShared>
__global__ __launch_bounds__(THREADS) void k_stats(Plan p) {
  // The bucket grid needs only the range of starts; validation happens in the
  // scatter, which reads both ends anyway. Starts outside [0, 2^62) belong to
  // invalid records and are left out of the range.
  constexpr int NW = THREADS / 64;
  __shared__ unsigned long long red[2][NW];
  if constexpr (kShared) {
    if (blockIdx.x >= p.n_own_tiles) {
      __shared__ ShStatsSmem sh;
      stats_shared<THREADS>(p, blockIdx.x, sh);
      return;
    }
  }
  const long long tile = blockIdx.x;
  const ChunkDesc cd = p.chunks[p.tile_chunk[tile]];
  const long long base = (tile - cd.tile_begin) * (long long)p.tile_elems;
  const long long end = min((long long)cd.count, base + p.tile_elems);
  unsigned long long mn = ULLONG_MAX, mxs = 0;
  auto take = [&](unsigned long long s) {
    if (s < (unsigned long long)kTimeLimit) {
      mn = s < mn ? s : mn;
      mxs = s > mxs ? s : mxs;
    }
  };
  if ((((uintptr_t)cd.s) & 15) == 0 && end - base == p.tile_elems && (p.tile_elems & (2 * THREADS - 1)) == 0) {
    // a full tile from a 16 B aligned array: pairs of starts, all loads issued first
    const ulonglong2* v = (const ulonglong2*)(cd.s + base);
    const int npairs = p.tile_elems / 2;
    constexpr int U = 4;
    for (int j0 = threadIdx.x; j0 < npairs; j0 += U * THREADS) {
      ulonglong2 x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = j0 + u * THREADS < npairs ? get_pair_nt(v + j0 + u * THREADS) : make_ulonglong2(ULLONG_MAX, ULLONG_MAX);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        take(x[u].x);
        take(x[u].y);
      }
    }
  } else {
    for (long long i = base + threadIdx.x; i < end; i += THREADS) take((unsigned long long)cd.s[i]);
  }
  mn = wave_red_minu(mn);
  mxs = wave_red_maxu(mxs);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
    red[0][wave] = mn;
    red[1][wave] = mxs;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < NW; ++w) {
      mn = red[0][w] < mn ? red[0][w] : mn;
      mxs = red[1][w] > mxs ? red[1][w] : mxs;
    }
    if (mn != ULLONG_MAX) {
      atomicMin(&p.stats[cd.seg].min_s, mn);
      atomicMax(&p.stats[cd.seg].max_s, mxs);
    }
  }
}

// Small tiles (at most 512 records): one wave per tile, four tiles per
// workgroup, so a lane reduces 8 records instead of a workgroup reducing 2 per
// thread (traces of many small record batches have mostly partial tiles).
template <bool kShared>
__global__ __launch_bounds__(256) void k_stats_small(Plan p) {
  if constexpr (kShared) {
    // blocks past those of the other tiles: one shared tile each
    const long long own_blocks = (p.n_own_tiles + 3) / 4;
    if (blockIdx.x >= own_blocks) {
      __shared__ ShStatsSmem sh;
      stats_shared<256>(p, p.n_own_tiles + (blockIdx.x - own_blocks), sh);
      return;
    }
  }
  const int lane = threadIdx.x & 63;
  const long long tile = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (tile >= p.n_own_tiles) return;
  const ChunkDesc cd = p.chunks[p.tile_chunk[tile]];
  const long long base = (tile - cd.tile_begin) * (long long)p.tile_elems;
  const long long end = min((long long)cd.count, base + p.tile_elems);
  unsigned long long mn = ULLONG_MAX, mxs = 0;
  long long v[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) {  // all loads first, from positions clamped into the tile (base < end)
    const long long i = base + lane + 64 * k;
    v[k] = __builtin_nontemporal_load(cd.s + (i < end ? i : end - 1));
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const unsigned long long s = (unsigned long long)v[k];
    if (base + lane + 64 * k < end && s < (unsigned long long)kTimeLimit) {
      mn = s < mn ? s : mn;
      mxs = s > mxs ? s : mxs;
    }
  }
  mn = wave_red_minu(mn);
  mxs = wave_red_maxu(mxs);
  if (lane == 0 && mn != ULLONG_MAX) {
    atomicMin(&p.stats[cd.seg].min_s, mn);
    atomicMax(&p.stats[cd.seg].max_s, mxs);
  }
}

// Start range and bucket geometry of each segment (a workgroup per segment)
// from a sample of its starts, with the reset pass on the side if asked. The
// scatter checks every start against the range (put_outside). A pass over all
// starts reads 8 of the 24 B per record that the build's first half moves. With its reset and geometry
// kernels it took 178 us of the large trace's 1370, 28 of the mid trace's 232,
// 75 of the streams' 660 and 66 of 440 on a batch of 128 traces; this takes 14,
// 9, 18 and 38. What bounds it is four dependent reads, so a wave takes a
// third of a chunk's sample, not a chunk (mid: 11 us). A third lies in runs of 8
// starts across the chunk, as chunks need not be one piece of time: 256 resources
// whose 200,000 new records come in three pieces, the last one in the middle,
// take 475 us, and 1555 with samples of the chunk's two ends, where k_range takes
// 1-2 us less; with 128 runs instead of 64 it takes 17, 9, 23 and 40.
template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_range(Plan p, bool reset) {
  constexpr int NW = THREADS / 64, K = 8;
  __shared__ unsigned long long red[2][NW];
  __shared__ const int64_t* s_at[kRangeChunks];
  __shared__ int64_t s_count[kRangeChunks];
  if (reset) reset_counters(p);
  const int seg = blockIdx.x;
  if (seg >= p.n_segs) return;
  const int c0 = p.seg_first[seg], nch = p.seg_first[seg + 1] - c0;
  bool all = true;  // the sample holds every record
  for (int j = threadIdx.x; j < nch; j += THREADS) {
    const ChunkDesc& cd = p.chunks[p.seg_chunk[c0 + j]];
    s_at[j] = cd.s;
    s_count[j] = cd.count;
  }
  __syncthreads();
  unsigned long long mn = ULLONG_MAX, mx = 0;
  for (int j = 0; j < nch; ++j) all = all && s_count[j] <= kRangeSample;
  // a wave per third of a chunk's sample, K loads in flight per lane
  constexpr int kParts = kRangeSample / (64 * K);
  const int lane = threadIdx.x & 63;
  for (int u = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); u < nch * kParts; u += NW) {
    const int j = u / kParts, part = u % kParts;
    const int64_t* s = s_at[j];
    const long long n = s_count[j];
    // runs of 8 starts, `hop` apart: the first and the last third of the sample,
    // and short chunks, run on; the others spread over what lies between
    long long at = 64ll * K * part, hop = 8;
    if (n > kRangeSample) {
      if (part == kParts - 1) {
        at = n - 64 * K;
      } else if (part) {
        const long long runs = 8 * K * (kParts - 2);
        hop = (n - 2 * 64 * K - 8) / runs;
        at = 64 * K + hop / 2 + 8ll * K * (part - 1) * hop;
      }
    }
    if (at >= n) continue;
    const long long mine = at + (lane >> 3) * hop + (lane & 7);
    unsigned long long x[K];
#pragma unroll
    for (int k = 0; k < K; ++k) x[k] = (unsigned long long)s[min(mine + 8 * k * hop, n - 1)];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (x[k] < (unsigned long long)kTimeLimit) {  // other starts belong to invalid records
        mn = x[k] < mn ? x[k] : mn;
        mx = x[k] > mx ? x[k] : mx;
      }
    }
  }
  mn = wave_red_minu(mn);
  mx = wave_red_maxu(mx);
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = mn;
    red[1][threadIdx.x >> 6] = mx;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < NW; ++w) {
      mn = red[0][w] < mn ? red[0][w] : mn;
      mx = red[1][w] > mx ? red[1][w] : mx;
    }
    if (mn <= mx && !all) {
      const unsigned long long pad = ((mx - mn) >> kRangePad) + 1;
      mn = mn > pad ? mn - pad : 0;
      mx = min(mx + pad, (unsigned long long)kTimeLimit - 1);
    }
    SegStats st;
    st.min_s = mn;
    st.max_s = mx;
    st.max_e = 0;
    st.far_e = 0;
    p.stats[seg] = st;
    p.geom[seg] = make_geom(st, p.segs[seg]);
  }
}

// The bucket geometry of every segment from its start range (one thread per
// segment, after the start-range pass).
__global__ void k_geom(Plan p) {
  const long long seg = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (seg < p.n_segs) p.geom[seg] = make_geom(p.stats[seg], p.segs[seg]);
}

// ----------------------------------------------------------------------------
// hist / scatter: regroup records by time bucket
// ----------------------------------------------------------------------------

// Buckets of one tile usually span a narrow window (records arrive roughly in
// time order), so per-tile counting uses an LDS window [bmin, bmin + HW): kHistWin
// buckets, or a quarter of the tile's records for tiles of at most kHistWin records.
// Wider tiles fall back to global atomics per record.

template <int THREADS, int IPT, bool kShared>
__global__ __launch_bounds__(THREADS) void k_hist(Plan p) {
  constexpr int NW = THREADS / 64;
  constexpr int HW = THREADS * IPT <= kHistWin ? THREADS * IPT / 4 : kHistWin;  // LDS bucket window
  __shared__ int s_rng[2][NW];
  __shared__ unsigned int hist[HW];
  if constexpr (kShared) {
    if (blockIdx.x >= p.n_own_tiles) {
      __shared__ ShTile T;
      hist_shared<THREADS, IPT>(p, blockIdx.x, T, s_rng, hist);
      return;
    }
  }
  const long long tile = blockIdx.x;
  const ChunkDesc cd = p.chunks[p.tile_chunk[tile]];
  const SegDesc sd = p.segs[cd.seg];
  const Geom g = seg_geom(p, cd.seg);
  const long long base = (tile - cd.tile_begin) * (long long)p.tile_elems;
  const long long end = min((long long)cd.count, base + p.tile_elems);
  int bk[IPT];
  int bmin = INT_MAX, bmax = -1;
  // the loads of all rounds first, from positions clamped into the tile
  long long svs[IPT], evs[IPT];
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const long long i = base + threadIdx.x + (long long)k * THREADS;
    const long long ic = i < end ? i : end - 1;
    svs[k] = cd.s[ic];
    evs[k] = cd.e[ic];
  }
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const long long i = base + threadIdx.x + (long long)k * THREADS;
    bk[k] = -1;
    if (i < end) {
      const long long s = svs[k], e = evs[k];
      if (rec_valid(s, e) && s < e) {
        bk[k] = bucket_of(s, g);
        bmin = min(bmin, bk[k]);
        bmax = max(bmax, bk[k]);
      }
    }
  }
  bmin = wave_reduce_i32<OpMinI>(bmin, INT_MAX);
  bmax = wave_reduce_i32<OpMaxI>(bmax, -1);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) { s_rng[0][wave] = bmin; s_rng[1][wave] = bmax; }
  for (int i = threadIdx.x; i < HW; i += THREADS) hist[i] = 0;
  __syncthreads();
  bmin = INT_MAX; bmax = -1;
  for (int w = 0; w < NW; ++w) { bmin = min(bmin, s_rng[0][w]); bmax = max(bmax, s_rng[1][w]); }
  if (bmax < 0) return;  // uniform: no valid record in this tile
  const bool windowed = bmax - bmin < HW;
  if (windowed) {
#pragma unroll
    for (int k = 0; k < IPT; ++k) {
      // one LDS atomic per distinct bucket of the wave, not one per record
      unsigned long long todo = __ballot(bk[k] >= 0);
      while (todo) {
        const int leader = __ffsll((long long)todo) - 1;
        const int lb = __builtin_amdgcn_readlane(bk[k], leader);
        const unsigned long long m = __ballot(bk[k] == lb);
        if (lane == leader) atomicAdd(&hist[lb - bmin], (unsigned int)__popcll(m));
        todo &= ~m;
      }
    }
    __syncthreads();
    for (int i = threadIdx.x; i <= bmax - bmin; i += THREADS)
      if (hist[i]) atomicAdd(&p.counts[sd.bucket_begin + bmin + i], hist[i]);
  } else {
#pragma unroll
    for (int k = 0; k < IPT; ++k)
      if (bk[k] >= 0) atomicAdd(&p.counts[sd.bucket_begin + bk[k]], 1u);
  }
}

// exclusive scan of bucket counts -> offsets (decoupled look-back), one tile
// of kScanTile buckets per workgroup in the order of a ticket
template <int THREADS>
__device__ __forceinline__ void scan_tile(const Plan& p) {
  constexpr int IPT = kScanTile / THREADS;
  __shared__ unsigned int s_bid;
  __shared__ long long lds[THREADS / 64];
  __shared__ unsigned long long s_excl;
  if (threadIdx.x == 0) s_bid = atomicAdd(&p.ticket[0], 1u);
  __syncthreads();
  const long long bid = s_bid;
  const long long b0 = bid * kScanTile + (long long)threadIdx.x * IPT;
  unsigned int c[IPT];
  long long tsum = 0;
  const bool slots = p.slot_cap > 0;
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    c[k] = 0u;
    if (b0 + k < p.n_buckets) {
      if (slots) {
        // counts of the single-pass scatter (capped: an overflow is redone exactly)
        const unsigned long long cu = p.cursor[b0 + k];
        const unsigned long long n = (cu & 0xFFFFFFFFull) + (cu >> 32);
        c[k] = (unsigned int)(n < (unsigned long long)p.slot_cap ? n : (unsigned long long)p.slot_cap);
        p.counts[b0 + k] = c[k];
      } else {
        c[k] = p.counts[b0 + k];
      }
    }
    tsum += c[k];
  }
  long long v[1] = {tsum}, ex[1], tot[1];
  block_excl_scan<THREADS, 1, OpSum>(v, ex, tot, 0, lds);
  // The counts of all earlier tiles: the first wave reads 64 predecessors at
  // once, nearest first (lane i: tile j - i), up to one whose inclusive sum is
  // known. One at a time, the last of 9 tiles waited for 8 round trips: with tiles
  // of 4096 buckets the launch took 12.8 us on the mid trace, 16 on 256 devices
  // with their streams and 6 on the small trace; with 1024 it takes 5.9, 9 and
  // 3.4. Tickets are taken in order, so every predecessor runs or has run.
  constexpr unsigned long long FLAG_AGG = 1ull << 62, FLAG_INC = 2ull << 62, VMASK = (1ull << 62) - 1;
  if (threadIdx.x < 64) {
    unsigned long long* st = p.scan_state;
    const int lane = threadIdx.x;
    if (lane == 0)
      __hip_atomic_store(&st[bid], (bid == 0 ? FLAG_INC : FLAG_AGG) | (unsigned long long)tot[0], __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    unsigned long long acc = 0;
    for (long long j = bid - 1; j >= 0;) {
      const unsigned long long w =
          j >= lane ? __hip_atomic_load(&st[j - lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : FLAG_INC;
      const unsigned long long none = __ballot((w & ~VMASK) == 0), inc = __ballot((w & ~VMASK) == FLAG_INC);
      // lanes up to the nearest inclusive sum (past tile 0 they hold an empty one)
      const unsigned long long use = inc ? (inc & (0ull - inc)) | ((inc & (0ull - inc)) - 1ull) : ~0ull;
      if (none & use) {
        __builtin_amdgcn_s_sleep(1);
        continue;
      }
      acc += (unsigned long long)wave_reduce_i64<OpSum>((use >> lane) & 1 ? (long long)(w & VMASK) : 0ll, 0ll);
      if (inc) break;
      j -= 64;
    }
    if (lane == 0) {
      if (bid > 0)
        __hip_atomic_store(&st[bid], FLAG_INC | (acc + (unsigned long long)tot[0]), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
      s_excl = acc;
    }
  }
  __syncthreads();
  unsigned long long run = s_excl + (unsigned long long)ex[0];
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    if (b0 + k < p.n_buckets) {
      p.offsets[b0 + k] = run;  // cursors stay relative: the scatter adds the bucket's base
      if (c[k] > (unsigned)p.cap) atomicAdd(p.oversized, 1ull);
    }
    run += c[k];
  }
  // the thread holding the last bucket also writes the grand total
  if (b0 < p.n_buckets && p.n_buckets <= b0 + IPT) p.offsets[p.n_buckets] = run;
}

template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_scan(Plan p) {
  scan_tile<THREADS>(p);
}

// The records of a tile that start outside the sampled range of its segment, few
// as a rule (fixed slots only), go to the segment's first or last bucket, in the
// 16 B form. One before the range lowers the segment's first start, and its end
// counts for the buckets after it; the end of one past the range must not pass for
// the largest end of the last bucket's 8 B records (clamped ones take that), and
// goes to the segment. Called by the waves that met one.
//
// Reading every start instead takes a pass over 8 of the build's first 24 B per
// record, and building again where a sample missed up to twice as long (256
// resources of 200,000 records, one start apart: 717 us with every start read,
// 1042 with a second build, 478 so). A tile that lies outside from end to end asks
// for the build with exact offsets at once: with a third of those records outside
// (while only a chunk's two ends were sampled), the adds to the same few counters
// took the two builds to 4.8 ms, 1.56 without them. The
// branch here is the wave's and the code behind it each lane's: with a branch per
// lane, or with wave operations or two paths behind it, the registers and compares
// of the records above change, and the scatter, which hardly ever comes here, takes
// 511-525 us for 1.25e8 records instead of 505.
struct OutsideArgs {
  const int64_t* s;    // the tile's records, n of them
  const int64_t* e;
  int n, slot;
  long long first;     // of the segment's buckets the first and the last
  long long last;
  long long min_s, cap;
  unsigned int cover;  // start_in_range: units of 2^s0 ns
  int s0;
  unsigned long long* cursor;
  unsigned long long* maxend;
  unsigned long long* oversized;
  SegStats* st;
  uint2* units;
};
template <int THREADS>
__device__ __forceinline__ void put_outside(const OutsideArgs& a) {
  auto outside = [&](long long sv, long long ev) {
    return rec_valid(sv, ev) && sv < ev && ((unsigned long long)(sv - a.min_s) >> a.s0) >= (unsigned long long)a.cover;
  };
  // a tile that lies outside from end to end is one of many: they would fill the slots
  if (outside(a.s[0], a.e[0]) && outside(a.s[a.n - 1], a.e[a.n - 1]) && a.n > THREADS) {
    if (threadIdx.x == 0) atomicAdd(a.oversized, 1ull);
    return;
  }
#pragma unroll 1
  for (int i = (int)threadIdx.x; i < a.n; i += THREADS) {
    const long long sv = a.s[i], ev = a.e[i];
    if (!outside(sv, ev)) continue;
    const bool past = sv >= a.min_s;
    const long long gb = past ? a.last : a.first;
    const unsigned long long old = atomicAdd(&a.cursor[gb], 1ull << 32);
    if ((long long)((old & 0xFFFFFFFFull) + (old >> 32)) == a.cap)
      atomicAdd(a.oversized, 1ull);  // slot overflow: the build is redone with exact offsets
    atomicMax(past ? &a.st->far_e : &a.maxend[gb * 3 + a.slot], (unsigned long long)ev);
    atomicMin(&a.st->min_s, (unsigned long long)sv);
    const long long rank = (long long)(old >> 32);
    if (rank < a.cap) {
      Elem el;
      el.s = sv;
      el.e_slot = (long long)((unsigned long long)ev | ((unsigned long long)a.slot << kSlotShift));
      *(Elem*)(a.units + 2 * gb * a.cap + 2 * a.cap - 2 * (rank + 1)) = el;
    }
  }
}

template <int THREADS, int IPT, bool kShared>
__global__ __launch_bounds__(THREADS) void k_scatter(Plan p) {
  constexpr int NW = THREADS / 64;
  // LDS bucket window: a quarter of the tile's records for tiles of at most kHistWin records
  constexpr int HW = THREADS * IPT <= kHistWin ? THREADS * IPT / 4 : kHistWin;
  __shared__ int s_rng[2][NW];
  __shared__ unsigned long long hist[HW];   // per window bucket: 8 B records | 16 B records << 32
  __shared__ unsigned long long bbase[HW];  // the same counts placed before this tile
  __shared__ unsigned long long bmaxe[HW];  // largest end of the tile's records
  __shared__ long long bunit[HW];           // first unit of the bucket's region
  if constexpr (kShared) {
    if (blockIdx.x >= p.n_own_tiles) {
      __shared__ ShTile T;
      __shared__ unsigned long long bmaxe12[2 * HW];
      scatter_shared<THREADS, IPT>(p, blockIdx.x, T, s_rng, hist, bbase, bmaxe, bmaxe12, bunit);
      return;
    }
  }
  const long long tile = blockIdx.x;
  const ChunkDesc cd = p.chunks[p.tile_chunk[tile]];
  const SegDesc sd = p.segs[cd.seg];
  const Geom g = seg_geom(p, cd.seg);
  const bool seg_n = seg_narrow(g);
  // 32-bit places within the tile: the loads take a wave-uniform base
  const long long base = (tile - cd.tile_begin) * (long long)p.tile_elems;
  const int n_tile = (int)min((long long)p.tile_elems, cd.count - base);
  const int64_t* ts = cd.s + base;
  const int64_t* te = cd.e + base;
  // per record: bucket (-1: none) and the 8 B form itself; a record in the 16 B
  // form (those of wide segments) is read again where it is needed
  int bk[IPT];
  bool out = false;  // a record of this thread starts outside the sampled range
  unsigned int kx[IPT], ex[IPT];
  int bmin = INT_MAX, bmax = -1;
  // the loads of all rounds first, from positions clamped into the tile
  // (n_tile > 0): they issue back to back instead of one masked block (and
  // one wait) per round; non-temporal, as this pass reads each record once
  long long svs[IPT], evs[IPT];
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const unsigned int ic = (unsigned int)min((int)threadIdx.x + k * THREADS, n_tile - 1);
    svs[k] = __builtin_nontemporal_load(ts + ic);
    evs[k] = __builtin_nontemporal_load(te + ic);
  }
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const int i = (int)threadIdx.x + k * THREADS;
    bk[k] = -1;
    kx[k] = 0;
    ex[k] = 0;
    if (i < n_tile) {
      const long long sv = svs[k], ev = evs[k];
      if (!rec_valid(sv, ev)) {
        // first bad record of the build: chunk << 40 | index (rare path)
        atomicMin(p.err, ((unsigned long long)cd.chunk_id << 40) | (unsigned long long)(base + i));
        p.owner_err[cd.owner] = 1u;
      } else if (sv < ev && !start_in_range(g, sv)) {
        out = true;
      } else if (sv < ev) {
        const unsigned long long rel = (unsigned long long)(sv - g.min_s);
        bk[k] = (int)geom_div(g, (unsigned int)(rel >> g.s0));
        // start and end relative to the bucket's first time, for narrow
        // segments (others don't use them): the start's distance fits 32 bits,
        // so the low words do, and the end is the start plus the length
        const unsigned int from = (unsigned int)rel - (((unsigned int)bk[k] * g.wx) << g.s0);
        const unsigned long long to = (unsigned long long)(ev - sv) + from + 1ull;
        kx[k] = (from << 2) | (unsigned int)cd.slot;
        ex[k] = to >> 32 ? 0xFFFFFFFFu : (unsigned int)to;  // far ends clamped
        bmin = min(bmin, bk[k]);
        bmax = max(bmax, bk[k]);
      }
    }
  }
  if (__ballot(out))
    put_outside<THREADS>(OutsideArgs{ts, te, n_tile, cd.slot, sd.bucket_begin, sd.bucket_begin + sd.nb - 1, g.min_s,
                                     p.slot_cap, range_units(g), g.s0, p.cursor, p.maxend, p.oversized + 1,
                                     p.stats + cd.seg, (uint2*)p.elems});
  bmin = wave_reduce_i32<OpMinI>(bmin, INT_MAX);
  bmax = wave_reduce_i32<OpMaxI>(bmax, -1);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long scap = p.slot_cap;
  if (lane == 0) { s_rng[0][wave] = bmin; s_rng[1][wave] = bmax; }
  for (int i = threadIdx.x; i < HW; i += THREADS) { hist[i] = 0; bmaxe[i] = 0; }
  __syncthreads();
  bmin = INT_MAX; bmax = -1;
  for (int w = 0; w < NW; ++w) { bmin = min(bmin, s_rng[0][w]); bmax = max(bmax, s_rng[1][w]); }
  if (bmax < 0) return;
  const unsigned long long slotbits = (unsigned long long)cd.slot << kSlotShift;
  unsigned long long* gmax = p.maxend;
  uint2* units = (uint2*)p.elems;
  auto region = [&](long long gb, long long& ub, long long& ucap) {
    if (scap) {
      ub = 2 * gb * scap;
      ucap = 2 * scap;
    } else {
      ub = 2 * (long long)p.offsets[gb];
      ucap = 2 * (long long)p.counts[gb];
    }
  };
  auto put_wide = [&](int k, long long ub, long long ucap, unsigned long long rank) {
    if (2 * ((long long)rank + 1) <= ucap) {
      const int i = (int)threadIdx.x + k * THREADS;
      Elem el;
      el.s = ts[i];
      el.e_slot = (long long)((unsigned long long)te[i] | slotbits);
      *(Elem*)(units + ub + ucap - 2 * ((long long)rank + 1)) = el;
    }
  };
  if (bmax - bmin < HW) {
    unsigned int rk[IPT];
    // the records of round k in bucket lb, as one wave (lanes `m`, this lane
    // among them or not): their ranks and largest end by one LDS atomic each
    auto reserve = [&](int k, int lb, bool in, unsigned long long m, int leader) {
      unsigned int e32 = 0xFFFFFFFFu;
      if (seg_n) e32 = (unsigned int)wave_reduce_i32<OpMaxU32>((int)(in ? ex[k] : 0u), 0);
      long long emax;
      if (e32 != 0xFFFFFFFFu) {
        // all 8 B records, none clamped: the largest end in 32 bits, relative to the bucket
        emax = bucket_lo(g, lb) + (long long)e32 - 1;
      } else {
        long long ev = 0;
        if (in) ev = te[threadIdx.x + k * THREADS];
        emax = wave_reduce_i64<OpMax>(ev, 0ll);
      }
      unsigned long long b = 0;
      if (lane == leader) {
        const unsigned long long n = (unsigned long long)__popcll(m);
        b = atomicAdd(&hist[lb - bmin], seg_n ? n : n << 32);
        atomicMax(&bmaxe[lb - bmin], (unsigned long long)emax);
      }
      b = (unsigned long long)readlane64((long long)b, leader);
      if (in) rk[k] = (seg_n ? (unsigned int)b : (unsigned int)(b >> 32)) + lanes_below(m);
    };
    if (seg_n) {
      // A round's 64 records mostly lie in one or two buckets. The first two of
      // every round get their ranks and largest ends from one LDS atomic of the
      // wave (lane 2k + i: bucket i of round k) instead of a dependent one per
      // bucket and round: the kernel is bound by these chains and by its waves
      // in flight as much as by its 24 B per record (large trace: 601 -> 567 us,
      // 504 with 2048-record tiles, 6.0 TB/s; mid 73 -> 60; 256 devices with
      // their streams 274 -> 213; the small trace 7.5 -> 5.9).
      int vb = 0;                     // bucket, window-relative
      unsigned int vn = 0, ve = 0;    // its records, and their largest end relative to the bucket
      unsigned int second = 0, done = 0;  // bit k: this lane's record of round k is in bucket 1 / has its rank already
#pragma unroll
      for (int k = 0; k < IPT; ++k) {
        rk[k] = 0;
        unsigned long long todo = __ballot(bk[k] >= 0);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          if (todo) {  // uniform
            const int leader = __ffsll((long long)todo) - 1;
            const int lb = __builtin_amdgcn_readlane(bk[k], leader);
            const bool in = bk[k] == lb;
            const unsigned long long m = __ballot(in);
            unsigned int e32 = (unsigned int)wave_reduce_i32<OpMaxU32>((int)(in ? ex[k] : 0u), 0);
            if (e32 == 0xFFFFFFFFu) {  // a far end (clamped): the true ends again
              long long ev = 0;
              if (in) ev = te[threadIdx.x + k * THREADS];
              const long long emax = wave_reduce_i64<OpMax>(ev, 0ll);
              if (lane == leader) atomicMax(&bmaxe[lb - bmin], (unsigned long long)emax);
              e32 = 0;
            }
            if (lane == 2 * k + i) {
              vb = lb - bmin;
              vn = (unsigned int)__popcll(m);
              ve = e32;
            }
            if (in) {
              rk[k] = lanes_below(m);
              second |= (unsigned int)i << k;
            }
            todo &= ~m;
          }
        }
        while (todo) {
          const int leader = __ffsll((long long)todo) - 1;
          const int lb = __builtin_amdgcn_readlane(bk[k], leader);
          const bool in = bk[k] == lb;
          const unsigned long long m = __ballot(in);
          reserve(k, lb, in, m, leader);
          if (in) done |= 1u << k;
          todo &= ~m;
        }
      }
      unsigned int before = 0;
      if (vn) {
        before = (unsigned int)atomicAdd(&hist[vb], (unsigned long long)vn);
        if (ve) atomicMax(&bmaxe[vb], (unsigned long long)(bucket_lo(g, vb + bmin) + (long long)ve - 1));
      }
#pragma unroll
      for (int k = 0; k < IPT; ++k) {
        const unsigned int b0 = (unsigned int)__builtin_amdgcn_readlane((int)before, 2 * k);
        const unsigned int b1 = (unsigned int)__builtin_amdgcn_readlane((int)before, 2 * k + 1);
        rk[k] += done & (1u << k) ? 0u : (second & (1u << k) ? b1 : b0);
      }
    } else {
#pragma unroll
      for (int k = 0; k < IPT; ++k) {
        rk[k] = 0;
        unsigned long long todo = __ballot(bk[k] >= 0);
        while (todo) {
          const int leader = __ffsll((long long)todo) - 1;
          const int lb = __builtin_amdgcn_readlane(bk[k], leader);
          const bool in = bk[k] == lb;
          const unsigned long long m = __ballot(in);
          reserve(k, lb, in, m, leader);
          todo &= ~m;
        }
      }
    }
    __syncthreads();
    for (int i = threadIdx.x; i <= bmax - bmin; i += THREADS) {
      const unsigned long long h = hist[i];
      if (h) {
        const long long gb = sd.bucket_begin + bmin + i;
        const unsigned long long old = atomicAdd(&p.cursor[gb], h);
        bbase[i] = old;
        long long ub, ucap;
        region(gb, ub, ucap);
        bunit[i] = ub;
        atomicMax(&gmax[gb * 3 + cd.slot], bmaxe[i]);
        const unsigned long long tot = (old & 0xFFFFFFFFull) + (old >> 32) + (h & 0xFFFFFFFFull) + (h >> 32);
        if (scap && tot > (unsigned long long)scap && tot - (h & 0xFFFFFFFFull) - (h >> 32) <= (unsigned long long)scap)
          atomicAdd(&p.oversized[1], 1ull);  // slot overflow: the build is redone with exact offsets
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < IPT; ++k) {
      if (bk[k] >= 0) {
        const int w = bk[k] - bmin;
        const unsigned long long bb = bbase[w];
        const long long ub = bunit[w];
        if (seg_n) {
          const unsigned long long rank = (bb & 0xFFFFFFFFull) + rk[k];
          const long long ucap = scap ? 2 * scap : 2 * (long long)p.counts[sd.bucket_begin + bk[k]];
          // non-temporal: written once here and read once by the merge, never cached in between
          if ((long long)rank < ucap) put_rec8(units + ub + (long long)rank, kx[k], ex[k]);
        } else {
          long long ub2, ucap;
          region(sd.bucket_begin + bk[k], ub2, ucap);
          put_wide(k, ub, ucap, (bb >> 32) + rk[k]);
        }
      }
    }
  } else {
#pragma unroll
    for (int k = 0; k < IPT; ++k) {
      if (bk[k] >= 0) {
        const long long gb = sd.bucket_begin + bk[k];
        const unsigned long long old = atomicAdd(&p.cursor[gb], seg_n ? 1ull : (1ull << 32));
        const long long ev = te[threadIdx.x + k * THREADS];
        atomicMax(&gmax[gb * 3 + cd.slot], (unsigned long long)ev);
        if (scap && (old & 0xFFFFFFFFull) + (old >> 32) == (unsigned long long)scap)
          atomicAdd(&p.oversized[1], 1ull);
        long long ub, ucap;
        region(gb, ub, ucap);
        if (seg_n) {
          if ((long long)(old & 0xFFFFFFFFull) < ucap) units[ub + (long long)(old & 0xFFFFFFFFull)] = make_uint2(kx[k], ex[k]);
        } else {
          put_wide(k, ub, ucap, old >> 32);
        }
      }
    }
  }
}

// ----------------------------------------------------------------------------
// carry / base: per-segment scans over buckets, one wave per segment. A round
// covers kSegRows x 64 buckets: all of its loads are issued first (row j,
// lane i: bucket c0 + 64 j + i, coalesced), then one DPP scan per row in
// bucket order, then the stores; so a round costs one memory round trip
// ----------------------------------------------------------------------------

constexpr int kSegRows = 8;

// The carry pass of segment `seg` by one whole wave (every lane calls).
__device__ __forceinline__ void carry_segment(const Plan& p, long long seg, int lane) {
  const SegDesc sd = p.segs[seg];
  const SegStats st = p.stats[seg];
  const long long nb = sd.nb;
  // the running max end before any record: just below the first start
  const long long init = st.min_s > st.max_s ? -1 : (long long)st.min_s - 1;
  long long run[3] = {init, init, init};
  for (long long c0 = 0; c0 < nb; c0 += 64 * kSegRows) {
    unsigned long long m[kSegRows][3];
#pragma unroll
    for (int j = 0; j < kSegRows; ++j) {
      const long long b = c0 + 64 * j + lane;
      m[j][0] = m[j][1] = m[j][2] = 0;
      if (b < nb) {
        p.bucket_seg[sd.bucket_begin + b] = (int32_t)seg;
        const unsigned long long* q = p.maxend + (sd.bucket_begin + b) * 3;
        m[j][0] = q[0];
        m[j][1] = q[1];
        m[j][2] = q[2];
      }
    }
#pragma unroll
    for (int j = 0; j < kSegRows; ++j) {
      if (c0 + 64 * j >= nb) break;  // wave-uniform: rows past the segment change nothing
      const long long b = c0 + 64 * j + lane;
      long long v[3];
      v[0] = m[j][0] ? (long long)m[j][0] : LLONG_MIN;
      const long long m1 = m[j][1] ? (long long)m[j][1] : LLONG_MIN;
      const long long m2 = m[j][2] ? (long long)m[j][2] : LLONG_MIN;
      v[1] = m1 > v[0] ? m1 : v[0];
      v[2] = m2 > v[1] ? m2 : v[1];
#pragma unroll
      for (int l = 0; l < 3; ++l) {
        long long all;
        const long long ex = wave_excl_scan_dpp<OpMax>(v[l], LLONG_MIN, all);
        if (b < nb) p.carry[(sd.bucket_begin + b) * 3 + l] = ex > run[l] ? ex : run[l];
        run[l] = all > run[l] ? all : run[l];
      }
    }
  }
  // largest end of the segment (level 2 holds every kind); no record: the min start
  run[2] = max(run[2], (long long)st.far_e);
  if (lane == 0) p.stats[seg].max_e = (unsigned long long)(run[2] > init ? run[2] : (init + 1 > 0 ? init + 1 : 0));
}

// Segments of many buckets (128 and more on average): a workgroup each. A wave
// scans 64 buckets at a time, row after row: segments of 700 buckets took the
// carry pass 16 us and the base pass 13. A workgroup takes 4 x 256 per round,
// all loads first: 11 and 10 (segments of 300: 7 and 5.5, now 5.5 and 5.3).
constexpr int kBigRows = 4;

__device__ __forceinline__ void carry_segment_big(const Plan& p, long long seg) {
  __shared__ long long lds[4 * 3];
  const SegDesc sd = p.segs[seg];
  const SegStats st = p.stats[seg];
  const long long nb = sd.nb;
  const long long init = st.min_s > st.max_s ? -1 : (long long)st.min_s - 1;
  long long run[3] = {init, init, init};
  for (long long c0 = 0; c0 < nb; c0 += 256 * kBigRows) {
    unsigned long long m[kBigRows][3];
#pragma unroll
    for (int j = 0; j < kBigRows; ++j) {
      const long long b = c0 + 256 * j + threadIdx.x;
      m[j][0] = m[j][1] = m[j][2] = 0;
      if (b < nb) {
        p.bucket_seg[sd.bucket_begin + b] = (int32_t)seg;
        const unsigned long long* q = p.maxend + (sd.bucket_begin + b) * 3;
        m[j][0] = q[0];
        m[j][1] = q[1];
        m[j][2] = q[2];
      }
    }
#pragma unroll
    for (int j = 0; j < kBigRows; ++j) {
      if (c0 + 256 * j >= nb) break;  // uniform
      const long long b = c0 + 256 * j + threadIdx.x;
      long long v[3], ex[3], all[3];
      v[0] = m[j][0] ? (long long)m[j][0] : LLONG_MIN;
      const long long m1 = m[j][1] ? (long long)m[j][1] : LLONG_MIN;
      const long long m2 = m[j][2] ? (long long)m[j][2] : LLONG_MIN;
      v[1] = m1 > v[0] ? m1 : v[0];
      v[2] = m2 > v[1] ? m2 : v[1];
      block_excl_scan<256, 3, OpMax>(v, ex, all, LLONG_MIN, lds);
#pragma unroll
      for (int l = 0; l < 3; ++l) {
        if (b < nb) p.carry[(sd.bucket_begin + b) * 3 + l] = ex[l] > run[l] ? ex[l] : run[l];
        run[l] = all[l] > run[l] ? all[l] : run[l];
      }
    }
  }
  run[2] = max(run[2], (long long)st.far_e);
  if (threadIdx.x == 0)
    p.stats[seg].max_e = (unsigned long long)(run[2] > init ? run[2] : (init + 1 > 0 ? init + 1 : 0));
}

__global__ __launch_bounds__(256) void k_base_big(Plan p) {
  __shared__ long long lds[4 * 3];
  const long long seg = blockIdx.x;
  const SegDesc sd = p.segs[seg];
  const long long nb = sd.nb;
  long long run[3] = {0, 0, 0};
  for (long long c0 = 0; c0 < nb; c0 += 256 * kBigRows) {
    long long v[kBigRows][3];
#pragma unroll
    for (int j = 0; j < kBigRows; ++j) {
      const long long b = c0 + 256 * j + threadIdx.x;
#pragma unroll
      for (int l = 0; l < 3; ++l) v[j][l] = b < nb ? p.bsum[(sd.bucket_begin + b) * 3 + l] : 0;
    }
#pragma unroll
    for (int j = 0; j < kBigRows; ++j) {
      if (c0 + 256 * j >= nb) break;  // uniform
      const long long b = c0 + 256 * j + threadIdx.x;
      long long ex[3], all[3];
      block_excl_scan<256, 3, OpSum>(v[j], ex, all, 0, lds);
#pragma unroll
      for (int l = 0; l < 3; ++l) {
        if (b < nb) p.base[(sd.bucket_begin + b) * 3 + l] = run[l] + ex[l];
        run[l] += all[l];
      }
    }
  }
  if (threadIdx.x < 3) p.seg_total[seg * 3 + threadIdx.x] = threadIdx.x == 0 ? run[0] : (threadIdx.x == 1 ? run[1] : run[2]);
}

template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_carry(Plan p) {
  const int lane = threadIdx.x & 63;
  const long long seg = (long long)blockIdx.x * (THREADS / 64) + (threadIdx.x >> 6);
  if (seg >= p.n_segs) return;
  carry_segment(p, seg, lane);
}

// The base pass of segment `seg` by one whole wave (every lane calls).
__device__ __forceinline__ void base_segment(const Plan& p, long long seg, int lane) {
  const SegDesc sd = p.segs[seg];
  const long long nb = sd.nb;
  long long run[3] = {0, 0, 0};
  for (long long c0 = 0; c0 < nb; c0 += 64 * kSegRows) {
    long long v[kSegRows][3];
#pragma unroll
    for (int j = 0; j < kSegRows; ++j) {
      const long long b = c0 + 64 * j + lane;
#pragma unroll
      for (int l = 0; l < 3; ++l) v[j][l] = b < nb ? p.bsum[(sd.bucket_begin + b) * 3 + l] : 0;
    }
#pragma unroll
    for (int j = 0; j < kSegRows; ++j) {
      if (c0 + 64 * j >= nb) break;  // wave-uniform: rows past the segment add nothing
      const long long b = c0 + 64 * j + lane;
#pragma unroll
      for (int l = 0; l < 3; ++l) {
        long long all;
        const long long ex = wave_excl_scan_dpp<OpSum>(v[j][l], 0, all);
        if (b < nb) p.base[(sd.bucket_begin + b) * 3 + l] = run[l] + ex;
        run[l] += all;
      }
    }
  }
  if (lane == 0) {
    for (int l = 0; l < 3; ++l) p.seg_total[seg * 3 + l] = run[l];
  }
}

template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_base(Plan p) {
  const int lane = threadIdx.x & 63;
  const long long seg = (long long)blockIdx.x * (THREADS / 64) + (threadIdx.x >> 6);
  if (seg >= p.n_segs) return;
  base_segment(p, seg, lane);
}

// Plans of many small segments (a batch of small traces): a wave takes
// kSegGroup consecutive segments. A segment of at most kSegGroup buckets is
// scanned by its own group of kSegGroup lanes (a lane per bucket, scans by
// lane shuffles within the group); the larger ones of the wave follow, one
// after another, with the whole wave as above.
constexpr int kSegGroup = 8;

// inclusive scan over the kSegGroup lanes of a group (identity in lanes past
// the segment's buckets)
template <class Op>
__device__ __forceinline__ long long group_incl_scan(long long v, int k) {
#pragma unroll
  for (int d = 1; d < kSegGroup; d <<= 1) {
    const long long o = __shfl_up(v, (unsigned)d, kSegGroup);
    if (k >= d) v = Op::apply(v, o);
  }
  return v;
}

// The carry pass of segments [w kSegGroup, (w + 1) kSegGroup) by one wave.
__device__ __forceinline__ void carry_group(const Plan& p, long long w, int lane) {
  const int k = lane & (kSegGroup - 1);
  const long long seg0 = w * kSegGroup;
  if (seg0 >= p.n_segs) return;
  const long long seg = seg0 + (lane / kSegGroup);
  const bool have = seg < p.n_segs;
  const SegDesc sd = have ? p.segs[seg] : SegDesc{0, 0, 0};
  const bool small = have && sd.nb <= kSegGroup;
  if (small) {  // uniform within each group
    const SegStats st = p.stats[seg];
    const long long init = st.min_s > st.max_s ? -1 : (long long)st.min_s - 1;
    long long v[3] = {LLONG_MIN, LLONG_MIN, LLONG_MIN};
    if (k < sd.nb) {
      const long long gb = sd.bucket_begin + k;
      p.bucket_seg[gb] = (int32_t)seg;
      const unsigned long long* q = p.maxend + gb * 3;
      const unsigned long long m0 = q[0], m1 = q[1], m2 = q[2];
      v[0] = m0 ? (long long)m0 : LLONG_MIN;
      v[1] = m1 && (long long)m1 > v[0] ? (long long)m1 : v[0];
      v[2] = m2 && (long long)m2 > v[1] ? (long long)m2 : v[1];
    }
    long long last2 = init;
#pragma unroll
    for (int l = 0; l < 3; ++l) {
      const long long inc = group_incl_scan<OpMax>(v[l], k);
      long long ex = __shfl_up(inc, 1u, kSegGroup);
      if (k == 0) ex = LLONG_MIN;
      if (k < sd.nb) p.carry[(sd.bucket_begin + k) * 3 + l] = ex > init ? ex : init;
      if (l == 2) last2 = __shfl(inc, kSegGroup - 1, kSegGroup);
    }
    const long long r2 = max(max(last2, (long long)st.far_e), init);
    if (k == 0) p.stats[seg].max_e = (unsigned long long)(r2 > init ? r2 : (init + 1 > 0 ? init + 1 : 0));
  }
  unsigned long long big = __ballot(k == 0 && have && !small);
  while (big) {
    const int g = __ffsll((long long)big) - 1;
    big &= big - 1;
    carry_segment(p, seg0 + g / kSegGroup, lane);
  }
}

template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_carry_grouped(Plan p) {
  carry_group(p, (long long)blockIdx.x * (THREADS / 64) + (threadIdx.x >> 6), threadIdx.x & 63);
}

// Fixed slots: the bucket scan and the carry pass read only what the scatter
// wrote, so one launch does both: workgroups [0, scan_blocks) scan (tiles in
// ticket order), the ones after give each wave a segment (or a group of
// kSegGroup segments), or take a segment themselves (kBig).
template <bool kGrouped, bool kBig = false>
__global__ __launch_bounds__(256) void k_scan_carry(Plan p, int scan_blocks) {
  if ((int)blockIdx.x < scan_blocks) {
    scan_tile<256>(p);
    return;
  }
  if constexpr (kBig) {
    carry_segment_big(p, blockIdx.x - scan_blocks);
    return;
  }
  const int lane = threadIdx.x & 63;
  const long long w = (long long)(blockIdx.x - scan_blocks) * 4 + (threadIdx.x >> 6);
  if constexpr (kGrouped) {
    carry_group(p, w, lane);
  } else {
    if (w < p.n_segs) carry_segment(p, w, lane);
  }
}

template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_base_grouped(Plan p) {
  const int lane = threadIdx.x & 63, k = lane & (kSegGroup - 1);
  const long long seg0 = ((long long)blockIdx.x * (THREADS / 64) + (threadIdx.x >> 6)) * kSegGroup;
  if (seg0 >= p.n_segs) return;
  const long long seg = seg0 + (lane / kSegGroup);
  const bool have = seg < p.n_segs;
  const SegDesc sd = have ? p.segs[seg] : SegDesc{0, 0, 0};
  const bool small = have && sd.nb <= kSegGroup;
  if (small) {  // uniform within each group
#pragma unroll
    for (int l = 0; l < 3; ++l) {
      const long long v = k < sd.nb ? p.bsum[(sd.bucket_begin + k) * 3 + l] : 0;
      const long long inc = group_incl_scan<OpSum>(v, k);
      if (k < sd.nb) p.base[(sd.bucket_begin + k) * 3 + l] = inc - v;
      const long long tot = __shfl(inc, kSegGroup - 1, kSegGroup);
      if (k == 0) p.seg_total[seg * 3 + l] = tot;
    }
  }
  unsigned long long big = __ballot(k == 0 && have && !small);
  while (big) {
    const int g = __ffsll((long long)big) - 1;
    big &= big - 1;
    base_segment(p, seg0 + g / kSegGroup, lane);
  }
}

// ----------------------------------------------------------------------------
// merge: per bucket, sort by start in LDS and flatten each level
// ----------------------------------------------------------------------------

// n items by the group, the loads of four rounds issued together.
template <int THREADS, class Load, class Put>
__device__ __forceinline__ void group_copy(int n, Load load, Put put) {
  constexpr int U = 4;
  for (int i0 = group_thread<THREADS>(); i0 < n; i0 += U * THREADS) {
    decltype(load(0)) x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = load(min(i0 + u * THREADS, n - 1));
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i0 + u * THREADS < n) put(i0 + u * THREADS, x[u]);
  }
}

// One group flattens bucket gb: sorted in LDS up to CAP records; beyond, by a
// workgroup's radix sort in global memory. A single wave takes buckets of at
// most CAP records only.
template <int THREADS, int CAP>
__device__ __forceinline__ void merge_bucket(const Plan& p, long long gb, SortSmem<THREADS, CAP>& sm) {
  constexpr int MAXI = CAP / THREADS;
  const int tid = group_thread<THREADS>();
  const BucketRecs br = bucket_recs(p, gb);
  const int seg = p.bucket_seg[gb];
  const long long off = (long long)p.offsets[gb];
  const unsigned long long mx[3] = {p.maxend[gb * 3], p.maxend[gb * 3 + 1], p.maxend[gb * 3 + 2]};
  FlatState st;
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    st.M[l] = p.carry[gb * 3 + l];
    st.P[l] = 0;
    st.R[l] = 0;
  }
  const SegDesc sd = p.segs[seg];
  const Geom g = seg_geom(p, seg);
  const long long bl = gb - sd.bucket_begin;
  // a slot overflow makes the host redo the build: write an empty bucket
  const long long n = br.overflow ? 0 : (long long)br.n8 + br.n16;
  const int nlev = sd.n_levels;
  Comp* comp[3] = {p.comp[0] + off, p.comp[1] + off, p.comp[2] + off};
  CompN* compn_b[3] = {p.compn[0] + off, p.compn[1] + off, p.compn[2] + off};
  // 16 B records of a narrow segment lie outside its sampled range: 16 B components
  CompN* const* compn = seg_narrow(g) && br.n16 == 0 ? compn_b : nullptr;
  if (n > 0) {
    const long long lo = bucket_from(g, bl);
    const long long first = bl == 0 ? min(lo, (long long)p.stats[seg].min_s) : lo;  // at or before every start
    if (n <= CAP) {
      const int ni = (int)n;
      group_copy<THREADS>(br.n8, [&](int i) { return br.narrow[i]; },
                          [&](int i, uint2 x) { sm.E[i] = widen(x, lo, mx); });
      group_copy<THREADS>(br.n16, [&](int i) { return br.wide[i]; }, [&](int i, Elem x) { sm.E[br.n8 + i] = x; });
      group_sync<THREADS>();
      const unsigned short* ord = sort_lds<THREADS, CAP>(sm, ni, first);
      if (nlev == 2) flatten_tile<THREADS, MAXI, 2>(sm.E, ord, ni, comp, compn, lo, st, sm.lds_scan);
      else flatten_tile<THREADS, MAXI, 3>(sm.E, ord, ni, comp, compn, lo, st, sm.lds_scan);
    } else if constexpr (THREADS >= 256) {
      // oversized bucket (exact offsets only): every record in the 16 B form
      // into the scratch copy, a stable LSD sort between it and the bucket's
      // own region (16 B per record), then flatten CAP records at a time,
      // carrying the running state across tiles
      Elem* a = p.elems2 + off;
      for (long long i = tid; i < br.n8; i += THREADS) a[i] = widen(br.narrow[i], lo, mx);
      for (long long i = tid; i < br.n16; i += THREADS) a[br.n8 + i] = br.wide[i];
      __threadfence_block();
      __syncthreads();
      const Elem* src = sort_global<THREADS, CAP>(sm, a, p.elems + off, n, lo);
      for (long long t0 = 0; t0 < n; t0 += CAP) {
        const int cnt = (int)min((long long)CAP, n - t0);
        for (int i = tid; i < cnt; i += THREADS) sm.E[i] = src[t0 + i];
        __syncthreads();
        if (nlev == 2) flatten_tile<THREADS, MAXI, 2>(sm.E, nullptr, cnt, comp, compn, lo, st, sm.lds_scan);
        else flatten_tile<THREADS, MAXI, 3>(sm.E, nullptr, cnt, comp, compn, lo, st, sm.lds_scan);
        __syncthreads();
      }
    }
  }
  if (tid == 0) {
#pragma unroll
    for (int l = 0; l < 3; ++l) {
      p.bsum[gb * 3 + l] = st.P[l];
      p.ncomp[gb * 3 + l] = (unsigned int)st.R[l] | (seg_narrow(g) && br.n16 ? kFarComps : 0u);
    }
  }
  group_sync<THREADS>();
}

// The buckets of list set `set` (kQueues lists taken as one): workgroup b takes
// every gridDim.x-th from the b-th on.
struct QueueView {
  const unsigned int* queue;
  long long cap;
  unsigned int len, first, total;  // per lane < kQueues: a list's length, and its first place among all
  __device__ __forceinline__ long long at(unsigned int idx) const {
    // the last list that starts at or before idx and is not empty
    const int q = 63 - __clzll((long long)__ballot(len > 0 && first <= idx));
    return (long long)queue[q * cap + (idx - (unsigned int)__builtin_amdgcn_readlane((int)first, q))];
  }
};
__device__ __forceinline__ QueueView queue_view(const Plan& p, int set) {
  QueueView v;
  const int lane = threadIdx.x & 63;
  v.queue = p.queue + (long long)set * kQueues * p.queue_cap;
  v.cap = p.queue_cap;
  v.len = lane < kQueues ? __hip_atomic_load(&p.qlen[(set * kQueues + lane) * kQueuePad], __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT)
                         : 0u;
  v.first = wave_excl_scan_u32<OpSumU>(v.len, 0u, v.total);
  return v;
}

// Appends bucket gb (one lane calls) to its list of list set `set`.
__device__ __forceinline__ void queue_push(const Plan& p, int set, long long gb) {
  const long long l = set * kQueues + ((gb >> 2) & (kQueues - 1));
  p.queue[l * p.queue_cap + atomicAdd(&p.qlen[l * kQueuePad], 1u)] = (unsigned int)gb;
}

// Wave path: each wave sorts and flattens one bucket of at most kWaveCap
// records with no workgroup barrier, in 32-bit arithmetic relative to the
// bucket's first time `lo`. It takes the buckets whose records are all in the
// scatter's 8 B form:
//   key = (start - lo) << 2 | slot    (start - lo < 2^30: bucket width <= 2^30)
//   end = end - lo + 1                (< 2^32; 0 stands for "before the bucket")
// Comparisons, maxima and measure differences are unchanged by the common
// shift, and the union measure of one bucket's records stays below 2^32, so
// every quantity of the flatten fits 32 bits. The sort is a counting sort on
// the top bits of the start into 128-512 sub-bins (about one per record), writing keys and ends to
// their sorted places in LDS, then an insertion sort inside each sub-bin that
// received two or more records (equal starts may end in any order: the merged
// result does not depend on it). Other buckets (more records, any record in
// the 16 B form, a crowded sub-bin) go to k_merge_rest's lists.

// N consecutive LDS words from a position that is a multiple of N: 16-byte
// reads when N is a multiple of 4, 8-byte reads when it is even, else words
template <int N>
__device__ __forceinline__ void lds_load(const unsigned int* src, unsigned int (&dst)[N]) {
  if constexpr (N % 2 == 1) {
#pragma unroll
    for (int j = 0; j < N; ++j) dst[j] = src[j];
  } else if constexpr (N % 4 == 2) {
#pragma unroll
    for (int j = 0; j < N; j += 2) {
      const uint2 v = *(const uint2*)(src + j);
      dst[j] = v.x;
      dst[j + 1] = v.y;
    }
  } else {
#pragma unroll
    for (int j = 0; j < N; j += 4) {
      const uint4 v = *(const uint4*)(src + j);
      dst[j] = v.x;
      dst[j + 1] = v.y;
      dst[j + 2] = v.z;
      dst[j + 3] = v.w;
    }
  }
}

template <int N>
__device__ __forceinline__ void lds_store(unsigned int* dst, const unsigned int (&src)[N]) {
  if constexpr (N == 4) {
    *(uint4*)dst = make_uint4(src[0], src[1], src[2], src[3]);
  } else if constexpr (N == 2) {
    *(uint2*)dst = make_uint2(src[0], src[1]);
  } else {
#pragma unroll
    for (int j = 0; j < N; ++j) dst[j] = src[j];
  }
}

// Flatten of one sorted bucket by one wave: lane owns sorted positions
// [lane*IPL, lane*IPL + IPL), kept in registers through the three phases
// (running max of ends, measures and break counts, component writes). A
// record outside level l takes part as the empty pair (0, 0), which changes
// no maximum, measure or break, so the phases need no branches; only the
// component stores are conditional. A position past the bucket holds the key
// 2 (rank 2, start lo) with end 0: outside every lower level, and in the top
// level the pair (1, 0), which also changes nothing there, because position 0
// holds a record whose end is at least 1 and comes first in the sweep.
template <int IPL, int NLEV>
__device__ __forceinline__ void wave_flatten(const Plan& p, WaveSmem& W, long long gb, long long off, int ni,
                                             long long lo, const long long (&carry)[3],
                                             const long long (&maxe)[3]) {
  const int lane = threadIdx.x & 63;
  const int q0 = lane * IPL;
  // positions past the bucket already hold the padding pair (key 2, end 0)
  unsigned int kv[IPL], ev[IPL];
  lds_load<IPL>(W.key + q0, kv);
  lds_load<IPL>(W.end + q0, ev);
  // start - lo + 1, the same shift as the ends (recomputed at each use: fewer
  // live registers than keeping it)
  auto sv = [&](int j) { return (kv[j] >> 2) + 1u; };
  // the top level holds every record; the ones below only ranks <= l (ranks
  // are 0..2, so rank <= 1 is rank != 2: both tests share one mask of the key)
  auto in_level = [&](int j, int l) {
    return l == NLEV - 1 || (l == 0 ? (kv[j] & 3u) == 0u : (kv[j] & 3u) != 2u);
  };
  auto s_in = [&](int j, int l) { return in_level(j, l) ? sv(j) : 0u; };
  auto e_in = [&](int j, int l) { return in_level(j, l) ? ev[j] : 0u; };
  // the largest end before each lane: earlier lanes, else the earlier buckets
  unsigned int M[NLEV];
#pragma unroll
  for (int l = 0; l < NLEV; ++l) {
    unsigned int tmax = 0;
#pragma unroll
    for (int j = 0; j < IPL; ++j) tmax = max(tmax, e_in(j, l));
    unsigned int tot;
    const unsigned int ex = wave_excl_scan_u32<OpMaxU>(tmax, 0u, tot);
    // carry - lo + 1 clamped to [0, 2^32 - 1], in wave-uniform 32-bit halves
    const long long d = carry[l] - lo;
    const int dh = (int)(d >> 32);
    const unsigned int dl = (unsigned int)d;
    const unsigned int cr = dh < 0 ? 0u : (dh > 0 || dl == 0xFFFFFFFFu ? 0xFFFFFFFFu : dl + 1u);
    M[l] = max(ex, cr);
  }
  // per-lane measure per level; break counts packed in 10-bit fields (<= 512 each)
  unsigned int acc[NLEV];
  unsigned int nbrk = 0;
#pragma unroll
  for (int l = 0; l < NLEV; ++l) {
    unsigned int Mb = M[l], a = 0, c = 0;
#pragma unroll
    for (int j = 0; j < IPL; ++j) {
      const unsigned int s = s_in(j, l), e = e_in(j, l);
      const unsigned int b = max(s, Mb);
      a += max(e, b) - b;
      c += s > Mb ? 1u : 0u;
      Mb = max(Mb, e);
    }
    acc[l] = a;
    nbrk |= c << (10 * l);
  }
  if constexpr (IPL == 8) {
    // opaque to the compiler: it recomputes the per-level selections of each
    // phase instead of keeping them all live (which spills at 64 VGPRs)
#pragma unroll
    for (int j = 0; j < IPL; ++j) asm volatile("" : "+v"(kv[j]), "+v"(ev[j]));
  }
  unsigned int P[NLEV], totp[NLEV];
#pragma unroll
  for (int l = 0; l < NLEV; ++l) P[l] = wave_excl_scan_u32<OpSumU>(acc[l], 0u, totp[l]);
  unsigned int totr;
  const unsigned int Rp = wave_excl_scan_u32<OpSumU>(nbrk, 0u, totr);
  // components of one level at a time are staged in LDS (the sorted keys and
  // ends are in registers by now) and then written out in full 64-lane rows
  if constexpr (IPL == 8) {
    // opaque to the compiler: it recomputes the per-level selections of each
    // phase instead of keeping them all live (which spills at 64 VGPRs)
#pragma unroll
    for (int j = 0; j < IPL; ++j) asm volatile("" : "+v"(kv[j]), "+v"(ev[j]));
  }
  uint2* stage = (uint2*)W.key;  // key[] and end[]: kWaveCap entries of 8 B
  wave_sync();
#pragma unroll
  for (int l = 0; l < NLEV; ++l) {
    unsigned int r = (Rp >> (10 * l)) & 0x3FFu;
    unsigned int Ml = M[l], Pl = P[l];
#pragma unroll
    for (int j = 0; j < IPL; ++j) {
      const unsigned int s = s_in(j, l), e = e_in(j, l);
      const bool brk = s > Ml;
      if (brk) stage[r] = make_uint2(kv[j] >> 2, Pl);  // CompN {start - lo, measure before}
      r += brk ? 1u : 0u;
      const unsigned int b = max(s, Ml);
      Pl += max(e, b) - b;
      Ml = max(Ml, e);
    }
    wave_sync();
    const int nl = (int)((totr >> (10 * l)) & 0x3FFu);
    uint2* out = (uint2*)(p.compn[l] + off);
    // non-temporal, like the bucketed records: the components (1.2 GB on the
    // large trace) would otherwise sit dirty in L2 and be written back while
    // the next kernels stream their own data
    for (int i = lane; i < nl; i += 64) {
      const uint2 c = stage[i];
      put_rec8(out + i, c.x, c.y);
    }
    wave_sync();
  }
  if (lane < 3) {
    long long bs = 0;
#pragma unroll
    for (int l = 0; l < NLEV; ++l) {
      if (lane == l) {
        bs = (long long)totp[l];
        // ends clamped to lo + 2^32 - 2: the level's union also covers up to
        // its largest true end, beyond what earlier buckets already covered
        const long long from = max(carry[l], lo + 0xFFFFFFFEll);
        if (maxe[l] > from) bs += maxe[l] - from;
      }
    }
    p.bsum[gb * 3 + lane] = bs;
    p.ncomp[gb * 3 + lane] = (totr >> (10 * lane)) & 0x3FFu;
  }
}

// Records of the first rounds that the wave path loads before it knows the
// bucket's count (fixed slots only).
constexpr int kWavePre = 4;

// The most records of a sub-bin that the wave path's insertion sort takes. A
// bucket with more in one (starts in a few places, as where phases of work lie
// between idle stretches) is handed over, and sorted with a second count
// (wave_split) by a wave of k_merge_rest. The split is not made in the wave
// kernel: its registers and code cost every bucket (large trace: 640 us for the
// merge instead of 508, 600 with the split in a called function). The line at
// 16: a trace of 32 + 32 resources in phases of 20 ms every 330 ms (4e6 records)
// takes 24 + 73 us in the two kernels at 8, 49 + 70 at 16, 83 + 48 at 24, and
// took 110 + 141 with sub-bins of up to 32 sorted by insertion and the others
// by the block path; but at 8, and on some traces at 12, a few buckets of evenly
// spread records go the long way too, and one such bucket costs the build 12 us
// (small trace at 8: 3.4 -> 8.9 us for k_merge_rest).
constexpr int kWaveFix = 16, kWaveFixSplit = 32;

// Whether the c keys from `ko` on have one start. Equal starts may stay as they
// are, however many: those of a coarse clock crowd their sub-bins, and need no
// sort.
__device__ __forceinline__ bool equal_starts(const unsigned int* ko, int c) {
  const unsigned int k0 = ko[0];
  for (int a = 1; a < c; a += 4) {
    unsigned int d = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) d |= ko[min(a + u, c - 1)] ^ k0;
    if (d >> 2) return false;
  }
  return true;
}

// The second count: each sub-bin is split into as many parts as it holds
// records, and the records' places come from counting the parts' starts up.
// W.bins holds the sub-bins' starts, kr and er the records; leaves W.key and
// W.end sorted, or returns true in a lane that found a part of more than
// kWaveFixSplit records.
template <int IPL, int NBINS>
__device__ __forceinline__ bool wave_split(WaveSmem& W, int ni, int ksh, const unsigned int (&kr)[IPL],
                                            const unsigned int (&er)[IPL]) {
  constexpr int wpl = NBINS >> 7;
  const int lane = threadIdx.x & 63;
  auto half = [&](unsigned int d) { return (W.bins[d >> 1] >> (16u * (d & 1u))) & 0xFFFFu; };
  unsigned int part[IPL];
#pragma unroll
  for (int r = 0; r < IPL; ++r) {
    const unsigned int d = kr[r] >> ksh, st = half(d);
    const unsigned int stop = (int)d + 1 < NBINS ? half(d + 1) : (unsigned int)ni;
    part[r] = st + __umulhi(kr[r] << (32 - ksh), stop - st);  // below ni <= NBINS; past the bucket: not used
  }
  wave_sync();
  unsigned int bw[wpl];
#pragma unroll
  for (int j = 0; j < wpl; ++j) bw[j] = 0;
  lds_store<wpl>(W.bins + lane * wpl, bw);
  wave_sync();
#pragma unroll
  for (int r = 0; r < IPL; ++r)
    if (lane + 64 * r < ni) atomicAdd(&W.bins[part[r] >> 1], 1u << (16u * (part[r] & 1u)));
  wave_sync();
  lds_load<wpl>(W.bins + lane * wpl, bw);
  unsigned int tot = 0, all;
#pragma unroll
  for (int j = 0; j < wpl; ++j) tot += (bw[j] & 0xFFFFu) + (bw[j] >> 16);
  unsigned int run = wave_excl_scan_u32<OpSumU>(tot, 0u, all);
#pragma unroll
  for (int j = 0; j < wpl; ++j) {
    const unsigned int a = run, b = run + (bw[j] & 0xFFFFu);
    run = b + (bw[j] >> 16);
    bw[j] = a | (b << 16);
  }
  lds_store<wpl>(W.bins + lane * wpl, bw);
  wave_sync();
#pragma unroll
  for (int r = 0; r < IPL; ++r) {
    // a position past the bucket stores to its own index
    unsigned int q = (unsigned int)(lane + 64 * r);
    if ((int)q < ni) {
      const unsigned int sh = 16u * (part[r] & 1u);
      q = (atomicAdd(&W.bins[part[r] >> 1], 1u << sh) >> sh) & 0xFFFFu;
    }
    W.key[q] = kr[r];
    W.end[q] = er[r];
  }
  wave_sync();
  // the parts' starts have become their stops: order inside each part
  bool crowded = false;
  for (int d = lane; d < ni; d += 64) {
    const int st = d ? (int)half((unsigned int)d - 1u) : 0, c = (int)half((unsigned int)d) - st;
    if (c < 2) continue;
    unsigned int* ko = W.key + st;
    unsigned int* eo = W.end + st;
    if (c > kWaveFixSplit) {
      crowded |= !equal_starts(ko, c);
      continue;
    }
    for (int a = 1; a < c; ++a) {
      const unsigned int kx = ko[a], ex = eo[a];
      int b = a - 1;
      while (b >= 0 && ko[b] > kx) {
        ko[b + 1] = ko[b];
        eo[b + 1] = eo[b];
        --b;
      }
      ko[b + 1] = kx;
      eo[b + 1] = ex;
    }
  }
  return crowded;
}

// W.key[0, ni) and W.end with it in order by a bitonic network, where starts
// crowd even in the parts. On the records themselves, in 32 bits: handing the
// bucket on to the 64-bit sort, which goes through indices, took 16 resources of
// 60,000 records in bursts of 24 within a microsecond 205 us to rebuild, 153 so.
__device__ __forceinline__ void wave_bitonic(WaveSmem& W, int ni) {
  const int lane = threadIdx.x & 63;
  int size = 2;
  while (size < ni) size <<= 1;
  for (int i = ni + lane; i < size; i += 64) W.key[i] = 0xFFFFFFFFu;  // above every key (kinds are 0 to 2)
  wave_sync();
  for (int k = 2; k <= size; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int i = lane; i < size / 2; i += 64) {
        const int a = ((i & ~(j - 1)) << 1) | (i & (j - 1)), b = a | j;
        const unsigned int x = W.key[a], y = W.key[b];
        if ((x > y) == ((a & k) == 0)) {
          const unsigned int ex = W.end[a], ey = W.end[b];
          W.key[a] = y;
          W.key[b] = x;
          W.end[a] = ey;
          W.end[b] = ex;
        }
      }
      wave_sync();
    }
  }
  for (int i = ni + lane; i < size; i += 64) {  // the flatten's padding pair again
    W.key[i] = 2u;
    W.end[i] = 0u;
  }
  wave_sync();
}

// Sort of one bucket of 64*(IPL-1) < ni <= 64*IPL records into W, then its
// flatten: every round but the last is full, so only the last one tests for
// positions past the bucket. With fixed slots (kSlots) the first kWavePre
// rounds come loaded in `pre` (read before the count was known, so past the
// end of a bucket of fewer records: places its slots hold). kSplit: with the
// second count, and any ni <= 64*IPL; always done. Else returns false (nothing
// written) when the bucket must be handed over.
template <int IPL, bool kSlots, bool kSplit = false>
__device__ __forceinline__ bool wave_bucket(const Plan& p, WaveSmem& W, long long gb, long long off, int ni,
                                            const uint2* rec, const uint2 (&pre)[kWavePre], long long lo, int nlev,
                                            const long long (&carry)[3], const long long (&maxe)[3]) {
  const int lane = threadIdx.x & 63;
  // round r holds position lane + 64 r; rounds before the last are inside the bucket
  auto in_bucket = [&](int r) { return (!kSplit && r < IPL - 1) || lane + 64 * r < ni; };
  unsigned int kr[IPL], er[IPL], rk[IPL];
  // every lane loads every round, from a position clamped into the bucket
  // (ni >= 1): the loads issue back to back instead of one masked block (and
  // one wait) each
  uint2 x[IPL];
#pragma unroll
  for (int r = 0; r < IPL; ++r) {
    if (kSlots && r < kWavePre) {
      x[r] = pre[r];
      continue;
    }
    // a 32-bit byte offset from the wave-uniform base (ni <= kWaveCap); the
    // last round clamps into the bucket, so it reads no lines past its end
    const unsigned int i = (unsigned int)(!kSplit && r < IPL - 1 ? lane + 64 * r : min(lane + 64 * r, ni - 1));
    x[r] = *(const uint2*)((const char*)rec + 8u * i);  // relative to lo: (start - lo) << 2 | slot, end - lo + 1
  }
  // a position past the bucket keeps the padding pair of the flatten: key 2
  // (rank 2, start lo), end 0; it is stored at its own index below
  unsigned int kor = 0;
#pragma unroll
  for (int r = 0; r < IPL; ++r) {
    const bool in = in_bucket(r);
    kr[r] = in ? x[r].x : 2u;
    er[r] = in ? x[r].y : 0u;
    kor |= kr[r];
  }
  kor >>= 2;
  kor = (unsigned int)wave_reduce_i32<OpOrI>((int)kor, 0);
  // sub-bins: about one per record (128 up to 128 records, 256 up to 256,
  // else 512: the round count fixes the range of ni); a lane owns 2*wpl of
  // them, two per LDS word
  constexpr int dbits = IPL <= 2 ? 7 : (IPL <= 4 ? 8 : 9);
  constexpr int nbins = 1 << dbits, wpl = nbins >> 7;
  unsigned int bw[wpl];
#pragma unroll
  for (int j = 0; j < wpl; ++j) bw[j] = 0;
  lds_store<wpl>(W.bins + lane * wpl, bw);
  wave_sync();
  const int hb = kor ? 32 - __clz((int)kor) : 0;
  const int ksh = 2 + (hb > dbits ? hb - dbits : 0);  // sub-bin = key >> ksh (ksh <= 25)
  // the atomics of all rounds are issued with no branch, so they overlap
  // instead of waiting one by one; a position past the bucket adds 0 to a
  // word of its own (word `lane`: there are at least 64), so lanes past the
  // bucket never pile onto one address
  // (sub-bin d = key >> ksh counts in half d & 1 of word d >> 1)
#pragma unroll
  for (int r = 0; r < IPL; ++r) {
    const bool in = in_bucket(r);
    const unsigned int w = in ? kr[r] >> (ksh + 1) : (unsigned int)lane;
    const unsigned int sh = in ? ((kr[r] >> ksh) & 1u) << 4 : 0u;
    rk[r] = __builtin_amdgcn_ubfe(atomicAdd(&W.bins[w], in ? 1u << sh : 0u), sh, 16);
  }
  wave_sync();
  // exclusive scan of the sub-bin counters (lane order = sub-bin order)
  lds_load<wpl>(W.bins + lane * wpl, bw);
  unsigned int tot = 0;
#pragma unroll
  for (int j = 0; j < wpl; ++j) tot += (bw[j] & 0xFFFFu) + (bw[j] >> 16);
  unsigned int all;
  unsigned int run = wave_excl_scan_u32<OpSumU>(tot, 0u, all);
#pragma unroll
  for (int j = 0; j < wpl; ++j) {
    const unsigned int a = run, b = run + (bw[j] & 0xFFFFu);
    run = b + (bw[j] >> 16);
    bw[j] = a | (b << 16);
  }
  lds_store<wpl>(W.bins + lane * wpl, bw);
  wave_sync();
  bool crowded = false;
  if constexpr (kSplit) {
    crowded = wave_split<IPL, nbins>(W, ni, ksh, kr, er);
    wave_sync();
    if (__ballot(crowded)) wave_bitonic(W, ni);
    if (nlev == 2) wave_flatten<IPL, 2>(p, W, gb, off, ni, lo, carry, maxe);
    else wave_flatten<IPL, 3>(p, W, gb, off, ni, lo, carry, maxe);
    return true;
  }
  unsigned int fix = 0;  // bit r: the record of round r is the second one of its sub-bin
  constexpr int G = IPL < 4 ? IPL : 4;  // rounds placed together (bounds the live registers)
#pragma unroll
  for (int r0 = 0; r0 < IPL; r0 += G) {
    unsigned int pos[G];
#pragma unroll
    for (int u = 0; u < G; ++u) {  // the reads of a group first (past the bucket: word `lane`)
      if (r0 + u >= IPL) break;  // a last group shorter than G
      const bool in = in_bucket(r0 + u);
      const unsigned int w = in ? kr[r0 + u] >> (ksh + 1) : (unsigned int)lane;
      const unsigned int sh = in ? ((kr[r0 + u] >> ksh) & 1u) << 4 : 0u;
      pos[u] = __builtin_amdgcn_ubfe(W.bins[w], sh, 16) + rk[r0 + u];
    }
#pragma unroll
    for (int u = 0; u < G; ++u) {
      // a position past the bucket stores to its own index (>= ni): never
      // read as a record, and no branch around the stores (distinct addresses)
      const int r = r0 + u;
      if (r >= IPL) break;
      const bool in = in_bucket(r);
      const unsigned int q = in ? pos[u] : (unsigned int)(lane + 64 * r);
      W.key[q] = kr[r];
      W.end[q] = er[r];
      fix |= (in && rk[r] == 1) ? 1u << r : 0u;
    }
  }
  wave_sync();
  // order inside each sub-bin by the full key, where it holds two or more
  // records: an insertion sort per such sub-bin
  auto fix_sub_bin = [&](unsigned int d) {
    const int st0 = (int)((W.bins[d >> 1] >> (16u * (d & 1u))) & 0xFFFFu);
    const int st1 = (int)d + 1 < nbins ? (int)((W.bins[(d + 1) >> 1] >> (16u * ((d + 1) & 1u))) & 0xFFFFu) : ni;
    const int c = st1 - st0;
    unsigned int* ko = W.key + st0;
    unsigned int* eo = W.end + st0;
    if (c > kWaveFix) {
      crowded |= !equal_starts(ko, c);
      return;
    }
    for (int a = 1; a < c; ++a) {
      const unsigned int kx = ko[a], ex = eo[a];
      int b = a - 1;
      while (b >= 0 && ko[b] > kx) {
        ko[b + 1] = ko[b];
        eo[b + 1] = eo[b];
        --b;
      }
      ko[b + 1] = kx;
      eo[b + 1] = ex;
    }
  };
  if (ksh > 2) {
    // the sub-bins to fix (each named by the lane that placed its second
    // record) are listed in the key array past the bucket's records, so the
    // work spreads evenly over the lanes: ceil(fixes / 64) rounds instead of
    // the largest number of fixes of one lane
    unsigned int nfix;
    const unsigned int fb = wave_excl_scan_u32<OpSumU>((unsigned int)__popc(fix), 0u, nfix);
    if (nfix <= 2u * (unsigned int)(kWaveCap - ni)) {  // 16-bit entries in the free words
      unsigned short* list = (unsigned short*)(W.key + ni);
      unsigned int q = fb;
#pragma unroll
      for (int r = 0; r < IPL; ++r) {
        if (fix & (1u << r)) list[q++] = (unsigned short)(kr[r] >> ksh);
      }
      wave_sync();
      for (unsigned int i = (unsigned int)lane; i < nfix; i += 64) fix_sub_bin(list[i]);
      wave_sync();
      // the list's words back to the padding key
      for (unsigned int i = (unsigned int)lane; 2 * i < nfix; i += 64) W.key[ni + i] = 2u;
    } else {
      // no room: each lane walks its own such records
      unsigned int todo = fix;
      while (todo) {
        const int rr = __builtin_ctz(todo);
        todo &= todo - 1u;
        unsigned int kk = kr[0];
#pragma unroll
        for (int j = 1; j < IPL; ++j) kk = rr == j ? kr[j] : kk;  // kr[rr] without indexing registers
        fix_sub_bin(kk >> ksh);
      }
    }
  }
  if (__ballot(crowded)) return false;
  wave_sync();
  if (nlev == 2) wave_flatten<IPL, 2>(p, W, gb, off, ni, lo, carry, maxe);
  else wave_flatten<IPL, 3>(p, W, gb, off, ni, lo, carry, maxe);
  return true;
}

// One bucket of ni records (1 <= ni <= kWaveCap, all in the 8 B form) by one
// wave, with as many records per lane as it needs: every slot costs the same
// instructions, filled or not. False: the bucket must be handed over.
template <bool kSlots>
__device__ __forceinline__ bool wave_merge(const Plan& p, WaveSmem& W, long long gb, long long off, int ni,
                                           const uint2* rec, const uint2 (&pre)[kWavePre], long long lo, int nlev,
                                           const long long (&carry)[3], const long long (&maxe)[3]) {
  if (ni <= 64) return wave_bucket<1, kSlots>(p, W, gb, off, ni, rec, pre, lo, nlev, carry, maxe);
  if (ni <= 128) return wave_bucket<2, kSlots>(p, W, gb, off, ni, rec, pre, lo, nlev, carry, maxe);
  if (ni <= 192) return wave_bucket<3, kSlots>(p, W, gb, off, ni, rec, pre, lo, nlev, carry, maxe);
  if (ni <= 256) return wave_bucket<4, kSlots>(p, W, gb, off, ni, rec, pre, lo, nlev, carry, maxe);
  if (ni <= 320) return wave_bucket<5, kSlots>(p, W, gb, off, ni, rec, pre, lo, nlev, carry, maxe);
  if (ni <= 384) return wave_bucket<6, kSlots>(p, W, gb, off, ni, rec, pre, lo, nlev, carry, maxe);
  if (ni <= 448) return wave_bucket<7, kSlots>(p, W, gb, off, ni, rec, pre, lo, nlev, carry, maxe);
  return wave_bucket<8, kSlots>(p, W, gb, off, ni, rec, pre, lo, nlev, carry, maxe);
}

// One wave per bucket, 8 waves per SIMD (64 VGPRs). Buckets that need the
// k_merge_rest go to its lists. kSlots: fixed slots of at least 128 records
// (2 slot_cap record places per bucket, whatever its count).
template <bool kSlots>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_merge_wave(Plan p) {
  __shared__ WaveSmem wsm[4];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // everything per bucket is wave-uniform
  const long long gb = (long long)blockIdx.x * 4 + wave;
  if (gb >= p.n_buckets) return;
  WaveSmem& W = wsm[wave];
  uint2 pre[kWavePre];
  if constexpr (kSlots) {
    // the first rounds load while the bucket's count is still on its way:
    // its slots start at a known place and hold 2 slot_cap >= 256 records
    const uint2* base = (const uint2*)p.elems + 2 * gb * (long long)p.slot_cap;
#pragma unroll
    for (int r = 0; r < kWavePre; ++r) pre[r] = base[lane + 64 * r];
  }
  // every per-bucket word is read here, before any of them is used, so the
  // reads travel together (only the segment's words wait for its index)
  BucketRecs br;
  if constexpr (kSlots) {
    // fixed slots (slot_cap > 0): the places need no other word
    const unsigned long long cu = p.cursor[gb];
    br.n8 = (int)(unsigned int)cu;
    br.n16 = (int)(cu >> 32);
    br.overflow = (long long)br.n8 + br.n16 > (long long)p.slot_cap;
    br.narrow = (const uint2*)p.elems + 2 * gb * (long long)p.slot_cap;
    br.wide = nullptr;  // never read here: such buckets are handed over
  } else {
    br = bucket_recs(p, gb);
  }
  const long long off = (long long)p.offsets[gb];
  const long long carry[3] = {p.carry[gb * 3], p.carry[gb * 3 + 1], p.carry[gb * 3 + 2]};
  const unsigned long long mx[3] = {p.maxend[gb * 3], p.maxend[gb * 3 + 1], p.maxend[gb * 3 + 2]};
  const int seg = p.bucket_seg[gb];
  const SegDesc sd = p.segs[seg];
  const Geom g = seg_geom(p, seg);
  const long long n = (long long)br.n8 + br.n16;
  // largest end per level of the bucket's own records (0: none)
  long long maxe[3];
  maxe[0] = (long long)mx[0];
  maxe[1] = max(maxe[0], (long long)mx[1]);
  maxe[2] = max(maxe[1], (long long)mx[2]);
  if (n == 0 || br.overflow) {
    // empty, or a slot overflow that makes the host redo the build
    // a use of the early loads on this path too, so that the compiler issues
    // them before the count's test instead of moving them below it
    if constexpr (kSlots) asm volatile("" ::"v"(pre[0].x), "v"(pre[1].x), "v"(pre[2].x), "v"(pre[3].x));
    asm volatile("" ::"s"(off), "s"(carry[0]), "s"(carry[1]), "s"(carry[2]), "s"(mx[0]), "s"(mx[1]), "s"(mx[2]),
                 "s"(sd.bucket_begin), "s"(sd.n_levels), "s"(g.min_s), "s"(g.wx), "s"(g.s0));
    if (lane < 3) {
      p.bsum[gb * 3 + lane] = 0;
      p.ncomp[gb * 3 + lane] = 0;
    }
    return;
  }
  bool done = false;
  if (br.n16 == 0 && n <= kWaveCap)  // only 8 B records (so the segment is narrow: buckets at most 2^30 ns wide)
    done = wave_merge<kSlots>(p, W, gb, off, (int)n, br.narrow, pre, bucket_lo(g, gb - sd.bucket_begin), sd.n_levels,
                              carry, maxe);
  if (!done && lane == 0) queue_push(p, n <= kWaveCap ? 0 : 1, gb);
}

// The buckets the wave path handed over. Those of more than kWaveCap records
// take a workgroup each. The others take a wave each: 8 B records with crowded
// sub-bins the wave path's code with its second count, 16 B records (64-bit
// keys) the workgroup's code. Waves count from the last
// workgroup down, so those without a large bucket take the small ones first.
// A build of 2.9e3 wide buckets (16 + 16 resources, 1e6 records over hours):
// 131 us with a workgroup per bucket and a radix sort, 57 with the counting
// sort, 38 so (27 with 352 records per bucket, 320 now). A few buckets take 17 us,
// which is one bucket's chain of dependent reads, barriers and scans.
template <int THREADS, int CAP>
__global__ __launch_bounds__(THREADS, CAP == 2048 ? 3 : 1) void k_merge_rest(Plan p) {
  constexpr int NW = THREADS / 64;
  __shared__ RestSmem<THREADS, CAP> u;
  {
    const QueueView v = queue_view(p, 1);
    for (unsigned int idx = blockIdx.x; idx < v.total; idx += gridDim.x) merge_bucket<THREADS, CAP>(p, v.at(idx), u.block);
  }
  const QueueView v = queue_view(p, 0);
  const int wave = group_wave<THREADS>();
  for (unsigned int idx = (gridDim.x - 1 - blockIdx.x) * NW + wave; idx < v.total; idx += gridDim.x * NW) {
    const long long gb = v.at(idx);
    const BucketRecs br = bucket_recs(p, gb);
    if (br.n16 == 0) {
      const int seg = p.bucket_seg[gb];
      const long long off = (long long)p.offsets[gb];
      long long carry[3], maxe[3];
#pragma unroll
      for (int l = 0; l < 3; ++l) {
        carry[l] = p.carry[gb * 3 + l];
        maxe[l] = (long long)p.maxend[gb * 3 + l];
      }
      maxe[1] = max(maxe[0], maxe[1]);
      maxe[2] = max(maxe[1], maxe[2]);
      const SegDesc sd = p.segs[seg];
      const long long lo = bucket_lo(seg_geom(p, seg), gb - sd.bucket_begin);
      const uint2 pre[kWavePre] = {};
      (void)wave_bucket<8, false, true>(p, u.wave[wave].w, gb, off, br.n8, br.narrow, pre, lo, sd.n_levels, carry, maxe);
      wave_sync();
    } else {
      merge_bucket<64, kWaveCap>(p, gb, u.wave[wave].one);
    }
  }
}

// ----------------------------------------------------------------------------
// small builds: a workgroup per segment does every step of the build
// ----------------------------------------------------------------------------

// When every segment is small, the passes above are ten launches of a few
// microseconds of latency each, with most of the GPU idle. Here one workgroup
// takes one segment through all of them, with barriers in place of launches:
// start range, geometry, scatter into the fixed slots (ranks, largest ends and
// counts in LDS), carry and offsets, the wave merges of its buckets, the block
// path for those that need it, and the base pass. It leaves the same
// per-bucket words and records as the passes. A slot overflow is reported
// like theirs, and the host redoes the build with exact offsets.
//
// The line lies at 4096 records per segment (kSmallRecords): up to there a
// thread keeps its eight records in registers between the start range and the
// scatter, and a build takes 16-35 us where the passes take 49 (a session of
// 4 resources, 1.8e3 records, with its upload and regions: 96 -> 54 us). One
// CU per segment runs out of VALU beyond: with 1e4 records per segment 51 us
// against 49, with 3e4 105 against 64. 512 threads: two workgroups per CU.
constexpr int kSmallThreads = 512;
constexpr int kSmallSort = 4;  // waves that sort buckets with 64-bit keys (their LDS: 10 KB each)

struct SmallSmem {
  union {
    WaveSmem w[kSmallThreads / 64];
    SortSmem<kSmallThreads, 2048> sort;
    SortSmem<64, kWaveCap> one[kSmallSort];
  } u;
  unsigned long long cnt[kSmallBuckets];  // 8 B records | 16 B records << 32
  unsigned long long maxe[kSmallBuckets * 3];
  long long carry[kSmallBuckets * 3];
  unsigned int off[kSmallBuckets];        // merged-interval offset within the segment
  unsigned int queue[kSmallBuckets];      // buckets the wave merges left
  unsigned int nq;
  const int64_t* s[kSmallChunks];
  const int64_t* e[kSmallChunks];
  int first[kSmallChunks];      // segment's record index of the chunk's first record
  int slot[kSmallChunks];
  long long red[2][kSmallThreads / 64];
  SegStats st;
  Geom g;
};

__global__ __launch_bounds__(kSmallThreads, 4) void k_build_small(Plan p) {
  constexpr int THREADS = kSmallThreads, K = kSmallRecords / THREADS, NW = THREADS / 64;
  __shared__ SmallSmem S;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int seg = blockIdx.x;
  const SegDesc sd = p.segs[seg];
  const SmallSeg ss = p.sseg[seg];
  const int nb = sd.nb, nch = ss.n_chunks, N = ss.count;
  for (int j = threadIdx.x; j < nch; j += THREADS) {
    const ChunkDesc cd = p.chunks[ss.chunk0 + j];
    S.s[j] = cd.s;
    S.e[j] = cd.e;
    S.first[j] = cd.tile_off;
    S.slot[j] = cd.slot;
  }
  for (int b = threadIdx.x; b < nb; b += THREADS) {
    S.cnt[b] = 0;
    S.maxe[3 * b] = S.maxe[3 * b + 1] = S.maxe[3 * b + 2] = 0;
  }
  if (threadIdx.x == 0) {
    S.nq = 0;
    if (blockIdx.x == 0 && p.ts) p.ts[kTsBuild] = __builtin_amdgcn_s_memrealtime();
  }
  __syncthreads();
  // a thread's K records: their chunks (the largest j with first[j] <= x),
  // then all loads back to back, from positions clamped into the segment
  long long sv[K], ev[K];
  int jj[K];
  long long mn = LLONG_MAX, mx = -1;  // start range (starts outside [0, 2^62) belong to invalid records)
  if (N > 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int x = min((int)threadIdx.x + k * THREADS, N - 1);
      int lo = 0, hi = nch - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (S.first[mid] <= x) lo = mid; else hi = mid - 1;
      }
      jj[k] = lo;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = min((int)threadIdx.x + k * THREADS, N - 1) - S.first[jj[k]];
      sv[k] = S.s[jj[k]][i];
      ev[k] = S.e[jj[k]][i];
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if ((unsigned long long)sv[k] < (unsigned long long)kTimeLimit) {
        mn = min(mn, sv[k]);
        mx = max(mx, sv[k]);
      }
    }
  }
  mn = -wave_reduce_i64<OpMax>(-mn, -LLONG_MAX);
  mx = wave_reduce_i64<OpMax>(mx, -1);
  if (lane == 0) {
    S.red[0][wave] = mn;
    S.red[1][wave] = mx;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < NW; ++w) {
      mn = min(mn, S.red[0][w]);
      mx = max(mx, S.red[1][w]);
    }
    SegStats st;
    st.min_s = mx < 0 ? ULLONG_MAX : (unsigned long long)mn;
    st.max_s = mx < 0 ? 0ull : (unsigned long long)mx;
    st.max_e = 0;
    st.far_e = 0;
    S.st = st;
    S.g = make_geom(st, sd);
  }
  __syncthreads();
  const Geom g = S.g;
  const bool narrow = seg_narrow(g);
  const long long scap = p.slot_cap;
  // scatter: lanes of one bucket and kind share one LDS atomic; the leader
  // reserves their ranks and folds their largest end in
  uint2* units = (uint2*)p.elems + 2 * sd.bucket_begin * scap;  // the segment's slots: 2 scap units per bucket
  const unsigned long long lt = (1ull << lane) - 1ull;
  {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int x = (int)threadIdx.x + k * THREADS;
      if ((wave << 6) + k * THREADS >= N) break;  // wave-uniform
      int key = -1;  // bucket << 2 | kind slot
      unsigned int kx = 0, ex = 0;
      if (x < N) {
        if (!rec_valid(sv[k], ev[k])) {
          // first bad record of the build: chunk << 40 | index (rare path)
          const ChunkDesc& cd = p.chunks[ss.chunk0 + jj[k]];
          atomicMin(p.err, ((unsigned long long)cd.chunk_id << 40) | (unsigned long long)(x - S.first[jj[k]]));
          p.owner_err[cd.owner] = 1u;
        } else if (sv[k] < ev[k]) {
          const int b = bucket_of(sv[k], g), slot = S.slot[jj[k]];
          const long long lo = bucket_lo(g, b);
          key = b << 2 | slot;
          kx = ((unsigned int)(sv[k] - lo) << 2) | (unsigned int)slot;
          ex = ev[k] - lo < 0xFFFFFFFFll ? (unsigned int)(ev[k] - lo + 1) : 0xFFFFFFFFu;  // far ends clamped
        }
      }
      unsigned long long todo = __ballot(key >= 0);
      while (todo) {
        const int leader = __ffsll((long long)todo) - 1;
        const int lk = __builtin_amdgcn_readlane(key, leader);
        const bool in = key == lk;
        const unsigned long long m = __ballot(in);
        const int b = lk >> 2;
        long long emax;
        unsigned int e32 = 0xFFFFFFFFu;
        if (narrow) e32 = (unsigned int)wave_reduce_i32<OpMaxU32>((int)(in ? ex : 0u), 0);
        if (e32 != 0xFFFFFFFFu) emax = bucket_lo(g, b) + (long long)e32 - 1;
        else emax = wave_reduce_i64<OpMax>(in ? ev[k] : 0ll, 0ll);
        unsigned long long old = 0;
        if (lane == leader) {
          const unsigned long long n = (unsigned long long)__popcll(m);
          old = atomicAdd(&S.cnt[b], narrow ? n : n << 32);
          atomicMax(&S.maxe[3 * b + (lk & 3)], (unsigned long long)emax);
        }
        old = (unsigned long long)readlane64((long long)old, leader);
        if (in) {
          const long long rank = (long long)(narrow ? (unsigned int)old : (unsigned int)(old >> 32)) + __popcll(m & lt);
          uint2* ub = units + 2 * b * scap;
          if (narrow) {
            if (rank < 2 * scap) ub[rank] = make_uint2(kx, ex);
          } else if (rank < scap) {
            Elem el;
            el.s = sv[k];
            el.e_slot = (long long)((unsigned long long)ev[k] | ((unsigned long long)(lk & 3) << kSlotShift));
            *(Elem*)(ub + 2 * scap - 2 * (rank + 1)) = el;
          }
        }
        todo &= ~m;
      }
    }
  }
  __syncthreads();
  // one wave: offsets of the merged intervals and the running largest end of
  // all earlier buckets per level
  if (wave == 0) {
    const long long init = S.st.min_s > S.st.max_s ? -1 : (long long)S.st.min_s - 1;
    long long run[3] = {init, init, init};
    unsigned int roff = 0, over = 0;
    for (int c0 = 0; c0 < nb; c0 += 64) {
      const int b = c0 + lane;
      unsigned int n = 0;
      long long v[3] = {LLONG_MIN, LLONG_MIN, LLONG_MIN};
      if (b < nb) {
        const unsigned long long cu = S.cnt[b];
        n = (unsigned int)cu + (unsigned int)(cu >> 32);
        if (n > (unsigned int)scap) {
          n = (unsigned int)scap;
          over = 1;
        }
        const long long m0 = (long long)S.maxe[3 * b], m1 = (long long)S.maxe[3 * b + 1], m2 = (long long)S.maxe[3 * b + 2];
        v[0] = m0 ? m0 : LLONG_MIN;
        v[1] = m1 > v[0] && m1 ? m1 : v[0];
        v[2] = m2 > v[1] && m2 ? m2 : v[1];
      }
      unsigned int all;
      const unsigned int ex = wave_excl_scan_u32<OpSumU>(n, 0u, all);
      if (b < nb) S.off[b] = roff + ex;
      roff += all;
#pragma unroll
      for (int l = 0; l < 3; ++l) {
        long long top;
        const long long e = wave_excl_scan_dpp<OpMax>(v[l], LLONG_MIN, top);
        if (b < nb) S.carry[3 * b + l] = e > run[l] ? e : run[l];
        run[l] = top > run[l] ? top : run[l];
      }
    }
    if (over) atomicAdd(&p.oversized[1], 1ull);  // slot overflow: the build is redone with exact offsets
    if (lane == 0) {
      SegStats st = S.st;
      st.max_e = (unsigned long long)(run[2] > init ? run[2] : (init + 1 > 0 ? init + 1 : 0));
      p.stats[seg] = st;
      p.geom[seg] = g;
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 3 * nb; i += THREADS) {
    const long long q = sd.bucket_begin * 3 + i;
    p.maxend[q] = S.maxe[i];
    p.carry[q] = S.carry[i];
  }
  for (int b = threadIdx.x; b < nb; b += THREADS) {
    const long long gb = sd.bucket_begin + b;
    const unsigned long long cu = S.cnt[b];
    const unsigned long long n = (cu & 0xFFFFFFFFull) + (cu >> 32);
    p.cursor[gb] = cu;
    p.counts[gb] = (unsigned int)(n < (unsigned long long)scap ? n : (unsigned long long)scap);
    p.offsets[gb] = (unsigned long long)(ss.elem0 + S.off[b]);
    p.bucket_seg[gb] = seg;
  }
  // merge: a wave per bucket
  for (int b = wave; b < nb; b += NW) {
    const long long gb = sd.bucket_begin + b;
    const unsigned long long cu = (unsigned long long)readlane64((long long)S.cnt[b], 0);
    const long long n = (long long)((cu & 0xFFFFFFFFull) + (cu >> 32));
    if (n == 0 || n > scap) {  // empty, or a slot overflow that makes the host redo the build
      if (lane < 3) {
        p.bsum[gb * 3 + lane] = 0;
        p.ncomp[gb * 3 + lane] = 0;
      }
      continue;
    }
    bool done = false;
    if (narrow && n <= kWaveCap) {
      const uint2* rec = units + 2 * b * scap;
      uint2 pre[kWavePre];
#pragma unroll
      for (int r = 0; r < kWavePre; ++r) pre[r] = rec[lane + 64 * r];  // slots hold 2 scap >= 256 units
      long long carry[3], maxe[3];
#pragma unroll
      for (int l = 0; l < 3; ++l) {
        carry[l] = readlane64(S.carry[3 * b + l], 0);
        maxe[l] = readlane64((long long)S.maxe[3 * b + l], 0);
      }
      maxe[1] = max(maxe[0], maxe[1]);
      maxe[2] = max(maxe[1], maxe[2]);
      const long long off = ss.elem0 + (long long)(unsigned int)__builtin_amdgcn_readfirstlane((int)S.off[b]);
      done = wave_merge<true>(p, S.u.w[wave], gb, off, (int)n, rec, pre, bucket_lo(g, b), sd.n_levels, carry, maxe);
      if (!done)
        done = wave_bucket<8, false, true>(p, S.u.w[wave], gb, off, (int)n, rec, pre, bucket_lo(g, b), sd.n_levels,
                                           carry, maxe);
    }
    if (!done && lane == 0) S.queue[atomicAdd(&S.nq, 1u)] = (unsigned int)b;
  }
  __syncthreads();
  // what is left, as k_merge_rest does it: buckets of at most kWaveCap records
  // by a wave each, kSmallSort at a time (a segment of wide buckets has all of
  // its here), then the larger ones by the workgroup
  const unsigned int nq = S.nq;
  if (wave < kSmallSort) {
    for (unsigned int q = wave; q < nq; q += kSmallSort) {
      const unsigned int b = (unsigned int)__builtin_amdgcn_readfirstlane((int)S.queue[q]);
      const unsigned long long cu = (unsigned long long)readlane64((long long)S.cnt[b], 0);
      if ((cu & 0xFFFFFFFFull) + (cu >> 32) <= (unsigned long long)kWaveCap)
        merge_bucket<64, kWaveCap>(p, sd.bucket_begin + b, S.u.one[wave]);
    }
  }
  __syncthreads();
  for (unsigned int q = 0; q < nq; ++q) {
    const unsigned int b = S.queue[q];
    const unsigned long long cu = S.cnt[b];
    if ((cu & 0xFFFFFFFFull) + (cu >> 32) > (unsigned long long)kWaveCap)
      merge_bucket<THREADS, 2048>(p, sd.bucket_begin + b, S.u.sort);
  }
  __syncthreads();
  if (wave == 0) base_segment(p, seg, lane);
}

// ----------------------------------------------------------------------------
// region: clip every resource by binary search, reduce, finalize in FP64
// ----------------------------------------------------------------------------

// Measure of level l of segment seg before time t.
__device__ __forceinline__ long long measure_before(const Plan& p, int seg, int l, long long t) {
  const SegDesc sd = p.segs[seg];
  const Geom g = seg_geom(p, seg);
  const SegStats st = p.stats[seg];
  if (g.empty || t <= (long long)st.min_s) return 0;
  if (t >= (long long)st.max_e) return p.seg_total[seg * 3 + l];
  const long long bl = t <= g.min_s ? 0 : bucket_index(g, (unsigned long long)(t - g.min_s));
  const long long gb = sd.bucket_begin + bl;
  const long long carry = p.carry[gb * 3 + l];
  const long long base = p.base[gb * 3 + l];
  const long long bs = p.bsum[gb * 3 + l];
  const unsigned int nc = p.ncomp[gb * 3 + l];
  const int cnt = (int)(nc & ~kFarComps);
  const long long off = (long long)p.offsets[gb];
  const long long lo = bucket_from(g, bl);
  const long long width = (long long)((unsigned long long)g.wx << g.s0);
  long long cs, pl, next;
  bool any;
  if (seg_narrow(g) && !(nc & kFarComps)) {
    const CompN* c = p.compn[l] + off;
    // past the last bucket's width no component starts: any x there will do
    const unsigned int x = (unsigned int)min(t - lo, 0x7FFFFFFFll);
    unsigned int c32;
    any = find_comp(
        [&](int k, unsigned int& s, long long& m) {
          const CompN v = c[k];
          s = v.cs;
          m = (long long)v.pl;
        },
        cnt, x, (unsigned int)width, bs, c32, pl, next);
    cs = lo + (long long)c32;
  } else {
    const Comp* c = p.comp[l] + off;
    const long long from = bl == 0 ? (long long)st.min_s : lo;  // at or before every start
    any = find_comp(
        [&](int k, long long& s, long long& m) {
          const Comp v = c[k];
          s = v.cs - from;
          m = v.pl;
        },
        cnt, t - from, lo + width - from, bs, cs, pl, next);
    cs += from;
  }
  if (!any) {
    // only the component carried in from earlier buckets lies before t
    const long long ext = carry + next;
    return base + (ext < t ? ext : t) - carry;
  }
  const long long ce = cs + (next - pl);
  return base + pl + (ce < t ? ce : t) - cs;
}

// The build's status words into the results (threads 0-2 of one workgroup, in
// the last kernel of a launch sequence), and back to their identities if asked.
__device__ __forceinline__ void put_status(const Plan& p, unsigned long long* status, bool reset) {
  const int i = threadIdx.x;
  if (i < 3) {
    unsigned long long* w = i == 0 ? p.err : p.oversized + (i - 1);
    status[i] = *w;
    if (reset) *w = i == 0 ? ULLONG_MAX : 0ull;
  }
}

__global__ void k_status(Plan p, unsigned long long* status, bool reset) { put_status(p, status, reset); }

// Plain regions: a slice of resources of one region per workgroup, eight
// threads per resource (level and end), clips them by binary search, writes
// their state times and adds its sums and maxima to the region's accumulator.
// The region's last slice to add makes the tree (FP64 ratios) and leaves the
// accumulator clear. Only atomics pass between the slices: a wave asks for the
// results of its adds and waits for them (s_waitcnt vmcnt(0): an atomic whose
// result is back is done in memory) before one of its lanes counts the slice.
// Relaxed atomics of several lanes are not ordered by the language, so the wait
// stands in the code, and a test reads the order in what is built from it. What
// the language offers costs more: a device-scope release per slice, which also
// writes back the L2 (large trace 1117 -> 1149 us, mid 172 -> 176, a batch of 128
// traces 376 -> 459), or the trees in a second kernel (1127 -> 1126, 168 -> 173,
// 370 -> 378, 256 devices with their streams 528 -> 540).
// A region of one slice needs no accumulator at all.
//
// The stage is a chain of about ten cache misses, and one CU has only so many
// in flight: a few regions (the rule below: up to 8192 resource clips, or at
// most 16 resources each) take slices of 8 resources, a wave, to spread over
// the CUs; more take slices of 32, with fewer accumulator atomics. Mid trace
// (16 regions x 128 resources): 13.0 us, against 17.5 with a workgroup per
// region and 15.8 as two kernels; small trace (1 x 8): 4.0 against 9.5.
__global__ __launch_bounds__(256) void k_region(Plan p, const RegionDesc* regions, long long* times, Tree* trees,
                                                unsigned long long* status, bool reset) {
  __shared__ long long lds[4 * 10];
  __shared__ long long tot[9];
  __shared__ Tree tree;
  __shared__ int s_last;
  if (blockIdx.x == 0 && blockIdx.y == 0) put_status(p, status, reset);
  const RegionDesc rd = regions[blockIdx.x];
  if (rd.n_ivl) return;  // a per-resource region: k_region_multi
  const int R = rd.n_hosts + rd.n_devices;
  const int slice = (int)blockDim.x >> 3;
  const int r0 = blockIdx.y * slice;
  if (r0 >= R && r0 > 0) return;  // uniform: past the region's resources
  const int slices = max(1, (R + slice - 1) / slice);
  const int r = r0 + (int)(threadIdx.x >> 3);
  const int l = (threadIdx.x >> 1) & 3, ep = threadIdx.x & 1;
  const bool host = r < rd.n_hosts;
  const long long E = rd.t1 - rd.t0;
  long long v[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  long long M = 0, D[3];
  if (r < R && l < (host ? 3 : 2)) M = measure_before(p, rd.seg_begin + r, l, ep ? rd.t1 : rd.t0);
  group_levels(M, D);
  if ((threadIdx.x & 7) == 0 && r < R) add_times(host, D, E, times + (rd.times_off + r) * 4, v);
  block_tree(v, lds);
  if (slices > 1) {
    unsigned long long* acc = p.racc + (long long)blockIdx.x * kRaccWords;
    if (threadIdx.x == 0)
      for (int i = 0; i < 9; ++i) tot[i] = v[i];
    __syncthreads();
    if (threadIdx.x < 64) {  // one wave: a lane per word, then one lane counts the slice
      unsigned long long old = 0;
      if (threadIdx.x < 6) old = atomicAdd(acc + threadIdx.x, (unsigned long long)tot[threadIdx.x]);
      else if (threadIdx.x < 9) old = atomicMax(acc + threadIdx.x, (unsigned long long)tot[threadIdx.x]);
      // every lane's result is back, so its add is done in memory, before the count goes out
      asm volatile("s_waitcnt vmcnt(0)" ::"v"((unsigned int)old), "v"((unsigned int)(old >> 32)) : "memory");
      if (threadIdx.x == 0) s_last = (int)atomicAdd(acc + 9, 1ull) == slices - 1;
    }
    __syncthreads();
    if (!s_last) return;
    if (threadIdx.x < 9) tot[threadIdx.x] = (long long)atomicExch(acc + threadIdx.x, 0ull);
    else if (threadIdx.x == 9) (void)atomicExch(acc + 9, 0ull);
    __syncthreads();
    if (threadIdx.x == 0)
      for (int i = 0; i < 9; ++i) v[i] = tot[i];
  }
  if (threadIdx.x == 0) tree = make_tree(E, rd.n_hosts, rd.n_devices, v);
  __syncthreads();
  put_trees(&tree, 1, trees + blockIdx.x);
}

// Regions given as per-resource interval lists (a region entered repeatedly,
// each resource on its own clock). The first part adds, per (interval, level,
// end of the interval), the level's measure before that end (the start with a
// minus sign) and each interval's length; the second turns them into state
// times (the remainder completes the resource's own time in the region) and
// the tree, with E the largest host in-region time (eq. 1), or the largest
// device one when no host process is in the region, and leaves the
// accumulators clear for the next pass (k_ivl_zero clears a new plan's).
//
// The first part is a chain of cache misses (16 regions x 128 resources x 32
// entries fit the GPU at once), so what a thread needs to start lies in its
// interval: 29 -> 26 us there, and with two launches fewer (the status words and
// the clearing) a pass takes 49 us instead of 56.
__global__ __launch_bounds__(256) void k_ivl_zero(const RegionDesc* regions, long long* macc) {
  const RegionDesc rd = regions[blockIdx.x];
  if (rd.n_ivl == 0) return;
  const int R = rd.n_hosts + rd.n_devices;
  for (int i = threadIdx.x; i < 4 * R; i += 256) macc[rd.times_off * 4 + i] = 0;
}

__global__ __launch_bounds__(256) void k_ivl_acc(Plan p, const IvlDesc* ivls, long long n_ivls, long long* macc) {
  const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
  const long long i = t >> 3;
  if (i >= n_ivls) return;
  const int l = (int)((t >> 1) & 3), ep = (int)(t & 1);
  const IvlDesc iv = ivls[i];
  unsigned long long* acc = (unsigned long long*)(macc + iv.row * 4);
  if (l == 3) {
    if (ep) atomicAdd(acc + 3, (unsigned long long)(iv.b - iv.a));
    return;
  }
  if (l >= iv.n_levels) return;
  const long long v = measure_before(p, iv.seg, l, ep ? iv.b : iv.a);
  atomicAdd(acc + l, (unsigned long long)(ep ? v : -v));  // two's complement: the sum is exact
}

template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_region_multi(Plan p, const RegionDesc* regions, long long* macc,
                                                          Tree* trees, long long* times, unsigned long long* status,
                                                          bool reset) {
  __shared__ long long lds[THREADS / 64 * 10];
  __shared__ Tree tree;
  __shared__ long long semax[2][THREADS / 64];
  if (status && blockIdx.x == 0) put_status(p, status, reset);
  const RegionDesc rd = regions[blockIdx.x];
  if (rd.n_ivl == 0) return;
  const int R = rd.n_hosts + rd.n_devices;
  // sums: U, W, MPI, Other, K, M ; maxes: U+W, K, K+M
  long long v[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  long long eh = 0, ed = 0;
  for (int r = threadIdx.x; r < R; r += THREADS) {
    long long* a = macc + (rd.times_off + r) * 4;
    const long long D[3] = {a[0], a[1], a[2]}, Er = a[3];
    a[0] = a[1] = a[2] = a[3] = 0;
    const bool host = r < rd.n_hosts;
    add_times(host, D, Er, times + (rd.times_off + r) * 4, v);
    if (host) eh = Er > eh ? Er : eh;
    else ed = Er > ed ? Er : ed;
  }
  eh = wave_reduce_i64<OpMax>(eh, 0);
  ed = wave_reduce_i64<OpMax>(ed, 0);
  if ((threadIdx.x & 63) == 0) {
    semax[0][threadIdx.x >> 6] = eh;
    semax[1][threadIdx.x >> 6] = ed;
  }
  block_tree(v, lds);  // its barriers also publish semax
  if (threadIdx.x == 0) {
    for (int w = 0; w < THREADS / 64; ++w) {
      eh = semax[0][w] > eh ? semax[0][w] : eh;
      ed = semax[1][w] > ed ? semax[1][w] : ed;
    }
    tree = make_tree(eh ? eh : ed, rd.n_hosts, rd.n_devices, v);
  }
  __syncthreads();
  put_trees(&tree, 1, trees + blockIdx.x);
}

// ----------------------------------------------------------------------------
// launchers
// ----------------------------------------------------------------------------

hipError_t launch_gather(const CopyChunk* chunks, int n, hipStream_t st) {
  // a launch holds fewer than 2^31 threads: a chunk past that (4.3e9 records) is cut
  constexpr long long kMaxPieces = 1ll << 22;
  GatherArgs g;
  g.n = 0;
  long long pieces = 0;
  auto flush = [&]() -> hipError_t {
    if (g.n == 0) return hipSuccess;
    g.first[g.n] = (unsigned int)pieces;
    hipLaunchKernelGGL(k_gather, dim3((unsigned)pieces), dim3(256), 0, st, g);
    g.n = 0;
    pieces = 0;
    return hipGetLastError();
  };
  for (int i = 0; i < n; ++i) {
    CopyChunk c = chunks[i];
    while (c.count > 0) {
      const long long room = (kMaxPieces - pieces) * (long long)kGatherPiece;
      if (g.n == kGatherChunks || room <= 0) {
        const hipError_t e = flush();
        if (e != hipSuccess) return e;
        continue;
      }
      CopyChunk part = c;
      part.count = std::min<long long>(c.count, room);
      g.first[g.n] = (unsigned int)pieces;
      g.c[g.n++] = part;
      pieces += (part.count + kGatherPiece - 1) / kGatherPiece;
      c.s += part.count;
      c.e += part.count;
      c.dst_s += part.count;
      c.dst_e += part.count;
      c.count -= part.count;
    }
  }
  return flush();
}

hipError_t launch_build_small(const Plan& p, hipStream_t st) {
  if (p.n_segs == 0) return hipSuccess;
  hipLaunchKernelGGL(k_build_small, dim3((unsigned)p.n_segs), dim3(kSmallThreads), 0, st, p);
  return hipGetLastError();
}

hipError_t launch_reset(const Plan& p, hipStream_t st) {
  const long long work = max(3 * p.n_buckets + p.n_segs, p.n_tiles) + 64;
  int blocks = (int)min(2048ll, (work + 255) / 256);
  hipLaunchKernelGGL(k_reset, dim3(blocks), dim3(256), 0, st, p);
  return hipGetLastError();
}

hipError_t launch_range(const Plan& p, bool reset, hipStream_t st) {
  // many segments (a batch of small traces: 1.6e4) hold few records each, so a
  // wave takes one (37 us, 44 with two waves); the reset pass wants a workgroup
  // per few hundred buckets
  const bool many = p.n_segs >= 2048;
  long long blocks = p.n_segs;
  if (reset) blocks = max(blocks, min(1024ll, (3 * p.n_buckets + 511) / 512));
  if (many)
    hipLaunchKernelGGL(k_range<64>, dim3((unsigned)blocks), dim3(64), 0, st, p, reset);
  else
    hipLaunchKernelGGL(k_range<512>, dim3((unsigned)blocks), dim3(512), 0, st, p, reset);
  return hipGetLastError();
}

hipError_t launch_stats(const Plan& p, hipStream_t st) {
  // the tiles of single chunks, then (in the same launch) the shared tiles
  const long long own = p.n_own_tiles, sh = p.n_tiles - p.n_own_tiles;
  if (p.tile_elems <= 512) {
    const unsigned blocks = (unsigned)((own + 3) / 4 + sh);
    if (sh > 0) hipLaunchKernelGGL(k_stats_small<true>, dim3(blocks), dim3(256), 0, st, p);
    else if (own > 0) hipLaunchKernelGGL(k_stats_small<false>, dim3(blocks), dim3(256), 0, st, p);
  } else if (sh > 0) {
    hipLaunchKernelGGL((k_stats<256, true>), dim3((unsigned)p.n_tiles), dim3(256), 0, st, p);
  } else if (own > 0) {
    hipLaunchKernelGGL((k_stats<256, false>), dim3((unsigned)p.n_tiles), dim3(256), 0, st, p);
  }
  if (p.n_segs > 0) hipLaunchKernelGGL(k_geom, dim3((unsigned)((p.n_segs + 255) / 256)), dim3(256), 0, st, p);
  return hipGetLastError();
}

// Count and scatter launches: one block per tile, the shared tiles (if any)
// after the others; plans share tiles only at 512 and 2048 records per tile.
hipError_t launch_hist(const Plan& p, hipStream_t st) {
  if (p.n_tiles == 0) return hipSuccess;
  const dim3 grid((unsigned)p.n_tiles);
  if (p.n_tiles > p.n_own_tiles) {
    switch (p.tile_elems) {
      case 512: hipLaunchKernelGGL((k_hist<128, 4, true>), grid, dim3(128), 0, st, p); break;
      case 2048: hipLaunchKernelGGL((k_hist<512, 4, true>), grid, dim3(512), 0, st, p); break;
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  switch (p.tile_elems) {
    case 512: hipLaunchKernelGGL((k_hist<128, 4, false>), grid, dim3(128), 0, st, p); break;
    case 2048: hipLaunchKernelGGL((k_hist<512, 4, false>), grid, dim3(512), 0, st, p); break;
    case 8192: hipLaunchKernelGGL((k_hist<1024, 8, false>), grid, dim3(1024), 0, st, p); break;
    default: hipLaunchKernelGGL((k_hist<512, 8, false>), grid, dim3(512), 0, st, p); break;
  }
  return hipGetLastError();
}

hipError_t launch_scan(const Plan& p, hipStream_t st) {
  const long long blocks = (p.n_buckets + kScanTile - 1) / kScanTile;
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(k_scan<256>, dim3((unsigned)blocks), dim3(256), 0, st, p);
  return hipGetLastError();
}

hipError_t launch_scatter(const Plan& p, hipStream_t st) {
  if (p.n_tiles == 0) return hipSuccess;
  const dim3 grid((unsigned)p.n_tiles);
  if (p.n_tiles > p.n_own_tiles) {
    switch (p.tile_elems) {
      case 512: hipLaunchKernelGGL((k_scatter<128, 4, true>), grid, dim3(128), 0, st, p); break;
      case 2048: hipLaunchKernelGGL((k_scatter<512, 4, true>), grid, dim3(512), 0, st, p); break;
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  switch (p.tile_elems) {
    case 512: hipLaunchKernelGGL((k_scatter<128, 4, false>), grid, dim3(128), 0, st, p); break;
    case 2048: hipLaunchKernelGGL((k_scatter<512, 4, false>), grid, dim3(512), 0, st, p); break;
    case 8192: hipLaunchKernelGGL((k_scatter<1024, 8, false>), grid, dim3(1024), 0, st, p); break;
    default: hipLaunchKernelGGL((k_scatter<512, 8, false>), grid, dim3(512), 0, st, p); break;
  }
  return hipGetLastError();
}

// many buckets per segment: the per-segment passes take a workgroup for each
static bool big_segments(const Plan& p) { return p.n_buckets >= 128 * (int64_t)p.n_segs; }

hipError_t launch_carry(const Plan& p, hipStream_t st) {
  if (p.n_segs == 0) return hipSuccess;
  if (p.seg_group > 1)
    hipLaunchKernelGGL(k_carry_grouped<64>, dim3((unsigned)((p.n_segs + kSegGroup - 1) / kSegGroup)), dim3(64), 0, st, p);
  else
    hipLaunchKernelGGL(k_carry<64>, dim3((unsigned)p.n_segs), dim3(64), 0, st, p);  // a wave per segment, spread over the CUs
  return hipGetLastError();
}

hipError_t launch_scan_carry(const Plan& p, hipStream_t st) {
  const long long scan_blocks = (p.n_buckets + kScanTile - 1) / kScanTile;
  const long long waves = p.seg_group > 1 ? (p.n_segs + kSegGroup - 1) / kSegGroup : p.n_segs;
  const long long blocks = scan_blocks + (waves + 3) / 4;
  if (blocks == 0) return hipSuccess;
  if (big_segments(p)) {
    hipLaunchKernelGGL((k_scan_carry<false, true>), dim3((unsigned)(scan_blocks + p.n_segs)), dim3(256), 0, st, p,
                       (int)scan_blocks);
    return hipGetLastError();
  }
  if (p.seg_group > 1)
    hipLaunchKernelGGL(k_scan_carry<true>, dim3((unsigned)blocks), dim3(256), 0, st, p, (int)scan_blocks);
  else
    hipLaunchKernelGGL(k_scan_carry<false>, dim3((unsigned)blocks), dim3(256), 0, st, p, (int)scan_blocks);
  return hipGetLastError();
}

hipError_t launch_merge_wave(const Plan& p, hipStream_t st) {
  if (p.n_buckets == 0) return hipSuccess;
  const dim3 grid((unsigned)((p.n_buckets + 3) / 4));
  if (p.slot_cap >= 128)
    hipLaunchKernelGGL(k_merge_wave<true>, grid, dim3(256), 0, st, p);
  else
    hipLaunchKernelGGL(k_merge_wave<false>, grid, dim3(256), 0, st, p);
  return hipGetLastError();
}

hipError_t launch_merge_rest(const Plan& p, int cap, hipStream_t st) {
  if (p.n_buckets == 0) return hipSuccess;
  // persistent workgroups (as many as fit) for the buckets the wave path handed over
  const unsigned grid = (unsigned)std::min<long long>(p.n_buckets, 768);
  if (cap == 2048)
    hipLaunchKernelGGL((k_merge_rest<256, 2048>), dim3(grid), dim3(256), 0, st, p);
  else
    hipLaunchKernelGGL((k_merge_rest<256, 4096>), dim3(grid), dim3(256), 0, st, p);
  return hipGetLastError();
}

hipError_t launch_base(const Plan& p, hipStream_t st) {
  if (p.n_segs == 0) return hipSuccess;
  if (big_segments(p)) {
    hipLaunchKernelGGL(k_base_big, dim3((unsigned)p.n_segs), dim3(256), 0, st, p);
    return hipGetLastError();
  }
  if (p.seg_group > 1)
    hipLaunchKernelGGL(k_base_grouped<64>, dim3((unsigned)((p.n_segs + kSegGroup - 1) / kSegGroup)), dim3(64), 0, st, p);
  else
    hipLaunchKernelGGL(k_base<64>, dim3((unsigned)p.n_segs), dim3(64), 0, st, p);  // a wave per segment, spread over the CUs
  return hipGetLastError();
}

hipError_t launch_region(const Plan& p, const RegionDesc* regions, int n_regions, int n_plain, int max_res, Tree* trees,
                         unsigned long long* status, bool reset, long long* times, const IvlDesc* ivls,
                         long long n_ivls, long long* macc, bool clear_macc, hipStream_t st) {
  // the status words go with the last kernel (of plain regions, or of those by
  // intervals), or alone
  if (n_plain == 0 && n_ivls == 0) {
    hipLaunchKernelGGL(k_status, dim3(1), dim3(64), 0, st, p, status, reset);
  } else if (n_plain > 0) {
    const int slice = max_res <= 16 || (long long)n_plain * max_res <= 8192 ? 8 : 32;
    const unsigned slices = (unsigned)std::max(1, (max_res + slice - 1) / slice);
    hipLaunchKernelGGL(k_region, dim3((unsigned)n_regions, slices), dim3(8 * slice), 0, st, p, regions, times, trees,
                       status, reset);
  }
  if (n_ivls > 0) {
    if (clear_macc) hipLaunchKernelGGL(k_ivl_zero, dim3((unsigned)n_regions), dim3(256), 0, st, regions, macc);
    hipLaunchKernelGGL(k_ivl_acc, dim3((unsigned)((8 * n_ivls + 255) / 256)), dim3(256), 0, st, p, ivls, n_ivls, macc);
    hipLaunchKernelGGL(k_region_multi<256>, dim3((unsigned)n_regions), dim3(256), 0, st, p, regions, macc, trees, times,
                       n_plain == 0 ? status : nullptr, reset);
  }
  return hipGetLastError();
}

}  // namespace hpop
