// Launchers of the reduction kernels (all asynchronous on `st`).
#pragma once
#include <hip/hip_runtime.h>

#include "hpop_internal.h"

namespace hpop {

constexpr int kScanTile = 1024;  // bucket counts per workgroup of the offset scan
constexpr int kHistWin = 512;    // LDS bucket window of one streaming tile

// One add call's chunk to copy into the record arena: `count` starts to dst_s, ends to dst_e.
struct CopyChunk {
  const int64_t* s;
  const int64_t* e;
  int64_t* dst_s;
  int64_t* dst_e;
  int64_t count;
};
hipError_t launch_gather(const CopyChunk* chunks, int n, hipStream_t st);  // host array, any n

hipError_t launch_build_small(const Plan& p, hipStream_t st);  // a plan with p.sseg: the whole build
hipError_t launch_reset(const Plan& p, hipStream_t st);
hipError_t launch_range(const Plan& p, bool reset, hipStream_t st);  // sampled start ranges (p.seg_first); reset: that pass too
hipError_t launch_stats(const Plan& p, hipStream_t st);
hipError_t launch_hist(const Plan& p, hipStream_t st);
hipError_t launch_scan(const Plan& p, hipStream_t st);
hipError_t launch_scatter(const Plan& p, hipStream_t st);
hipError_t launch_carry(const Plan& p, hipStream_t st);
hipError_t launch_scan_carry(const Plan& p, hipStream_t st);  // fixed slots: scan and carry in one launch
hipError_t launch_merge_wave(const Plan& p, hipStream_t st);
hipError_t launch_merge_rest(const Plan& p, int cap, hipStream_t st);
hipError_t launch_base(const Plan& p, hipStream_t st);
// Regions (n_plain of them [t0, t1), the rest per resource) and the status
// words {first bad record, oversized buckets, slot overflows}. trees and
// status: device or page-locked host memory. reset: the build's own status
// words go back to their identities once they are stored. clear_macc: the
// intervals' accumulators are cleared first (every pass leaves them clear).
hipError_t launch_region(const Plan& p, const RegionDesc* regions, int n_regions, int n_plain, int max_res, Tree* trees,
                         unsigned long long* status, bool reset, long long* times, const IvlDesc* ivls,
                         long long n_ivls, long long* macc, bool clear_macc, hipStream_t st);

}  // namespace hpop
