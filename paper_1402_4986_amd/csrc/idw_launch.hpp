// Host-side launch descriptors shared by the C-ABI layer and the kernel translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "idw_device.hpp"

namespace idw {

// Everything a forward launch needs; pointers are device pointers.
struct FwdArgs {
  DevPts data;
  int64_t n = 0;
  DevPts query;
  int64_t m = 0;
  int dim = 2;
  int pmode = PM_GEN;
  double p = 2.0;
  unsigned flags = 0;
  int q_per_lane = 8;
  bool kahan = false;  // FP32 sweep with per-pair Kahan compensation
  bool rel = false;    // FP32 relative weights (p >= kRelP): needs rmin
  const unsigned long long* rmin = nullptr;  // [m] nearest squared distance (FP32 bits)
  int split = 1;
  int64_t chunk = 0;  // data points per split chunk (a multiple of 64; of the tile but in the finest splits)
  const double* hdr = nullptr;
  void* out_z = nullptr;
  double* out_den = nullptr;
  uint8_t* flag = nullptr;
  double2* part = nullptr;
  const int* list = nullptr;
  const int* count = nullptr;
  int fix_cmax = 1;              // most data chunks per flagged query in the FP64 fix-up
  double4* fpart = nullptr;      // [kFixGrid] fix-up chunk partials
  bool small = false;            // one kernel after the sweep (k_fwd_finish_small)
};

// Everything a backward launch needs.
struct BwdArgs {
  DevPts data;
  int64_t n = 0;
  DevPts query;
  int64_t m = 0;
  int dim = 2;
  int pmode = PM_GEN;
  double p = 2.0;
  unsigned flags = 0;
  int q_per_lane = 4;    // query sweep: queries per lane
  int x_per_lane = 4;    // data sweep: data points per lane
  int split_q = 1;       // data chunks of the query sweep
  int64_t chunk_q = 0;
  int split_z = 1;       // query chunks of the data sweep
  int64_t chunk_z = 0;
  double4* part_q = nullptr;  // [split_q][m] (P, Gx, Gy, Gz)
  double* part_z = nullptr;   // [split_z][n]
  double* part_x = nullptr;   // [split_z][n][dim] data-coordinate sums (null: not requested)
  int fused_groups = 0;       // fused FP32 sweep: query-block groups (= dz partial rows)
  int fused_ranges = 0;       // fused FP32 sweep: data ranges (= query partial rows)
  int64_t fused_chunk = 0;
  const double* hdr = nullptr;
  const void* grad_out = nullptr;
  const void* saved_z = nullptr;
  const double* saved_den = nullptr;
  const uint8_t* route = nullptr;  // [m] settled QueryRoute of each query
  bool rel = false;                // fused FP32 sweep with relative weights (p >= kRelP)
  void* grad_z = nullptr;
  void* grad_q = nullptr;
  void* grad_x = nullptr;
  double* wg_dp = nullptr;      // [nwg_dp] dp partials of the query merge's workgroups
  int nwg_dp = 0;
  double* grad_p = nullptr;     // null: not requested
  const int* list = nullptr;    // flagged queries, ascending
  const int* count = nullptr;
  double* slot_coef = nullptr;  // [m] per flagged slot: g/D (or g/h at a hit)
  int* slot_hits = nullptr;     // [m] per flagged slot: hit count h
  double* slot_dp = nullptr;    // [m] per flagged slot: dp contribution
  double* slot_z = nullptr;     // [m] per flagged slot: FP64 Z
  double* slot_den = nullptr;   // [m] per flagged slot: FP64 denominator
  int fix_cmax = 1;
  double4* fpart = nullptr;     // [kFixGrid] fix-up chunk partials
};

// The nearest-distance check of candidate queries (k_near_check).
struct NearArgs {
  DevPts data;
  int64_t n = 0;
  DevPts query;
  int64_t m = 0;  // queries in all (bounds the candidates)
  int dim = 2;
  bool f64 = false;
  bool excl = false;
  const int* list = nullptr;   // query indices
  const int* count = nullptr;  // number of them (device)
  const int* list2 = nullptr;  // taken instead where the first count is 0 (nullable)
  const int* count2 = nullptr;
  const double* hdr = nullptr;
  unsigned long long* minb = nullptr;  // [m] per-query minimum (bits)
  bool all = false;   // every query 0..m-1 (the lists and counts unused)
  bool init = false;  // set the minima to +inf first
};

// The header kernels (bounding box, thresholds, cleared counts).
struct HeaderArgs {
  DevPts data;
  int64_t n = 0;
  double p = 2.0;
  bool rel = false;
  double* part = nullptr;  // [nblocks] partial boxes
  int nblocks = 1;
  double* hdr = nullptr;
};

// Per-query routes and lists.
struct RouteArgs {
  int64_t m = 0;
  const double* hdr = nullptr;
  int* hint = nullptr;      // header int slots
  uint8_t* route = nullptr; // [m]
  int* list = nullptr;      // [m] candidates, then the F_FP64 queries
  int* bcnt = nullptr;      // [m / kCountBlock + 1] scratch
  unsigned long long* minb = nullptr;  // [m]
};

// The grid of the nearest-distance searches (idw_grid.hpp).
struct GridArgs {
  DevPts data;
  int64_t n = 0;
  DevPts query;
  int64_t m = 0;
  int dim = 2;
  bool f64 = false;
  bool excl = false;
  bool nearest = false;              // search: ring search over all queries, else candidate check
  const double* hdr = nullptr;
  int* hint = nullptr;               // header int slots (flagged count, then GridInt)
  int* cnt = nullptr;                // [ncell_max + 1] cell counts, then scatter cursors
  int* start = nullptr;              // [ncell_max + 1] first record of each cell
  int* bsum = nullptr;               // [scan blocks] block sums of the counts
  int64_t ncell_max = 0;
  void* rec = nullptr;               // [n] P4<T>: scaled coordinates and point index
  const int* list = nullptr;         // candidate check: candidate queries
  uint8_t* route = nullptr;          // candidate check: QueryRoute written per candidate
  unsigned long long* minb = nullptr;  // ring search: nearest squared distance (bits)
  int* blist = nullptr;              // [m] queries handed to the brute-force check
};

constexpr int kTile = 512;        // data points staged in LDS per tile (2 per thread)
constexpr int kFixGrid = 1024;    // workgroups of the FP64 fix-up kernels
constexpr int kCountBlock = 4096; // flags per compaction block (16 per thread)

// Forwards that k_fwd_finish_small ends.  Few pairs, so that even if every query is a candidate or
// a hit (passes over the data by one workgroup of four queries) the call is no longer than with
// the general kernels (8,192 x 8,192: 38.8 us against 37.8, all hits 126 against 194; 10,240 x
// 10,240, twice the pairs: 43.8 against 45.6, but all candidates 104 against 94); neither set so
// long that a workgroup per four queries, or one workgroup's pass over the data, would be; and,
// since a pass gets longer with n while the launches that it saves matter less with n m, a limit
// on n^2 m: with four neighbouring hits 12,288 x 4,096 takes 64 us and 16,384 x 2,048 70 (the
// general kernels 44 and 43; without hits 31.9 and 24.6 against 35.2 and 33.5), but 16,384 x 4,096
// 91, against 50, with nothing to gain without hits (40.4 against 41.6).
constexpr int64_t kSmallPairs = int64_t(1) << 26;
constexpr int64_t kSmallSet = 16384;
constexpr int64_t kSmallPass = int64_t(5) << 37;
inline bool small_call(int64_t n, int64_t m) {
  return n <= kSmallSet && m <= kSmallSet && n * m <= kSmallPairs && n * n * m <= kSmallPass;
}

// Per-layout entry points (one translation unit per layout keeps builds parallel).
#define IDW_DECLARE_LAYOUT(NAME)                                                 \
  hipError_t fwd_sweep_##NAME(const FwdArgs& a, bool f64, hipStream_t st);       \
  hipError_t fwd_fixup_##NAME(const FwdArgs& a, bool f64, hipStream_t st);       \
  hipError_t header_##NAME(const HeaderArgs& a, int dim, bool f64, hipStream_t st); \
  hipError_t bwd_query_##NAME(const BwdArgs& a, bool f64, hipStream_t st);       \
  hipError_t bwd_data_##NAME(const BwdArgs& a, bool f64, hipStream_t st);        \
  hipError_t bwd_datax_##NAME(const BwdArgs& a, bool f64, hipStream_t st);       \
  hipError_t bwd_fixup_##NAME(const BwdArgs& a, bool f64, hipStream_t st);      \
  hipError_t bwd_fused_##NAME(const BwdArgs& a, bool f64, hipStream_t st);       \
  hipError_t near_check_##NAME(const NearArgs& a, hipStream_t st);              \
  hipError_t grid_##NAME(const GridArgs& a, bool build, hipStream_t st);

IDW_DECLARE_LAYOUT(soa)
IDW_DECLARE_LAYOUT(aos)
IDW_DECLARE_LAYOUT(aoas)
IDW_DECLARE_LAYOUT(hybrid)
IDW_DECLARE_LAYOUT(soaos)

// Layout-independent kernels (idw_common.hip).
hipError_t bbox_final(const double* part, int nblocks, int dim, double p, bool f32_scaling,
                      bool rel, double* hdr, hipStream_t st);
// The split partials' merge, or (split 1) the sweep's own routes: collects the candidates too.
hipError_t merge_split(const FwdArgs& a, const RouteArgs& r, bool f64, hipStream_t st);
// Routes from the saved denominators, candidates collected.
hipError_t flags_from_den(const double* den, const RouteArgs& r, bool f64, hipStream_t st);
// Settles the candidates by their minima and lists the F_FP64 queries in ascending order.
hipError_t settle(const RouteArgs& r, bool f64, hipStream_t st);
hipError_t compact_flags(const uint8_t* flag, int64_t m, int* bcnt, int* list, int* count,
                         uint8_t want, hipStream_t st);
// The merges of the adjoint's partials that were requested, in one launch: grad_q and the dp
// partials (query), grad_z (data), grad_x (its partials are a.split_z rows).
hipError_t bwd_merge(const BwdArgs& a, bool query, bool data, bool x, bool f64, hipStream_t st);
hipError_t dp_final(const double* wg_dp, int nwg, const double* slot_dp, const int* count,
                    double* grad_p, hipStream_t st);
// Grid geometry, the per-call gates (mode 0: candidate check; mode 1: ring search of all m
// queries) and cleared counts; then the exclusive scan of the cell counts.
hipError_t grid_setup(const GridArgs& a, int mode, const int* ncand, hipStream_t st);
hipError_t grid_scan(const GridArgs& a, hipStream_t st);

}  // namespace idw
