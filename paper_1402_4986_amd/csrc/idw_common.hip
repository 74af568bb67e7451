// Layout-independent kernels: extent/threshold header, split merge, deterministic
// compaction of flagged queries, and the final dp reduction.
#include <math.h>

#include "idw_bwd.hpp"
#include "idw_device.hpp"
#include "idw_fwd.hpp"
#include "idw_launch.hpp"

namespace idw {

// Reduces the per-workgroup extent partials and fills the workspace header.
template <int DIM>
__global__ __launch_bounds__(kWG) void k_bbox_final(const double* __restrict__ part, int nb, double p, int f32s,
                                                    int rel, double* __restrict__ hdr) {
  __shared__ double red[kWG / 64][Box<double, DIM>::N];
  Box<double, DIM> b;
  b.clear();
  for (int k = threadIdx.x; k < nb; k += kWG) {
    const double* o = part + k * kBboxStride;
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      b.v[d] = fmax(b.v[d], -o[d]);
      b.v[DIM + d] = fmax(b.v[DIM + d], o[3 + d]);
    }
    b.v[2 * DIM] = fmax(b.v[2 * DIM], o[6]);
  }
  b.template reduce<kWG>(red);
  if (threadIdx.x == 0) {
    double mn[3] = {0.0, 0.0, 0.0}, mx[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      mn[d] = -b.v[d];
      mx[d] = b.v[DIM + d];
    }
    finish_header(hdr, mn, mx, DIM, b.v[2 * DIM], p, f32s != 0, rel != 0);
  }
}

hipError_t bbox_final(const double* part, int nblocks, int dim, double p, bool f32_scaling,
                      bool rel, double* hdr, hipStream_t st) {
  if (dim == 3)
    hipLaunchKernelGGL(k_bbox_final<3>, dim3(1), dim3(kWG), 0, st, part, nblocks, p, f32_scaling ? 1 : 0, rel ? 1 : 0,
                       hdr);
  else
    hipLaunchKernelGGL(k_bbox_final<2>, dim3(1), dim3(kWG), 0, st, part, nblocks, p, f32_scaling ? 1 : 0, rel ? 1 : 0,
                       hdr);
  return hipGetLastError();
}

// Merges split partials (TwoSum-compensated FP64), finalises and collects the candidates; with
// split 1 the sweep has finalised and only the candidates are collected.  P threads share a
// query: thread part k adds the k-th part of its chunks in chunk order, then the parts are added
// in order.  P = 4 for few queries, whose chunks are many: 10,240 queries in 80 chunks 4.8 us,
// where one thread per query took 7.9 us for 20 chunks.
template <typename T, int P>
__global__ __launch_bounds__(kWG) void k_merge(const double2* __restrict__ part, int64_t m,
                                               int split, const double* __restrict__ hdr,
                                               T* __restrict__ out_z, double* __restrict__ out_den,
                                               uint8_t* __restrict__ flag, int* __restrict__ hint,
                                               int* __restrict__ list, unsigned long long* __restrict__ minb) {
  constexpr int NQ = kWG / P;
  __shared__ double4 sums[P > 1 ? kWG : 1];
  const int64_t i = static_cast<int64_t>(blockIdx.x) * NQ + threadIdx.x % NQ;
  uint8_t r = F_FP32;
  double nh = 0.0, nl = 0.0, dh = 0.0, dl = 0.0;
  if (split > 1 && i < m) {
    const int k = threadIdx.x / NQ, len = (split + P - 1) / P;
    const int c1 = (k + 1) * len < split ? (k + 1) * len : split;
#pragma unroll 4
    for (int c = k * len; c < c1; ++c) {
      const double2 v = part[static_cast<int64_t>(c) * m + i];
      two_sum_acc(nh, nl, v.x);
      two_sum_acc(dh, dl, v.y);
    }
  }
  if constexpr (P > 1) {
    sums[threadIdx.x] = make_double4(nh, nl, dh, dl);
    __syncthreads();
    if (threadIdx.x < NQ)
      for (int k = 1; k < P; ++k) {
        const double4 v = sums[k * NQ + threadIdx.x];
        two_sum_acc(nh, nl, v.x);
        two_sum_acc(dh, dl, v.z);
        nl += v.y;
        dl += v.w;
      }
  }
  if (threadIdx.x < NQ && i < m) {
    if (split > 1) {
      const double num = nh + nl, den = dh + dl;
      out_z[i] = static_cast<T>(num / den);
      if (out_den) out_den[i] = den * hdr[H_DEN_UNIT];
      r = route_of(den, hdr, false);
      flag[i] = r;
    } else {
      r = flag[i];
    }
  }
  append_candidates(r == F_CANDIDATE, i, hint, list, minb, min_bits(infT<T>()));
}

template <typename T>
static hipError_t merge_split_t(const FwdArgs& a, const RouteArgs& r, hipStream_t st) {
  // below this many queries one thread per query leaves most of the chip idle
  const bool few = a.split >= 8 && a.m < 65536;
  const int64_t per = few ? kWG / 4 : kWG;
  dim3 grid(static_cast<unsigned>((a.m + per - 1) / per));
  if (few)
    hipLaunchKernelGGL((k_merge<T, 4>), grid, dim3(kWG), 0, st, a.part, a.m, a.split, a.hdr,
                       static_cast<T*>(a.out_z), a.out_den, r.route, r.hint, r.list, r.minb);
  else
    hipLaunchKernelGGL((k_merge<T, 1>), grid, dim3(kWG), 0, st, a.part, a.m, a.split, a.hdr,
                       static_cast<T*>(a.out_z), a.out_den, r.route, r.hint, r.list, r.minb);
  return hipGetLastError();
}

hipError_t merge_split(const FwdArgs& a, const RouteArgs& r, bool f64, hipStream_t st) {
  return f64 ? merge_split_t<double>(a, r, st) : merge_split_t<float>(a, r, st);
}

// Backward route of each query from its saved denominator (caller units); candidates are
// then settled by the same nearest-distance check as in the forward.
template <typename T>
__global__ __launch_bounds__(kWG) void k_flags_from_den(const double* __restrict__ den, int64_t m,
                                                        const double* __restrict__ hdr,
                                                        uint8_t* __restrict__ flag, int* __restrict__ hint,
                                                        int* __restrict__ list,
                                                        unsigned long long* __restrict__ minb) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * kWG + threadIdx.x;
  uint8_t r = F_FP32;
  if (i < m) flag[i] = r = route_of(den[i], hdr, true);
  append_candidates(r == F_CANDIDATE, i, hint, list, minb, min_bits(infT<T>()));
}

hipError_t flags_from_den(const double* den, const RouteArgs& r, bool f64, hipStream_t st) {
  dim3 grid(static_cast<unsigned>((r.m + kWG - 1) / kWG));
  if (f64)
    hipLaunchKernelGGL(k_flags_from_den<double>, grid, dim3(kWG), 0, st, den, r.m, r.hdr, r.route, r.hint, r.list,
                       r.minb);
  else
    hipLaunchKernelGGL(k_flags_from_den<float>, grid, dim3(kWG), 0, st, den, r.m, r.hdr, r.route, r.hint, r.list,
                       r.minb);
  return hipGetLastError();
}

// ---- Settling: every candidate gets its route from its minimum, and the F_FP64 queries are
// listed in ascending order.  Thread t of a workgroup owns 16 consecutive queries.  Up to
// kSettleOne queries one workgroup does it all (one launch, 2.3 us at 1,000 or 10,240 queries);
// beyond, one pass settles and counts per kCountBlock queries, and a second lists, each
// workgroup adding the counts before its own (a scan kernel where these are too many). ----
constexpr int kOwn = 16;
constexpr int kSettleWG = 1024;
constexpr int64_t kSettleOne = 4 * kOwn * kSettleWG;
constexpr int kSettlePrefix = 4096;  // most blocks whose counts a workgroup adds up itself

// Settles the thread's queries [i, i + 16); returns the mask of those routed to FP64.
template <typename T>
__device__ __forceinline__ unsigned settle_own(uint8_t* __restrict__ route, int64_t i, int64_t m,
                                               const double* __restrict__ hdr,
                                               const unsigned long long* __restrict__ minb) {
  unsigned mask = 0;
  if (i + kOwn <= m) {  // the route array is 256-byte aligned and i a multiple of 16
    const uint4 w = *reinterpret_cast<const uint4*>(route + i);
    if ((w.x | w.y | w.z | w.w) == 0u) return 0u;  // all F_FP32
  }
  for (int u = 0; u < kOwn; ++u) {
    if (i + u >= m) break;
    const uint8_t r = route[i + u];
    if (r == F_FP32) continue;
    uint8_t s = r;
    if (r == F_CANDIDATE) {
      s = settle_route<T>(r, minb[i + u], hdr);
      route[i + u] = s;
    }
    if (s == F_FP64) mask |= 1u << u;
  }
  return mask;
}

// Exclusive prefix of c over the NT threads of a workgroup and their total.
template <int NT>
__device__ __forceinline__ int block_prefix(int c, int* __restrict__ wsum, int& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int v = c;
#pragma unroll
  for (int x = 1; x < 64; x <<= 1) {
    const int up = __shfl_up(v, x);
    v += lane >= x ? up : 0;
  }
  if (lane == 63) wsum[wave] = v;
  __syncthreads();
  int before = 0;
  total = 0;
  for (int w = 0; w < NT / 64; ++w) {
    before += w < wave ? wsum[w] : 0;
    total += wsum[w];
  }
  __syncthreads();
  return before + v - c;
}

template <typename T>
__global__ __launch_bounds__(kSettleWG) void k_settle_one(uint8_t* __restrict__ route, int64_t m,
                                                          const double* __restrict__ hdr,
                                                          const unsigned long long* __restrict__ minb,
                                                          int* __restrict__ list, int* __restrict__ count) {
  __shared__ int wsum[kSettleWG / 64];
  int at = 0;
  for (int64_t base = 0; base < m; base += kOwn * kSettleWG) {
    const int64_t i = base + static_cast<int64_t>(threadIdx.x) * kOwn;
    const unsigned mask = i < m ? settle_own<T>(route, i, m, hdr, minb) : 0u;
    if (!__syncthreads_or(mask != 0u)) continue;
    int total;
    int pos = at + block_prefix<kSettleWG>(__popc(mask), wsum, total);
    for (unsigned k = mask; k; k &= k - 1) list[pos++] = static_cast<int>(i) + __ffs(k) - 1;
    at += total;
  }
  if (threadIdx.x == 0) *count = at;
}

template <typename T>
__global__ __launch_bounds__(kWG) void k_settle_count(uint8_t* __restrict__ route, int64_t m,
                                                      const double* __restrict__ hdr,
                                                      const unsigned long long* __restrict__ minb,
                                                      int* __restrict__ bcnt) {
  __shared__ int wsum[kWG / 64];
  const int64_t i = static_cast<int64_t>(blockIdx.x) * kCountBlock + threadIdx.x * kOwn;
  const unsigned mask = i < m ? settle_own<T>(route, i, m, hdr, minb) : 0u;
  int total;
  block_prefix<kWG>(__popc(mask), wsum, total);
  if (threadIdx.x == 0) bcnt[blockIdx.x] = total;
}

// Lists block b's F_FP64 queries after those of the blocks before it; the last block writes
// the total.  (The candidates are settled: the routes hold F_FP32 and F_FP64 only.)
__global__ __launch_bounds__(kWG) void k_settle_list(const uint8_t* __restrict__ route, int64_t m,
                                                     const int* __restrict__ bcnt, int nb,
                                                     int* __restrict__ list, int* __restrict__ count) {
  __shared__ int wsum[kWG / 64];
  const int own = bcnt[blockIdx.x];
  const bool last = static_cast<int>(blockIdx.x) == nb - 1;
  if (own == 0 && !last) return;
  int before = 0;
  for (int b = threadIdx.x; b < static_cast<int>(blockIdx.x); b += kWG) before += bcnt[b];
  int base;
  block_prefix<kWG>(before, wsum, base);
  if (last && threadIdx.x == 0) *count = base + own;
  if (own == 0) return;
  const int64_t i = static_cast<int64_t>(blockIdx.x) * kCountBlock + threadIdx.x * kOwn;
  int c = 0;
  for (int u = 0; u < kOwn; ++u) c += i + u < m && route[i + u] == F_FP64 ? 1 : 0;
  int total;
  int pos = base + block_prefix<kWG>(c, wsum, total);
  for (int u = 0; u < kOwn; ++u)
    if (i + u < m && route[i + u] == F_FP64) list[pos++] = static_cast<int>(i + u);
}

// ---- Deterministic, order-preserving compaction of the queries whose route byte equals
// `want` into an index list.  Block b owns bytes [b*4096, (b+1)*4096); thread t owns 16
// consecutive bytes of it. ----
constexpr int kPerThread = kCountBlock / kWG;

__device__ __forceinline__ int local_count(const uint8_t* __restrict__ flag, int64_t m,
                                           int64_t base, uint8_t want) {
  int c = 0;
#pragma unroll
  for (int u = 0; u < kPerThread; ++u) {
    const int64_t i = base + u;
    if (i < m) c += flag[i] == want ? 1 : 0;
  }
  return c;
}

__global__ __launch_bounds__(kWG) void k_count(const uint8_t* __restrict__ flag, int64_t m,
                                               uint8_t want, int* __restrict__ bcnt) {
  __shared__ double red[kWG];
  const int64_t base = static_cast<int64_t>(blockIdx.x) * kCountBlock + threadIdx.x * kPerThread;
  const double c = block_sum(static_cast<double>(local_count(flag, m, base, want)), red);
  if (threadIdx.x == 0) bcnt[blockIdx.x] = static_cast<int>(c);
}

// Exclusive scan of the block counts in place (single workgroup), total into *count.
__global__ __launch_bounds__(kWG) void k_scan(int* __restrict__ bcnt, int nb,
                                              int* __restrict__ count) {
  __shared__ int buf[kWG];
  __shared__ int carry;
  const int t = threadIdx.x;
  if (t == 0) carry = 0;
  __syncthreads();
  for (int base = 0; base < nb; base += kWG) {
    const int v = (base + t < nb) ? bcnt[base + t] : 0;
    buf[t] = v;
    __syncthreads();
    for (int off = 1; off < kWG; off <<= 1) {  // Hillis-Steele inclusive scan
      const int add = t >= off ? buf[t - off] : 0;
      __syncthreads();
      buf[t] += add;
      __syncthreads();
    }
    if (base + t < nb) bcnt[base + t] = carry + buf[t] - v;
    __syncthreads();
    if (t == kWG - 1) carry += buf[t];
    __syncthreads();
  }
  if (t == 0) *count = carry;
}

__global__ __launch_bounds__(kWG) void k_emit(const uint8_t* __restrict__ flag, int64_t m,
                                              uint8_t want, const int* __restrict__ boff,
                                              int* __restrict__ list) {
  __shared__ int buf[kWG];
  const int t = threadIdx.x;
  const int64_t base = static_cast<int64_t>(blockIdx.x) * kCountBlock + t * kPerThread;
  const int c = local_count(flag, m, base, want);
  buf[t] = c;
  __syncthreads();
  for (int off = 1; off < kWG; off <<= 1) {
    const int add = t >= off ? buf[t - off] : 0;
    __syncthreads();
    buf[t] += add;
    __syncthreads();
  }
  int pos = boff[blockIdx.x] + buf[t] - c;
  for (int u = 0; u < kPerThread; ++u) {
    const int64_t i = base + u;
    if (i < m && flag[i] == want) list[pos++] = static_cast<int>(i);
  }
}

template <typename T>
static hipError_t settle_t(const RouteArgs& r, hipStream_t st) {
  if (r.m <= kSettleOne) {
    hipLaunchKernelGGL((k_settle_one<T>), dim3(1), dim3(kSettleWG), 0, st, r.route, r.m, r.hdr, r.minb, r.list,
                       r.hint);
    return hipGetLastError();
  }
  const int nb = static_cast<int>((r.m + kCountBlock - 1) / kCountBlock);
  hipLaunchKernelGGL((k_settle_count<T>), dim3(nb), dim3(kWG), 0, st, r.route, r.m, r.hdr, r.minb, r.bcnt);
  if (nb <= kSettlePrefix) {
    hipLaunchKernelGGL(k_settle_list, dim3(nb), dim3(kWG), 0, st, r.route, r.m, r.bcnt, nb, r.list, r.hint);
  } else {
    hipLaunchKernelGGL(k_scan, dim3(1), dim3(kWG), 0, st, r.bcnt, nb, r.hint);
    hipLaunchKernelGGL(k_emit, dim3(nb), dim3(kWG), 0, st, r.route, r.m, static_cast<uint8_t>(F_FP64), r.bcnt,
                       r.list);
  }
  return hipGetLastError();
}

hipError_t settle(const RouteArgs& r, bool f64, hipStream_t st) {
  return f64 ? settle_t<double>(r, st) : settle_t<float>(r, st);
}

hipError_t compact_flags(const uint8_t* flag, int64_t m, int* bcnt, int* list, int* count,
                         uint8_t want, hipStream_t st) {
  const int nb = static_cast<int>((m + kCountBlock - 1) / kCountBlock);
  hipLaunchKernelGGL(k_count, dim3(nb), dim3(kWG), 0, st, flag, m, want, bcnt);
  hipLaunchKernelGGL(k_scan, dim3(1), dim3(kWG), 0, st, bcnt, nb, count);
  hipLaunchKernelGGL(k_emit, dim3(nb), dim3(kWG), 0, st, flag, m, want, bcnt, list);
  return hipGetLastError();
}

__global__ __launch_bounds__(kWG) void k_dp_final(const double* __restrict__ wg_dp, int nwg,
                                                  const double* __restrict__ slot_dp,
                                                  const int* __restrict__ count,
                                                  double* __restrict__ grad_p) {
  dp_final_block(wg_dp, nwg, slot_dp, *count, grad_p);
}

// ---- grid of the nearest-distance searches: geometry and gates, scan of the counts ----
// Geometry: square cells of side h = (largest box side) / (floor(ncell_max^(1/dim)) - 1),
// at least 2.5 times the near-coincidence distance (so the box q +- r' of the candidate
// check meets at most two cells per axis), hence at most ncell_max cells.
// Every workgroup also clears its part of the counts when the grid is used.  `ncand` is the
// number of candidates (mode 0).
__global__ __launch_bounds__(kWG) void k_grid_setup(double* __restrict__ hdr, int* __restrict__ hint,
                                                    const int* __restrict__ ncand, int dim, int64_t ncell_max,
                                                    int mode, int64_t mall, int* __restrict__ cnt) {
  const int64_t cand = mode == 1 ? mall : static_cast<int64_t>(*ncand);
  const bool use = cand > 0 && (mode == 1 || cand >= kGridMinCand);
  if (use)
    for (int64_t c = static_cast<int64_t>(blockIdx.x) * kWG + threadIdx.x; c <= ncell_max;
         c += static_cast<int64_t>(gridDim.x) * kWG)
      cnt[c] = 0;
  if (blockIdx.x != 0 || threadIdx.x != 0) return;
  hint[GI_FALLBACK] = 0;
  hint[GI_BRUTE] = use ? 0 : static_cast<int>(cand);
  hint[GI_GRID] = use ? static_cast<int>(cand) : 0;
  if (!use) return;
  double emax = 0.0;
  for (int k = 0; k < dim; ++k) emax = fmax(emax, hdr[H_BEXT + k]);
  int base = static_cast<int>(floor(pow(static_cast<double>(ncell_max), 1.0 / dim))) - 1;
  if (base < 1) base = 1;
  auto cells = [&](int b) {  // (b + 1)^dim
    int64_t c = 1;
    for (int k = 0; k < dim; ++k) c *= b + 1;
    return c;
  };
  while (base > 1 && cells(base) > ncell_max) --base;  // pow may round the root up
  double h = fmax(emax / base, 2.5 * sqrt(hdr[H_NEAR_R2]));
  if (!(h > 0.0) || !(h < __builtin_huge_val())) h = 1.0;
  hdr[H_GRID_H] = h;
  hdr[H_GRID_INVH] = 1.0 / h;
  for (int k = 0; k < 3; ++k) {
    int g = 1;
    if (k < dim) {
      const double c = floor(hdr[H_BEXT + k] / h) + 1.0;
      g = c < static_cast<double>(base + 1) ? static_cast<int>(c) : base + 1;
      if (g < 1) g = 1;
    }
    hdr[H_GRID_G + k] = static_cast<double>(g);
  }
}

__device__ __forceinline__ int64_t grid_ncell(const double* __restrict__ hdr) {
  return static_cast<int64_t>(hdr[H_GRID_G]) * static_cast<int64_t>(hdr[H_GRID_G + 1]) *
         static_cast<int64_t>(hdr[H_GRID_G + 2]);
}

constexpr int kScanPer = kGridScanBlock / kWG;  // cells per thread in the count scan

__global__ __launch_bounds__(kWG) void k_grid_blocksum(const int* __restrict__ cnt, const double* __restrict__ hdr,
                                                       const int* __restrict__ hint, int* __restrict__ bsum) {
  __shared__ double red[kWG];
  if (hint[GI_GRID] <= 0) {
    if (threadIdx.x == 0) bsum[blockIdx.x] = 0;
    return;
  }
  const int64_t ncell = grid_ncell(hdr);
  const int64_t base = static_cast<int64_t>(blockIdx.x) * kGridScanBlock + threadIdx.x * kScanPer;
  long long c = 0;
  for (int u = 0; u < kScanPer; ++u)
    if (base + u < ncell) c += cnt[base + u];
  const double tot = block_sum(static_cast<double>(c), red);
  if (threadIdx.x == 0) bsum[blockIdx.x] = static_cast<int>(tot);
}

// start[c] = exclusive prefix of the counts; the counts become scatter cursors (= start);
// start[ncell] = the number of points.
__global__ __launch_bounds__(kWG) void k_grid_offsets(int* __restrict__ cnt, const double* __restrict__ hdr,
                                                      const int* __restrict__ hint, const int* __restrict__ boff,
                                                      int* __restrict__ start) {
  __shared__ int buf[kWG];
  if (hint[GI_GRID] <= 0) return;
  const int64_t ncell = grid_ncell(hdr);
  const int t = threadIdx.x;
  const int64_t base = static_cast<int64_t>(blockIdx.x) * kGridScanBlock + t * kScanPer;
  int loc[kScanPer];
  int c = 0;
  for (int u = 0; u < kScanPer; ++u) {
    loc[u] = base + u < ncell ? cnt[base + u] : 0;
    c += loc[u];
  }
  buf[t] = c;
  __syncthreads();
  for (int off = 1; off < kWG; off <<= 1) {  // Hillis-Steele inclusive scan
    const int add = t >= off ? buf[t - off] : 0;
    __syncthreads();
    buf[t] += add;
    __syncthreads();
  }
  int pos = boff[blockIdx.x] + buf[t] - c;
  for (int u = 0; u < kScanPer; ++u) {
    const int64_t cell = base + u;
    if (cell < ncell) {
      start[cell] = pos;
      cnt[cell] = pos;
      pos += loc[u];
      if (cell == ncell - 1) start[ncell] = pos;
    }
  }
}

hipError_t grid_setup(const GridArgs& a, int mode, const int* ncand, hipStream_t st) {
  int64_t blocks = (a.ncell_max + kWG) / kWG;
  if (blocks > 1024) blocks = 1024;
  hipLaunchKernelGGL(k_grid_setup, dim3(static_cast<unsigned>(blocks)), dim3(kWG), 0, st, const_cast<double*>(a.hdr),
                     a.hint, ncand, a.dim, a.ncell_max, mode, a.m, a.cnt);
  return hipGetLastError();
}

hipError_t grid_scan(const GridArgs& a, hipStream_t st) {
  const int nb = static_cast<int>((a.ncell_max + kGridScanBlock - 1) / kGridScanBlock);
  hipLaunchKernelGGL(k_grid_blocksum, dim3(nb), dim3(kWG), 0, st, a.cnt, a.hdr, a.hint, a.bsum);
  hipLaunchKernelGGL(k_scan, dim3(1), dim3(kWG), 0, st, a.bsum, nb, a.hint + GI_TOTAL);
  hipLaunchKernelGGL(k_grid_offsets, dim3(nb), dim3(kWG), 0, st, a.cnt, a.hdr, a.hint, a.bsum, a.start);
  return hipGetLastError();
}

hipError_t bwd_merge(const BwdArgs& a, bool query, bool data, bool x, bool f64, hipStream_t st) {
  if (f64)
    return a.dim == 3 ? launch_bwd_merge<double, 3>(a, query, data, x, st)
                      : launch_bwd_merge<double, 2>(a, query, data, x, st);
  return a.dim == 3 ? launch_bwd_merge<float, 3>(a, query, data, x, st)
                    : launch_bwd_merge<float, 2>(a, query, data, x, st);
}

hipError_t dp_final(const double* wg_dp, int nwg, const double* slot_dp, const int* count,
                    double* grad_p, hipStream_t st) {
  hipLaunchKernelGGL(k_dp_final, dim3(1), dim3(kWG), 0, st, wg_dp, nwg, slot_dp, count, grad_p);
  return hipGetLastError();
}

}  // namespace idw

namespace idw {

// Zero fill with a kernel (a memset node is never recorded into a captured graph).
__global__ __launch_bounds__(kWG) void k_fill_zero(uint32_t* __restrict__ p, int64_t words) {
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * kWG + threadIdx.x; i < words;
       i += static_cast<int64_t>(gridDim.x) * kWG)
    p[i] = 0u;
}

hipError_t fill_zero(void* p, size_t bytes, hipStream_t st) {
  const int64_t words = static_cast<int64_t>(bytes / 4);
  if (words == 0) return hipSuccess;
  int64_t blocks = (words + kWG - 1) / kWG;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_fill_zero, dim3(static_cast<unsigned>(blocks)), dim3(kWG), 0, st,
                     static_cast<uint32_t*>(p), words);
  return hipGetLastError();
}

}  // namespace idw
