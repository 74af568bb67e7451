// Forward sweep of Shepard IDW (Section 2.1, Eq. 1) for gfx950.
//
// One workgroup = 256 lanes x Q queries held in registers.  Data points are streamed
// through LDS in tiles of kTile records (double-buffered: the global loads of tile t+1 are
// in flight while tile t is consumed), and every record is broadcast from LDS to all lanes
// of the wavefront (the shared-memory tiling of Section 4.2, re-derived for wave64).  Each
// lane accumulates sum w*z and sum w for its queries in plain arithmetic over 64-record
// blocks and adds every block sum into an FP64 running sum (a TwoSum pair in the FP64
// sweep), so the sum error is that of a 64-term sum, not of an n-term one.  The ratio is
// taken in FP64.  A query whose
// denominator exceeds the near-coincidence threshold (or is not finite) is flagged for the
// FP64 fix-up kernel, which recomputes it exactly, including the exact-hit rule.
#pragma once

#include <math.h>

#include <type_traits>

#include "idw_device.hpp"
#include "idw_launch.hpp"
#include "idw_phase.hpp"

namespace idw {

__device__ __forceinline__ float fmaT(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fmaT(double a, double b, double c) { return fma(a, b, c); }

__device__ __forceinline__ float maxT(float a, float b) { return fmaxf(a, b); }
__device__ __forceinline__ double maxT(double a, double b) { return fmax(a, b); }

template <typename T>
__device__ __forceinline__ T infT() {
  return __builtin_huge_valf();
}
template <>
__device__ __forceinline__ double infT<double>() {
  return __builtin_huge_val();
}

// Squared distance from query coordinates q to a staged record d.
template <typename T, int DIM>
__device__ __forceinline__ T sqdist(const T (&q)[3], const P4<T>& d) {
  const T dx = q[0] - d.x;
  const T dy = q[1] - d.y;
  T r2 = dx * dx;
  r2 = fmaT(dy, dy, r2);
  if constexpr (DIM == 3) {
    const T dz = q[2] - d.z;
    r2 = fmaT(dz, dz, r2);
  }
  return r2;
}

// Stage one record into LDS form: coordinates scaled by s; {x, y, v, 0} or {x, y, z, v}.
template <typename T, int DIM>
__device__ __forceinline__ P4<T> stage(const T (&c)[3], T v, T s) {
  P4<T> r;
  r.x = c[0] * s;
  r.y = c[1] * s;
  if constexpr (DIM == 3) {
    r.z = c[2] * s;
    r.w = v;
  } else {
    r.z = v;
    r.w = T(0);
  }
  return r;
}

// Kahan-compensated running sum in the working precision, updated on every pair: s carries
// the sum and e the rounding error lost so far (s + e is the compensated sum).
template <typename T>
struct KahanSum {
  T s, e;
  __device__ __forceinline__ void zero() { s = e = T(0); }
  __device__ __forceinline__ void add(T x) {
    const T y = x + e;
    const T t = s + y;
    e = y - (t - s);
    s = t;
  }
  __device__ __forceinline__ double value() const { return static_cast<double>(s) + static_cast<double>(e); }
};

// Consume one LDS tile: for each of the lane's Q queries, accumulate w*z and w.
// KH = false: plain sums over 64-record blocks, each added into a BlockSum.
// KH = true: a Kahan step on every pair into a KahanSum (about 3 more VALU operations per
// accumulator and pair; the accuracy variant).
// REL = true: relative weights, the squared distance multiplied by the query's sigma
// before the weight is taken (one more multiply per pair).
// Records [begin, end) of the tile, begin a multiple of 64: a full tile (FULL), whole 64-record
// blocks, or with TAIL a last block of fewer.  Padding records are never visited, so that no
// weight of theirs, however small, reaches the denominator.
template <typename T, int DIM, int PM, int Q, bool DIAG, int UNR, bool KH = false, bool REL = false,
          bool TAIL = false, bool FULL = false, int DEG = 10, typename Acc>
__device__ __forceinline__ void fwd_tile(const RecTile<T, DIM, kTile>& tl, int64_t jt, int begin, int end,
                                         const T (&qc)[Q][3], const int64_t (&qi)[Q], T nhp,
                                         const T (&sg)[Q], Acc (&num)[Q], Acc (&den)[Q]) {
  constexpr int CH = 64;
  const int lim = FULL ? kTile : end;
  if constexpr (KH) {
#pragma unroll UNR
    for (int jj = begin; jj < lim; ++jj) {
      const P4<T> d = tl.get(jj);
      const T dv = (DIM == 3) ? d.w : d.z;
#pragma unroll
      for (int k = 0; k < Q; ++k) {
        T r2 = sqdist<T, DIM>(qc[k], d);
        if constexpr (REL) r2 *= sg[k];
        T w = weight_sweep<PM, DEG>(r2, nhp);
        if constexpr (DIAG) {
          if (jt + jj == qi[k]) w = T(0);
        }
        num[k].add(w * dv);
        den[k].add(w);
      }
    }
    return;
  }
  auto block = [&](int c0) {
    T an[Q], ad[Q];
#pragma unroll
    for (int k = 0; k < Q; ++k) {
      an[k] = T(0);
      ad[k] = T(0);
    }
    const int ce = TAIL ? ((lim - c0) < CH ? (lim - c0) : CH) : CH;
#pragma unroll UNR
    for (int jj = 0; jj < ce; ++jj) {
      const P4<T> d = tl.get(c0 + jj);
      const T dv = (DIM == 3) ? d.w : d.z;
#pragma unroll
      for (int k = 0; k < Q; ++k) {
        T r2 = sqdist<T, DIM>(qc[k], d);
        if constexpr (REL) r2 *= sg[k];
        T w = weight_sweep<PM, DEG>(r2, nhp);
        if constexpr (DIAG) {
          if (jt + c0 + jj == qi[k]) w = T(0);
        }
        an[k] = fmaT(w, dv, an[k]);
        ad[k] += w;
      }
    }
#pragma unroll
    for (int k = 0; k < Q; ++k) {
      num[k].add(an[k]);
      den[k].add(ad[k]);
    }
  };
  // FP64 general p goes block by block; unrolled over the tile, the compiler keeps every
  // 64-record block's partial sums live until the tile's end, which differs by at most 2%
  // either way for the other FP64 weights.
  if constexpr (PM == PM_GEN || !FULL) {
#pragma unroll 1
    for (int c0 = begin; c0 < lim; c0 += CH) block(c0);
  } else {
    for (int c0 = 0; c0 < lim; c0 += CH) block(c0);
  }
}

// Whole 64-record blocks [0, end) in FP32 without a self pair: groups of 4 records, whose 4 Q weights form one
// run of transcendentals (idw_phase.hpp).  The same operations in the same order per query
// as fwd_tile, so the same bits.  Bound by instruction issue: 6 plain instructions and a
// reciprocal per pair at p = 2, 20.6 cycles with the waves in step.  Against records read one
// by one with the transcendentals between the plain instructions (3 waves per SIMD): 1M x 1M
// p = 2 177 -> 154 ms; 3-D mixture, p = 2.5, 80.3 -> 66.8 ms; per-pair Kahan sums, p = 3,
// 102,400 x 99,991, 3.95 -> 2.75 ms; the 64 batched instances 58.7 -> 45.0 ms.  Unrolled over
// the whole 64-record block instead of 4 groups: within 0.3% in 2-D, 2-4% slower in 3-D.
template <int DIM, int PM, int Q, bool KH, bool REL, typename Acc>
__device__ __forceinline__ void fwd_tile_run(const RecTile<float, DIM, kTile>& tl, int end,
                                             const float (&qc)[Q][3], float nhp, const float (&sg)[Q], Acc (&num)[Q], Acc (&den)[Q]) {
  constexpr int CH = 64, G = 4;
#pragma unroll 1
  for (int c0 = 0; c0 < end; c0 += CH) {
    float an[Q], ad[Q];
#pragma unroll
    for (int k = 0; k < Q; ++k) an[k] = ad[k] = 0.f;
#pragma unroll 4
    for (int j = 0; j < CH; j += G) {
      RecGroup<DIM, G> d;
      d.load(tl, c0 + j);
      float w[G * Q];
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int k = 0; k < Q; ++k) {
          w[g * Q + k] = d.r2(qc[k], g);
          if constexpr (REL) w[g * Q + k] *= sg[k];
        }
      weight_run<PM>(w, nhp);
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int k = 0; k < Q; ++k) {
          if constexpr (KH) {
            num[k].add(w[g * Q + k] * d.v[g]);
            den[k].add(w[g * Q + k]);
          } else {
            an[k] = fmaf(w[g * Q + k], d.v[g], an[k]);
            ad[k] += w[g * Q + k];
          }
        }
    }
    if constexpr (!KH) {
#pragma unroll
      for (int k = 0; k < Q; ++k) {
        num[k].add(an[k]);
        den[k].add(ad[k]);
      }
    }
  }
}

// Whole 64-record blocks [0, end) in FP64 for the reciprocal weights (p = 2 and 4), without a
// self pair: four records' reciprocals from one (rcp64_w4).  Bound by FP64 issue: 8 instructions
// and a quarter of an estimate, about 44 cycles per pair and wave against 51.5 with a reciprocal
// each.  The next group's records are read ahead.  Calls of 131,072 x 131,072: p = 2 5.75 -> 5.16
// ms, p = 4 6.22 -> 5.62; 3-D 6.72 -> 6.30 and 7.24 -> 6.84.
template <int DIM, int PM, int Q, typename Acc>
__device__ __forceinline__ void fwd_tile_rcp4(const RecTile<double, DIM, kTile>& tl, int end,
                                              const double (&qc)[Q][3], Acc (&num)[Q], Acc (&den)[Q]) {
  static_assert(PM == PM_2 || PM == PM_4, "reciprocal weights");
  constexpr int CH = 64, G = 4;
#pragma unroll 1
  for (int c0 = 0; c0 < end; c0 += CH) {
    double an[Q], ad[Q];
#pragma unroll
    for (int k = 0; k < Q; ++k) an[k] = ad[k] = 0.0;
    P4<double> d[G];
#pragma unroll
    for (int g = 0; g < G; ++g) d[g] = tl.get(c0 + g);
#pragma unroll 2
    for (int j = 0; j < CH; j += G) {
      double v[G], w[Q][G];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        v[g] = DIM == 3 ? d[g].w : d[g].z;
#pragma unroll
        for (int k = 0; k < Q; ++k) w[k][g] = sqdist<double, DIM>(qc[k], d[g]);
      }
#pragma unroll
      for (int g = 0; g < G; ++g) d[g] = tl.get(c0 + ((j + G + g) & (CH - 1)));  // the next group
#pragma unroll
      for (int k = 0; k < Q; ++k) {
        rcp64_w4(w[k]);
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const double t = PM == PM_4 ? w[k][g] * w[k][g] : w[k][g];
          an[k] = fma(t, v[g], an[k]);
          ad[k] += t;
        }
      }
    }
#pragma unroll
    for (int k = 0; k < Q; ++k) {
      num[k].add(an[k]);
      den[k].add(ad[k]);
    }
  }
}

// Finalise one query from its (num, den) in scaled units.
template <typename T>
__device__ __forceinline__ void fwd_finish(int64_t i, double num, double den, const double* hdr,
                                           T* __restrict__ out_z, double* __restrict__ out_den,
                                           uint8_t* __restrict__ out_flag) {
  out_z[i] = static_cast<T>(num / den);
  if (out_den) out_den[i] = den * hdr[H_DEN_UNIT];
  out_flag[i] = route_of(den, hdr, false);
}

// Register-blocking and occupancy knobs of a sweep kernel: UNR = unroll of the FP64
// per-record loop, WMIN / WMAX = waves per SIMD the register allocation aims at.  FP32: an
// even number of waves (idw_phase.hpp), 4, or 2 for the 8-query builds.  FP64 (1M x 1M): Q = 2
// is faster than 4 for general p (1036 -> 957 ms) and within 1.2% elsewhere; general p is
// faster 2-deep (p = 1.7: 931 -> 894 ms), the others 4-deep (p = 2: 359 against 364 ms).
template <typename T, int Q, int PM = PM_GEN>
struct SweepTune {
  static constexpr bool kF32 = sizeof(T) == 4;
  static constexpr int UNR = PM == PM_GEN ? 2 : 4;
  static constexpr int WMIN = kF32 ? (Q >= 8 ? 2 : 4) : 1;
  static constexpr int WMAX = kF32 ? WMIN : 8;
  static constexpr int DEG = 10;  // last power of the FP64 general-p series
};
// |p / 2| <= kPowLow (p = 1.7, 65,536 x 262,144: 137 cycles per pair and wave with the series
// through r^10 and a comparison for zero, 131 without the comparison, 108 through r^6).
template <int Q>
struct SweepTuneLow : SweepTune<double, Q, PM_GEN> {
  static constexpr int DEG = 6;
};

// REL: relative weights; rmin holds each query's nearest squared distance (FP32 bits,
// scaled units, from k_near_check over all queries) and the sums leave the kernel
// multiplied by sigma^(p/2), i.e. in scaled units like those of the direct form.
template <typename T, int DIM, int L, int PM, int Q, bool KH = false, bool REL = false,
          typename Tune = SweepTune<T, Q, PM>>
__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(Tune::WMIN, Tune::WMAX))) void k_fwd_sweep(DevPts data, int64_t n, DevPts query, int64_t m,
                                                   int64_t chunk, int split, T nhp, unsigned flags,
                                                   const double* __restrict__ hdr,
                                                   T* __restrict__ out_z,
                                                   double* __restrict__ out_den,
                                                   uint8_t* __restrict__ out_flag,
                                                   double2* __restrict__ part,
                                                   const unsigned long long* __restrict__ rmin,
                                                   double p) {
  __shared__ RecTile<T, DIM, kTile> tile[2];
  const int tid = threadIdx.x;
  const int64_t q0 = static_cast<int64_t>(blockIdx.x) * (kWG * Q);
  const int64_t jb = static_cast<int64_t>(blockIdx.y) * chunk;
  const int64_t je = (jb + chunk < n) ? jb + chunk : n;
  const T s = static_cast<T>(hdr[H_SCALE]);

  T qc[Q][3], sg[Q];
  double fs[Q];
  int64_t qi[Q];
#pragma unroll
  for (int k = 0; k < Q; ++k) {
    qi[k] = q0 + tid + static_cast<int64_t>(k) * kWG;
    T c[3] = {T(0), T(0), T(0)};
    sg[k] = T(1);
    fs[k] = 1.0;
    if (qi[k] < m) {
      Loader<T, DIM, L>::query(query, qi[k], c);
      if constexpr (REL) {
        float sgf = 1.0f;
        rel_from_min(__builtin_bit_cast(float, static_cast<unsigned int>(rmin[qi[k]])), p, sgf,
                     fs[k]);
        sg[k] = static_cast<T>(sgf);
      }
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) qc[k][d] = c[d] * s;
  }
  using Acc = std::conditional_t<KH, KahanSum<T>, BlockSum<T>>;
  Acc nacc[Q], dacc[Q];
#pragma unroll
  for (int k = 0; k < Q; ++k) {
    nacc[k].zero();
    dacc[k].zero();
  }

  // The tables' weight of a NaN distance is 0: a NaN coordinate is found here, once per record
  // (a comparison per pair cost 6 of 137 cycles).
  constexpr bool kSeekNan = sizeof(T) == 8 && PM == PM_GEN;
  bool bad = false;
  T rc[2][3], rv[2];
  auto fetch = [&](int t) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int64_t j = jb + static_cast<int64_t>(t) * kTile + u * kWG + tid;
      if (j < je) {
        Loader<T, DIM, L>::data(data, j, rc[u], rv[u]);
        if constexpr (kSeekNan) {
#pragma unroll
          for (int d = 0; d < DIM; ++d) bad |= rc[u][d] != rc[u][d];
        }
      } else {  // padding record: far away, zero value -> weight (near) 0
        rc[u][0] = rc[u][1] = rc[u][2] = padT<T>();
        rv[u] = T(0);
      }
    }
  };
  auto put = [&](int b) {
#pragma unroll
    for (int u = 0; u < 2; ++u) tile[b].put(u * kWG + tid, stage<T, DIM>(rc[u], rv[u], s));
  };

  const int ntiles = static_cast<int>((je - jb + kTile - 1) / kTile);
  const bool excl = (flags & 1u) != 0;
  if constexpr (sizeof(T) == 8 && PM == PM_GEN) pow_table_init(nhp);  // FP64 weight tables (synchronised below)
  fetch(0);
  put(0);
  __syncthreads();
  for (int t = 0; t < ntiles; ++t) {
    if (t + 1 < ntiles) fetch(t + 1);
    const int64_t jt = jb + static_cast<int64_t>(t) * kTile;
    const int cnt = static_cast<int>((je - jt) < kTile ? (je - jt) : kTile);
    const bool diag = excl && jt < q0 + kWG * Q && q0 < jt + kTile;
    const auto& tl = tile[t & 1];
    if (diag) {
      fwd_tile<T, DIM, PM, Q, true, 1, KH, REL, true>(tl, jt, 0, cnt, qc, qi, nhp, sg, nacc, dacc);
    } else {
      const int whole = cnt & ~63;
      if constexpr (sizeof(T) == 4) {
        fwd_tile_run<DIM, PM, Q, KH, REL>(tl, whole, qc, nhp, sg, nacc, dacc);
      } else if constexpr (PM == PM_2 || PM == PM_4) {
        fwd_tile_rcp4<DIM, PM, Q>(tl, whole, qc, nacc, dacc);
      } else if (whole == kTile) {
        fwd_tile<T, DIM, PM, Q, false, Tune::UNR, KH, REL, false, true, Tune::DEG>(tl, jt, 0, kTile, qc, qi, nhp, sg,
                                                                                   nacc, dacc);
      } else if (whole > 0) {
        fwd_tile<T, DIM, PM, Q, false, Tune::UNR, KH, REL, false, false, Tune::DEG>(tl, jt, 0, whole, qc, qi, nhp, sg,
                                                                                    nacc, dacc);
      }
      if (whole < cnt)
        fwd_tile<T, DIM, PM, Q, false, 1, KH, REL, true>(tl, jt, whole, cnt, qc, qi, nhp, sg, nacc, dacc);
    }
    if (t + 1 < ntiles) put((t + 1) & 1);
    __syncthreads();
  }

  if constexpr (kSeekNan) bad = __syncthreads_or(bad);
#pragma unroll
  for (int k = 0; k < Q; ++k) {
    if (qi[k] < m) {
      double num = nacc[k].value();
      double den = dacc[k].value();
      if (kSeekNan && bad) den = __builtin_nan("");  // to the FP64 fix-up
      if constexpr (REL) {
        num *= fs[k];
        den *= fs[k];
      }
      if (split == 1)
        fwd_finish<T>(qi[k], num, den, hdr, out_z, out_den, out_flag);
      else
        part[static_cast<int64_t>(blockIdx.y) * m + qi[k]] = make_double2(num, den);
    }
  }
}

// Nearest-distance check of the candidate queries (route F_CANDIDATE, collected in a list by
// append_candidates, which also sets their minima to +inf):
//  k_near_check  takes work items (block of kWG * Q candidates, data chunk) in turn: the
//                data chunk goes through LDS tiles as in the forward sweep, each query keeps
//                its smallest squared distance in scaled units (the leave-one-out self pair
//                excluded) and folds it into its minimum by an integer atomic min on the
//                bits of the non-negative value (order-independent, so deterministic).  The
//                data range is cut into as many chunks as keep about kNearGrid workgroups
//                busy when the candidates are few, none when they fill the grid;
//  settle_route  (the settling kernels) gives a candidate with a data point closer than 1e-6
//                of the extent F_FP64, the others F_FP32 (their sweep results stand).
// 5 VALU operations per pair (2 sub, mul + fma, min).  k_near_init sets minima to +inf where
// every query, or a list of them, needs its nearest distance.
constexpr int kNearGrid = 1024;      // workgroups of the nearest-distance check
// Fewest data points per chunk: one tile.  A few candidates (the common case from p = 2 on)
// make one block, whose time is that of its chunk (131,072 or 1M points: 480 us with chunks of
// 8192 points).
constexpr int kNearMinChunk = kTile;

template <typename T>
__device__ __forceinline__ unsigned long long min_bits(T v) {  // v >= 0: bits order as values
  if constexpr (sizeof(T) == 4)
    return static_cast<unsigned long long>(__builtin_bit_cast(unsigned int, v));
  else
    return __builtin_bit_cast(unsigned long long, v);
}
template <typename T>
__device__ __forceinline__ T from_min_bits(unsigned long long b) {
  if constexpr (sizeof(T) == 4)
    return __builtin_bit_cast(float, static_cast<unsigned int>(b));
  else
    return __builtin_bit_cast(double, b);
}

// With list == nullptr every query 0..mall-1 takes part (the relative-weight forward needs
// the nearest distance of each query); otherwise the *count queries of list.
template <typename T>
__global__ __launch_bounds__(kWG) void k_near_init(const int* __restrict__ list, const int* __restrict__ count,
                                                   int64_t mall, unsigned long long* __restrict__ minb) {
  const int64_t cnt = list ? static_cast<int64_t>(*count) : mall;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * kWG + threadIdx.x; i < cnt;
       i += static_cast<int64_t>(gridDim.x) * kWG)
    minb[list ? list[i] : i] = min_bits(infT<T>());
}

// Route of a query after the nearest-distance check.
template <typename T>
__device__ __forceinline__ uint8_t settle_route(uint8_t r, unsigned long long minb, const double* __restrict__ hdr) {
  if (r != F_CANDIDATE) return r;
  return from_min_bits<T>(minb) < static_cast<T>(hdr[H_NEAR_R2]) ? F_FP64 : F_FP32;
}

template <typename T, int DIM, int L, int Q, bool EXCL>
__global__ __launch_bounds__(kWG) void k_near_check(DevPts data, int64_t n, DevPts query,
                                                    const int* __restrict__ list,
                                                    const int* __restrict__ count,
                                                    const int* __restrict__ list2,
                                                    const int* __restrict__ count2, int64_t mall,
                                                    const double* __restrict__ hdr,
                                                    unsigned long long* __restrict__ minb) {
  __shared__ P4<T> tile[2][kTile];
  int64_t cnt = list ? static_cast<int64_t>(*count) : mall;
  if (cnt == 0 && list2) {  // a second list where the first is empty
    list = list2;
    cnt = *count2;
  }
  const int tid = threadIdx.x;
  const T s = static_cast<T>(hdr[H_SCALE]);
  constexpr int64_t kQB = static_cast<int64_t>(kWG) * Q;
  const int64_t nblk = (cnt + kQB - 1) / kQB;
  if (nblk == 0) return;
  // data chunks per candidate block: fill the grid when the candidates are few
  int64_t C = kNearGrid / nblk;
  const int64_t cmax = (n + kNearMinChunk - 1) / kNearMinChunk;
  if (C > cmax) C = cmax;
  if (C < 1) C = 1;
  const int64_t len = ((n + C - 1) / C + kTile - 1) / kTile * kTile;
  C = (n + len - 1) / len;
  const int64_t total = nblk * C;
  for (int64_t w = blockIdx.x; w < total; w += gridDim.x) {  // uniform over the workgroup
    const int64_t b0 = (w / C) * kQB;
    const int64_t jb = (w % C) * len;
    const int64_t je = jb + len < n ? jb + len : n;
    T qc[Q][3], mn[Q];
    int64_t qi[Q];
#pragma unroll
    for (int k = 0; k < Q; ++k) {
      const int64_t slot = b0 + tid + static_cast<int64_t>(k) * kWG;
      qi[k] = slot < cnt ? (list ? list[slot] : slot) : -1;
      T c[3] = {T(0), T(0), T(0)};
      if (qi[k] >= 0) Loader<T, DIM, L>::query(query, qi[k], c);
#pragma unroll
      for (int d = 0; d < 3; ++d) qc[k][d] = c[d] * s;
      mn[k] = infT<T>();
    }
    T rc[2][3], rv[2];
    auto fetch = [&](int t) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int64_t j = jb + static_cast<int64_t>(t) * kTile + u * kWG + tid;
        if (j < je) {
          Loader<T, DIM, L>::data(data, j, rc[u], rv[u]);
        } else {  // padding record: infinitely far
          rc[u][0] = rc[u][1] = rc[u][2] = infT<T>();
          rv[u] = T(0);
        }
      }
    };
    auto put = [&](int b) {
#pragma unroll
      for (int u = 0; u < 2; ++u) tile[b][u * kWG + tid] = stage<T, DIM>(rc[u], rv[u], s);
    };
    const int ntiles = static_cast<int>((je - jb + kTile - 1) / kTile);
    fetch(0);
    put(0);
    __syncthreads();
    for (int t = 0; t < ntiles; ++t) {
      if (t + 1 < ntiles) fetch(t + 1);
      const int64_t jt = jb + static_cast<int64_t>(t) * kTile;
      const P4<T>* tl = tile[t & 1];
#pragma unroll 4
      for (int jj = 0; jj < kTile; ++jj) {
        const P4<T> d = tl[jj];
#pragma unroll
        for (int k = 0; k < Q; ++k) {
          T r2 = sqdist<T, DIM>(qc[k], d);
          if constexpr (EXCL) r2 = (jt + jj == qi[k]) ? infT<T>() : r2;
          mn[k] = r2 < mn[k] ? r2 : mn[k];
        }
      }
      if (t + 1 < ntiles) put((t + 1) & 1);
      __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < Q; ++k)
      if (qi[k] >= 0) atomicMin(&minb[qi[k]], min_bits(mn[k]));
  }
}

// FP64 recomputation of flagged queries.  The pattern of the improved CDP version
// (Section 3.1): a block of threads strides over the data points of one query with
// ceil(len / 256) points per lane, then a block reduction.  When few queries are flagged,
// each query's data range is cut into C chunks swept by different workgroups (C from the
// flagged count, so the grid of kFixGrid workgroups stays busy); chunk partials are
// merged in chunk order by k_fwd_fixmerge.  Exact d == 0 detection, Neumaier sums per lane,
// fixed-order tree reductions.  Writes Z and D (caller units; +inf at an exact hit, whose
// Z is the mean of the coincident values).
__device__ __forceinline__ int fix_chunks(int cnt, int cmax) {
  if (cnt <= 0) return 0;
  int c = kFixGrid / cnt;
  if (c > cmax) c = cmax;
  return c < 1 ? 1 : c;
}

constexpr int kWaves = kWG / 64;

// A lane's FP64 sums for one query, and its totals.
struct FixSums {
  double num, den, hz;
  long long h;
};
struct FixAcc {
  NSum num, den;
  double hz = 0.0;
  long long h = 0;
  template <typename T, int DIM>
  static __device__ __forceinline__ double dist(const T (&qt)[3], const T (&cc)[3]) {
    double r2 = 0.0;
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      const double e = static_cast<double>(qt[d]) - static_cast<double>(cc[d]);
      r2 += e * e;
    }
    return r2;
  }
  template <typename T, int DIM, int PM>
  __device__ __forceinline__ void add(const T (&qt)[3], const T (&cc)[3], T v, double nhp) {
    const double r2 = dist<T, DIM>(qt, cc);
    if (r2 == 0.0) {
      ++h;
      hz += static_cast<double>(v);
    } else {
      const double wgt = weight<PM>(r2, nhp);
      num.add(wgt * static_cast<double>(v));
      den.add(wgt);
    }
  }
  // A tree over the lanes of each wave; the first lane leaves the wave's sums in *out.
  __device__ __forceinline__ void reduce(FixSums* out) const {
    FixSums s = {num.value(), den.value(), hz, h};
#pragma unroll
    for (int x = 1; x < 64; x <<= 1) {
      s.num += __shfl_xor(s.num, x);
      s.den += __shfl_xor(s.den, x);
      s.hz += __shfl_xor(s.hz, x);
      s.h += __shfl_xor(s.h, x);
    }
    if ((threadIdx.x & 63) == 0) *out = s;
  }
};
// The waves' sums in order.
__device__ __forceinline__ FixSums fix_total(const FixSums (&red)[kWaves]) {
  FixSums s = red[0];
#pragma unroll
  for (int w = 1; w < kWaves; ++w) {
    s.num += red[w].num;
    s.den += red[w].den;
    s.hz += red[w].hz;
    s.h += red[w].h;
  }
  return s;
}

// Sums over data points [j0, j1) of query i in FP64, over the workgroup; every thread gets the
// totals (two barriers, where four block_sum()s have 40).  Call uniformly.
template <typename T, int DIM, int L, int PM>
__device__ __forceinline__ FixSums fix_query(const DevPts& data, const DevPts& query, int64_t i, int64_t j0, int64_t j1,
                                             bool excl, double nhp, FixSums (&red)[kWaves]) {
  T qt[3] = {T(0), T(0), T(0)};
  Loader<T, DIM, L>::query(query, i, qt);
  FixAcc acc;
  for (int64_t j = j0 + threadIdx.x; j < j1; j += kWG) {
    if (excl && j == i) continue;
    T cc[3] = {T(0), T(0), T(0)}, v;
    Loader<T, DIM, L>::data(data, j, cc, v);
    acc.template add<T, DIM, PM>(qt, cc, v, nhp);
  }
  __syncthreads();  // the last call's totals are read
  acc.reduce(&red[threadIdx.x >> 6]);
  __syncthreads();
  return fix_total(red);
}

// The same sums for the queries i[0] and i[1], each record read once.  At general p, whose weight is
// a long chain of operations, hits go through as selects so that the two chains overlap (four
// hits, 16,384 x 1,000, p = 1.7: 86 us against 97); the other weights keep the branch (all hits,
// 8,192 x 8,192, p = 2: 126 us against 139).  red: a row per query.
template <typename T, int DIM, int L, int PM>
__device__ __forceinline__ void fix_pair(const DevPts& data, const DevPts& query, const int64_t (&i)[2], int64_t n,
                                         bool excl, double nhp, FixSums (&red)[2][kWaves]) {
  T qt[2][3] = {};
  FixAcc acc[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) Loader<T, DIM, L>::query(query, i[k], qt[k]);
  for (int64_t j = threadIdx.x; j < n; j += kWG) {
    T cc[3] = {T(0), T(0), T(0)}, v;
    Loader<T, DIM, L>::data(data, j, cc, v);
    if constexpr (PM == PM_GEN) {
      double w[2];
      bool hit[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const double r2 = FixAcc::dist<T, DIM>(qt[k], cc);
        hit[k] = r2 == 0.0;
        w[k] = weight<PM>(r2, nhp);
      }
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const bool self = excl && j == i[k], on = hit[k] && !self;
        const double z = self ? 0.0 : static_cast<double>(v), u = hit[k] || self ? 0.0 : w[k];
        acc[k].h += on ? 1 : 0;
        acc[k].hz += on ? z : 0.0;
        acc[k].num.add(u * z);  // of no account once there is a hit
        acc[k].den.add(u);
      }
    } else {
#pragma unroll
      for (int k = 0; k < 2; ++k)
        if (!(excl && j == i[k])) acc[k].template add<T, DIM, PM>(qt[k], cc, v, nhp);
    }
  }
  __syncthreads();  // the last call's totals are read
#pragma unroll
  for (int k = 0; k < 2; ++k) acc[k].reduce(&red[k][threadIdx.x >> 6]);
  __syncthreads();
}

// Smallest squared distances (scaled units) of the queries q[0..K-1] over a workgroup's share of
// a pass over the data, per wave: mins[k][wave].  Queries past m take any place.
template <typename T, int DIM, int L, int K>
__device__ __forceinline__ void near_min(const DevPts& data, const DevPts& query, const int64_t (&q)[K], int64_t m,
                                         int64_t n, bool excl, T s, T (*mins)[kWaves]) {
  T mn[K], c[K][3];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    mn[k] = infT<T>();
    c[k][0] = c[k][1] = c[k][2] = T(0);
    if (q[k] < m) Loader<T, DIM, L>::query(query, q[k], c[k]);
#pragma unroll
    for (int d = 0; d < 3; ++d) c[k][d] *= s;
  }
  for (int64_t j = threadIdx.x; j < n; j += kWG) {
    T x[3] = {T(0), T(0), T(0)}, v;
    Loader<T, DIM, L>::data(data, j, x, v);
    const P4<T> rec = stage<T, DIM>(x, v, s);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      T r2 = sqdist<T, DIM>(c[k], rec);
      if (excl && j == q[k]) r2 = infT<T>();
      mn[k] = r2 < mn[k] ? r2 : mn[k];
    }
  }
#pragma unroll
  for (int k = 0; k < K; ++k) {
#pragma unroll
    for (int x = 1; x < 64; x <<= 1) {
      const T o = __shfl_xor(mn[k], x);
      mn[k] = o < mn[k] ? o : mn[k];
    }
    if ((threadIdx.x & 63) == 0) mins[k][threadIdx.x >> 6] = mn[k];
  }
}

template <typename T>
__device__ __forceinline__ void fix_write(const FixSums& s, int64_t i, T* __restrict__ out_z,
                                          double* __restrict__ out_den) {
  const double Z = s.h > 0 ? s.hz / static_cast<double>(s.h) : s.num / s.den;
  out_z[i] = static_cast<T>(Z);
  if (out_den) out_den[i] = s.h > 0 ? __builtin_huge_val() : s.den;
}

template <typename T, int DIM, int L, int PM>
__global__ __launch_bounds__(kWG) void k_fwd_fixup(DevPts data, int64_t n, DevPts query,
                                                   double nhp, unsigned flags,
                                                   const int* __restrict__ list,
                                                   const int* __restrict__ count, int cmax,
                                                   double4* __restrict__ fpart,
                                                   T* __restrict__ out_z,
                                                   double* __restrict__ out_den) {
  __shared__ FixSums red[kWaves];
  const int cnt = *count;
  const int C = fix_chunks(cnt, cmax);
  const int64_t total = static_cast<int64_t>(cnt) * C;
  const int64_t len = C > 0 ? (n + C - 1) / C : 0;
  const bool excl = (flags & 1u) != 0;
  for (int64_t w = blockIdx.x; w < total; w += gridDim.x) {
    const int64_t i = list[w / C];
    const int64_t j0 = (w % C) * len;
    const int64_t j1 = (j0 + len < n) ? j0 + len : n;
    const FixSums s = fix_query<T, DIM, L, PM>(data, query, i, j0, j1, excl, nhp, red);
    if (threadIdx.x == 0) {
      if (C == 1)
        fix_write<T>(s, i, out_z, out_den);
      else
        fpart[w] = make_double4(s.num, s.den, s.hz, static_cast<double>(s.h));
    }
  }
}

// Everything after the sweep of a small forward (small_call) in one launch: a wave merges its
// query's partials (lane c takes chunks c, c + 64, ..., then a fixed tree over the lanes) and
// finds the route; the workgroup then settles its candidates by their nearest distance, in one
// pass over the data, and recomputes the queries routed to FP64, two in a pass.  Such a call is
// mostly launches: with this kernel in place of five (merge, nearest-distance check, settling,
// fix-up and its merge) a call of 1,024 x 1,000 takes 13 us in place of 28.7, one of 4,096 x 4,099
// 20 in place of 32.  A pass of one workgroup is a chain of loads and FP64 operations, 17 us (p = 2)
// or 26 (p = 1.7) over 16,384 points: one for each of four neighbouring hits made a call of 16,384
// x 1,000 slower (84 and 116 us) than the five kernels, which cut a query's data among workgroups
// (80 and 107); in pairs it takes 66 and 86.
template <typename T, int DIM, int L, int PM>
__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_fwd_finish_small(DevPts data, int64_t n, DevPts query, int64_t m, int split,
                                                          double nhp, unsigned flags,
                                                          const double* __restrict__ hdr,
                                                          const double2* __restrict__ part, T* __restrict__ out_z,
                                                          double* __restrict__ out_den,
                                                          const uint8_t* __restrict__ route,
                                                          int* __restrict__ count) {
  __shared__ FixSums red[2][kWaves];
  __shared__ uint8_t routes[kWaves];
  __shared__ T mins[kWaves][kWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const bool excl = (flags & 1u) != 0;
  const int64_t first = static_cast<int64_t>(blockIdx.x) * kWaves;
  const int64_t i = first + wave;
  uint8_t r = F_FP32;
  if (i < m) {
    if (split > 1) {
      double nh = 0.0, nl = 0.0, dh = 0.0, dl = 0.0;
      for (int c = lane; c < split; c += 64) {
        const double2 v = part[static_cast<int64_t>(c) * m + i];
        two_sum_acc(nh, nl, v.x);
        two_sum_acc(dh, dl, v.y);
      }
#pragma unroll
      for (int x = 1; x < 64; x <<= 1) {
        const double a = __shfl_xor(nh, x), b = __shfl_xor(nl, x), c = __shfl_xor(dh, x), d = __shfl_xor(dl, x);
        two_sum_acc(nh, nl, a);
        two_sum_acc(dh, dl, c);
        nl += b;
        dl += d;
      }
      const double num = nh + nl, den = dh + dl;
      r = route_of(den, hdr, false);
      if (lane == 0) {
        out_z[i] = static_cast<T>(num / den);
        if (out_den) out_den[i] = den * hdr[H_DEN_UNIT];
      }
    } else {
      r = route[i];  // the sweep has finalised
    }
  }
  if (lane == 0) routes[wave] = r;
  if (!__syncthreads_or(lane == 0 && r != F_FP32)) return;
  unsigned cand = 0, fp64 = 0;  // bit k: the group's query k; uniform over the workgroup
#pragma unroll
  for (int k = 0; k < kWaves; ++k) {
    cand |= routes[k] == F_CANDIDATE ? 1u << k : 0u;
    fp64 |= routes[k] == F_FP64 ? 1u << k : 0u;
  }
  if (cand) {
    const T s = static_cast<T>(hdr[H_SCALE]);
    if (cand & (cand - 1)) {
      const int64_t q[kWaves] = {first, first + 1, first + 2, first + 3};
      near_min<T, DIM, L>(data, query, q, m, n, excl, s, mins);
    } else {
      const int64_t q[1] = {first + __ffs(cand) - 1};
      near_min<T, DIM, L>(data, query, q, m, n, excl, s, mins);
    }
    __syncthreads();
    for (unsigned c = cand; c; c &= c - 1) {
      const int k = __ffs(c) - 1;
      const T (&row)[kWaves] = mins[cand & (cand - 1) ? k : 0];
      T mn = row[0];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) mn = row[w] < mn ? row[w] : mn;
      if (settle_route<T>(F_CANDIDATE, min_bits(mn), hdr) == F_FP64) fp64 |= 1u << k;
    }
  }
  fp64 = __builtin_amdgcn_readfirstlane(fp64);
  const int fixed = __popc(fp64);
  while (fp64) {  // two at a time
    const int k0 = __ffs(fp64) - 1;
    fp64 &= fp64 - 1;
    if (fp64) {
      const int k1 = __ffs(fp64) - 1;
      fp64 &= fp64 - 1;
      fix_pair<T, DIM, L, PM>(data, query, {first + k0, first + k1}, n, excl, nhp, red);
      if (lane == 0 && (wave == k0 || wave == k1)) fix_write<T>(fix_total(red[wave == k1]), i, out_z, out_den);
    } else {
      const FixSums s = fix_query<T, DIM, L, PM>(data, query, first + k0, 0, n, excl, nhp, red[0]);
      if (lane == 0 && wave == k0) fix_write<T>(s, i, out_z, out_den);
    }
  }
  // one atomic per workgroup (they take 11 ns each on one address)
  if (threadIdx.x == 0 && fixed > 0) atomicAdd(count, fixed);
}

// Merges the chunk partials of split fix-up queries (chunk order, TwoSum) and finalises.
template <typename T>
__global__ __launch_bounds__(kWG) void k_fwd_fixmerge(const int* __restrict__ list,
                                                      const int* __restrict__ count, int cmax,
                                                      const double4* __restrict__ fpart,
                                                      T* __restrict__ out_z,
                                                      double* __restrict__ out_den) {
  const int cnt = *count;
  const int C = fix_chunks(cnt, cmax);
  if (C <= 1) return;
  for (int64_t sl = static_cast<int64_t>(blockIdx.x) * kWG + threadIdx.x; sl < cnt;
       sl += static_cast<int64_t>(gridDim.x) * kWG) {
    double nh = 0.0, nl = 0.0, dh = 0.0, dl = 0.0, hz = 0.0, h = 0.0;
    for (int c = 0; c < C; ++c) {
      const double4 v = fpart[static_cast<int64_t>(sl) * C + c];
      two_sum_acc(nh, nl, v.x);
      two_sum_acc(dh, dl, v.y);
      hz += v.z;
      h += v.w;
    }
    const int64_t i = list[sl];
    const double Z = h > 0.0 ? hz / h : (nh + nl) / (dh + dl);
    out_z[i] = static_cast<T>(Z);
    if (out_den) out_den[i] = h > 0.0 ? __builtin_huge_val() : dh + dl;
  }
}

// Bounding box and largest |value| as maxima: [0..DIM-1] negated minima, [DIM..2 DIM-1] maxima,
// [2 DIM] the value.
template <typename T, int DIM>
struct Box {
  static constexpr int N = 2 * DIM + 1;
  T v[N];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int k = 0; k < 2 * DIM; ++k) v[k] = -infT<T>();
    v[2 * DIM] = T(0);
  }
  __device__ __forceinline__ void add(const T (&c)[3], T z) {
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      v[d] = maxT(v[d], -c[d]);
      v[DIM + d] = maxT(v[DIM + d], c[d]);
    }
    v[2 * DIM] = maxT(v[2 * DIM], z < T(0) ? -z : z);
  }
  // Over the NT threads of a workgroup; the result is in the first wave.
  template <int NT>
  __device__ __forceinline__ void reduce(T (*red)[N]) {
    constexpr int W = NT / 64;
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < N; ++k)
#pragma unroll
      for (int x = 1; x < 64; x <<= 1) v[k] = maxT(v[k], __shfl_xor(v[k], x));
    if (lane == 0)
#pragma unroll
      for (int k = 0; k < N; ++k) red[threadIdx.x >> 6][k] = v[k];
    __syncthreads();
    if (threadIdx.x < 64)
#pragma unroll
      for (int k = 0; k < N; ++k) {
        v[k] = red[lane % W][k];
#pragma unroll
        for (int x = 1; x < W; x <<= 1) v[k] = maxT(v[k], __shfl_xor(v[k], x));
      }
  }
};

// Bounding box and header in one workgroup, for n <= kSmallBoxMax.
template <typename T, int DIM, int L>
__global__ __launch_bounds__(kSmallBox) void k_bbox_small(DevPts data, int64_t n, double p, int f32s, int rel,
                                                          double* __restrict__ hdr) {
  __shared__ T red[kSmallBox / 64][Box<T, DIM>::N];
  Box<T, DIM> b;
  b.clear();
  constexpr int kPer = static_cast<int>(kSmallBoxMax / kSmallBox);
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int64_t j = static_cast<int64_t>(u) * kSmallBox + threadIdx.x;
    if (j < n) {
      T c[3] = {T(0), T(0), T(0)}, z;
      Loader<T, DIM, L>::data(data, j, c, z);
      b.add(c, z);
    }
  }
  b.template reduce<kSmallBox>(red);
  if (threadIdx.x == 0) {
    double mn[3] = {0.0, 0.0, 0.0}, mx[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      mn[d] = -static_cast<double>(b.v[d]);
      mx[d] = static_cast<double>(b.v[DIM + d]);
    }
    finish_header(hdr, mn, mx, DIM, static_cast<double>(b.v[2 * DIM]), p, f32s != 0, rel != 0);
  }
}

// Per-workgroup bounding box of the data coordinates and largest |value|, in the
// kBboxStride-double record of each workgroup.
template <typename T, int DIM, int L>
__global__ __launch_bounds__(kWG) void k_bbox(DevPts data, int64_t n, double* __restrict__ part) {
  __shared__ T red[kWG / 64][Box<T, DIM>::N];
  Box<T, DIM> b;
  b.clear();
  for (int64_t j = static_cast<int64_t>(blockIdx.x) * kWG + threadIdx.x; j < n;
       j += static_cast<int64_t>(gridDim.x) * kWG) {
    T c[3] = {T(0), T(0), T(0)}, z;
    Loader<T, DIM, L>::data(data, j, c, z);
    b.add(c, z);
  }
  b.template reduce<kWG>(red);
  if (threadIdx.x == 0) {
    double* o = part + blockIdx.x * kBboxStride;
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      o[d] = -static_cast<double>(b.v[d]);
      o[3 + d] = static_cast<double>(b.v[DIM + d]);
    }
    o[6] = static_cast<double>(b.v[2 * DIM]);
  }
}

// ---------------------------------------------------------------------------------------
// Host launchers for one layout (instantiated once per layout translation unit).
// ---------------------------------------------------------------------------------------
template <typename T, int DIM, int L, int PM>
hipError_t launch_fwd_sweep_q(const FwdArgs& a, hipStream_t st) {
  const int Q = a.q_per_lane;
  const int64_t qpb = static_cast<int64_t>(kWG) * Q;
  dim3 grid(static_cast<unsigned>((a.m + qpb - 1) / qpb), static_cast<unsigned>(a.split));
  const T nhp = static_cast<T>(-0.5 * a.p);
  T* z = static_cast<T*>(a.out_z);
#define IDW_FWD_ARGS                                                                          \
  a.data, a.n, a.query, a.m, a.chunk, a.split, nhp, a.flags, a.hdr, z, a.out_den, a.flag, a.part, \
      a.rmin, a.p
#define IDW_FWD_Q(QQ)                                                                       \
  case QQ:                                                                                  \
    hipLaunchKernelGGL((k_fwd_sweep<T, DIM, L, PM, QQ>), grid, dim3(kWG), 0, st, IDW_FWD_ARGS); \
    break;
  if constexpr (sizeof(T) == 4) {
    if (a.rel) {  // relative weights: general-p form only
      if constexpr (PM == PM_GEN) {
        if (!a.rmin) return hipErrorInvalidValue;
        if (a.kahan && Q == 4)
          hipLaunchKernelGGL((k_fwd_sweep<T, DIM, L, PM, 4, true, true>), grid, dim3(kWG), 0, st, IDW_FWD_ARGS);
        else if (!a.kahan && Q == 4)
          hipLaunchKernelGGL((k_fwd_sweep<T, DIM, L, PM, 4, false, true>), grid, dim3(kWG), 0, st, IDW_FWD_ARGS);
        else if (!a.kahan && Q == 8)
          hipLaunchKernelGGL((k_fwd_sweep<T, DIM, L, PM, 8, false, true>), grid, dim3(kWG), 0, st, IDW_FWD_ARGS);
        else
          return hipErrorInvalidValue;
        return hipGetLastError();
      } else {
        return hipErrorInvalidValue;
      }
    }
    if (a.kahan) {  // per-pair Kahan variant, 4 queries per lane
      if (Q != 4) return hipErrorInvalidValue;
      hipLaunchKernelGGL((k_fwd_sweep<T, DIM, L, PM, 4, true>), grid, dim3(kWG), 0, st, IDW_FWD_ARGS);
      return hipGetLastError();
    }
    switch (Q) {
      IDW_FWD_Q(2)
      IDW_FWD_Q(4)
      IDW_FWD_Q(8)
      default:
        return hipErrorInvalidValue;
    }
  } else {
    if constexpr (PM == PM_GEN) {
      if (0.5 * a.p <= kPowLow && Q == 2) {
        hipLaunchKernelGGL((k_fwd_sweep<T, DIM, L, PM, 2, false, false, SweepTuneLow<2>>), grid, dim3(kWG), 0, st,
                           IDW_FWD_ARGS);
        return hipGetLastError();
      }
    }
    switch (Q) {
      IDW_FWD_Q(2)
      IDW_FWD_Q(4)
      default:
        return hipErrorInvalidValue;
    }
  }
#undef IDW_FWD_Q
#undef IDW_FWD_ARGS
  return hipGetLastError();
}

template <typename T, int DIM, int L>
hipError_t launch_fwd_sweep_pm(const FwdArgs& a, hipStream_t st) {
  switch (a.pmode) {
    case PM_1: return launch_fwd_sweep_q<T, DIM, L, PM_1>(a, st);
    case PM_2: return launch_fwd_sweep_q<T, DIM, L, PM_2>(a, st);
    case PM_3: return launch_fwd_sweep_q<T, DIM, L, PM_3>(a, st);
    case PM_4: return launch_fwd_sweep_q<T, DIM, L, PM_4>(a, st);
    case PM_25: return launch_fwd_sweep_q<T, DIM, L, PM_25>(a, st);
    default: return launch_fwd_sweep_q<T, DIM, L, PM_GEN>(a, st);
  }
}

template <int L>
hipError_t launch_fwd_sweep(const FwdArgs& a, bool f64, hipStream_t st) {
  if (f64) return a.dim == 3 ? launch_fwd_sweep_pm<double, 3, L>(a, st) : launch_fwd_sweep_pm<double, 2, L>(a, st);
  return a.dim == 3 ? launch_fwd_sweep_pm<float, 3, L>(a, st) : launch_fwd_sweep_pm<float, 2, L>(a, st);
}

template <typename T, int DIM, int L, int PM>
hipError_t launch_fwd_fixup_t(const FwdArgs& a, hipStream_t st) {
  if (a.small) {
    hipLaunchKernelGGL((k_fwd_finish_small<T, DIM, L, PM>), dim3(static_cast<unsigned>((a.m + kWaves - 1) / kWaves)),
                       dim3(kWG), 0, st, a.data, a.n, a.query, a.m, a.split, -0.5 * a.p, a.flags, a.hdr, a.part,
                       static_cast<T*>(a.out_z), a.out_den, a.flag, const_cast<int*>(a.count));
    return hipGetLastError();
  }
  hipLaunchKernelGGL((k_fwd_fixup<T, DIM, L, PM>), dim3(kFixGrid), dim3(kWG), 0, st, a.data,
                     a.n, a.query, -0.5 * a.p, a.flags, a.list, a.count, a.fix_cmax, a.fpart,
                     static_cast<T*>(a.out_z), a.out_den);
  if (a.fix_cmax > 1)  // data ranges that may be cut into chunks
    hipLaunchKernelGGL((k_fwd_fixmerge<T>), dim3(4), dim3(kWG), 0, st, a.list, a.count, a.fix_cmax,
                       a.fpart, static_cast<T*>(a.out_z), a.out_den);
  return hipGetLastError();
}

template <typename T, int DIM, int L>
hipError_t launch_fwd_fixup_pm(const FwdArgs& a, hipStream_t st) {
  switch (a.pmode) {
    case PM_1: return launch_fwd_fixup_t<T, DIM, L, PM_1>(a, st);
    case PM_2: return launch_fwd_fixup_t<T, DIM, L, PM_2>(a, st);
    case PM_3: return launch_fwd_fixup_t<T, DIM, L, PM_3>(a, st);
    case PM_4: return launch_fwd_fixup_t<T, DIM, L, PM_4>(a, st);
    case PM_25: return launch_fwd_fixup_t<T, DIM, L, PM_25>(a, st);
    default: return launch_fwd_fixup_t<T, DIM, L, PM_GEN>(a, st);
  }
}

template <int L>
hipError_t launch_fwd_fixup(const FwdArgs& a, bool f64, hipStream_t st) {
  if (f64) return a.dim == 3 ? launch_fwd_fixup_pm<double, 3, L>(a, st) : launch_fwd_fixup_pm<double, 2, L>(a, st);
  return a.dim == 3 ? launch_fwd_fixup_pm<float, 3, L>(a, st) : launch_fwd_fixup_pm<float, 2, L>(a, st);
}

template <typename T, int DIM, int L>
hipError_t launch_near_check_t(const NearArgs& a, hipStream_t st) {
  constexpr int Q = sizeof(T) == 4 ? 4 : 2;
  const unsigned gl = static_cast<unsigned>(a.m < 64 * kWG ? (a.m + kWG - 1) / kWG + 1 : 64);
  const int* list = a.all ? nullptr : a.list;
  if (!a.all && !a.list) return hipErrorInvalidValue;
  if (a.init)
    hipLaunchKernelGGL((k_near_init<T>), dim3(gl), dim3(kWG), 0, st, list, a.count, a.m, a.minb);
  if (a.excl)
    hipLaunchKernelGGL((k_near_check<T, DIM, L, Q, true>), dim3(kNearGrid), dim3(kWG), 0, st, a.data, a.n,
                       a.query, list, a.count, a.list2, a.count2, a.m, a.hdr, a.minb);
  else
    hipLaunchKernelGGL((k_near_check<T, DIM, L, Q, false>), dim3(kNearGrid), dim3(kWG), 0, st, a.data, a.n,
                       a.query, list, a.count, a.list2, a.count2, a.m, a.hdr, a.minb);
  return hipGetLastError();
}

template <int L>
hipError_t launch_near_check(const NearArgs& a, hipStream_t st) {
  if (a.f64) return a.dim == 3 ? launch_near_check_t<double, 3, L>(a, st) : launch_near_check_t<double, 2, L>(a, st);
  return a.dim == 3 ? launch_near_check_t<float, 3, L>(a, st) : launch_near_check_t<float, 2, L>(a, st);
}

// The header of a call: one kernel for few data points, else per-workgroup boxes and their
// reduction (idw_common.hip).
template <typename T, int DIM, int L>
hipError_t launch_header_t(const HeaderArgs& a, hipStream_t st) {
  if (a.n <= kSmallBoxMax) {
    hipLaunchKernelGGL((k_bbox_small<T, DIM, L>), dim3(1), dim3(kSmallBox), 0, st, a.data, a.n, a.p,
                       sizeof(T) == 4 ? 1 : 0, a.rel ? 1 : 0, a.hdr);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((k_bbox<T, DIM, L>), dim3(a.nblocks), dim3(kWG), 0, st, a.data, a.n, a.part);
  return bbox_final(a.part, a.nblocks, DIM, a.p, sizeof(T) == 4, a.rel, a.hdr, st);
}

template <int L>
hipError_t launch_header(const HeaderArgs& a, int dim, bool f64, hipStream_t st) {
  if (f64) return dim == 3 ? launch_header_t<double, 3, L>(a, st) : launch_header_t<double, 2, L>(a, st);
  return dim == 3 ? launch_header_t<float, 3, L>(a, st) : launch_header_t<float, 2, L>(a, st);
}

}  // namespace idw
