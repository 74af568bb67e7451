// Fused adjoint sweep: the query-direction sums (P_i, G_i, for dp and dq) and the
// data-direction sums (dz_j = sum_i a_i w_ij, a_i = g_i / D_i, and, for the gradient with
// respect to the data coordinates, X_j = sum_i a_i (w_ij / r2_ij)(z_j - Z_i)(q_i - x_j))
// from ONE evaluation of each pair's weight.
//
// FP64 (k_bwd_fused): lanes own Q queries each (registers).  Data points are staged in LDS in
// batches of 64, each batch stored twice in a row, so that at step s lane L reads record
// (L + s) of the doubled batch -- data point (L + s) mod 64 -- with a compile-time offset and
// no bank conflicts.  Query-direction sums accumulate per lane as in the query sweep.  For the
// data direction every lane forms s_L = sum_k a_k w_k for its point of the step, and a
// running sum travels one lane per step (lane L receives the sum held by lane L+1), picking
// up the contribution of each lane for the same data point.  After 64 steps lane L holds the
// sum over the wave's 64 x Q queries for batch point (L - 1) mod 64.  X_j rides the same
// rotation with one running sum per coordinate.
//
// FP32 (k_bwd_fused32): lanes own data points and waves own queries, see there.
//
// Work decomposition of both: workgroup (qg, dr) sweeps data range dr for the query blocks
// qg, qg + G, qg + 2G, ...; it writes the query partials of range dr (as the query sweep
// with a data split) and accumulates its dz partial row qg across its query blocks (the
// data sweep's split-over-queries format), so the existing fixed-order merges apply.
#pragma once

#include "idw_bwd.hpp"
#include "idw_device.hpp"
#include "idw_fwd.hpp"

namespace idw {

constexpr int kBatch = 64;  // data points per rotation batch (one wave)

// Data points per LDS tile and threads per workgroup of the FP64 form (the tiles, batches
// doubled, and the per-wave sums take 40 KB of LDS).
constexpr int kFTile64 = 256;
constexpr int kFNT64 = 256;

// Lane L takes the running sum of lane L+1 (wave rotate left by one), as two 32-bit halves.
__device__ __forceinline__ double rotate_in(double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(static_cast<unsigned int>(b)), 0x134, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(static_cast<unsigned int>(b >> 32)), 0x134, 0xF, 0xF,
                                             false);
  return __builtin_bit_cast(double, (static_cast<unsigned long long>(static_cast<unsigned int>(hi)) << 32) |
                                        static_cast<unsigned int>(lo));
}

// One 64-point batch.  MASK: some pairs must be skipped (padding records beyond the data
// range, or the leave-one-out self pair); those get r2 = 1 and zero value factors.
// Returns the dz running sum; with NDX, ax holds the X running sums.
template <typename T, int DIM, int PM, int Q, bool NDP, bool NDQ, bool NDX, bool MASK, int UNR>
__device__ __forceinline__ T bwdf_batch(const P4<T>* __restrict__ rec, int lane, int64_t jb, int64_t je,
                                        bool excl, const T (&qc)[Q][3], const T (&zq)[Q], const T (&aq)[Q],
                                        const int64_t (&qi)[Q], T nhp, T (&ap)[Q], T (&ag)[Q][3], T (&ax)[3]) {
  T acc = T(0);
  ax[0] = ax[1] = ax[2] = T(0);
  const P4<T>* r0 = rec + lane;
#pragma unroll UNR
  for (int s = 0; s < kBatch; ++s) {
    const P4<T> d = r0[s];
    const T dv = (DIM == 3) ? d.w : d.z;
    T sz = T(0);
    T sx[3] = {T(0), T(0), T(0)};
    int64_t j = 0;
    bool valid = true;
    if constexpr (MASK) {
      j = jb + ((lane + s) & (kBatch - 1));
      valid = j < je;
    }
    T rcp[Q];
    if constexpr (PairRcp<T, PM>::on) {
      static_assert(Q == 2, "two queries per lane");
#pragma unroll
      for (int k = 0; k < Q; ++k) {
        rcp[k] = sqdist<T, DIM>(qc[k], d);
        if constexpr (MASK) {
          if (!valid || (excl && j == qi[k])) rcp[k] = T(1);
        }
      }
      rcp64_w2(rcp[0], rcp[1]);
    }
#pragma unroll
    for (int k = 0; k < Q; ++k) {
      const T dx = qc[k][0] - d.x;
      const T dy = qc[k][1] - d.y;
      T dz = T(0);
      T r2 = dx * dx;
      r2 = fmaT(dy, dy, r2);
      if constexpr (DIM == 3) {
        dz = qc[k][2] - d.z;
        r2 = fmaT(dz, dz, r2);
      }
      T c = dv - zq[k];
      T a = aq[k];
      if constexpr (MASK) {
        if (!valid || (excl && j == qi[k])) {
          r2 = T(1);
          c = T(0);
          a = T(0);
        }
      }
      T w, f = T(0), lg = T(0);
      if constexpr (PairRcp<T, PM>::on)
        wterms_rcp<PM, NDQ || NDX, NDP>(r2, rcp[k], w, f, lg);
      else
        wterms<PM, NDQ || NDX, NDP, PowTab<T, PM, NDP || NDX>::on>(r2, nhp, w, f, lg);
      const T t = w * c;
      if constexpr (NDP) ap[k] = fmaT(t, lg, ap[k]);
      if constexpr (NDQ || NDX) {
        const T u = wr_times<PM>(t, c, f);  // (w / r2)(z - Z)
        if constexpr (NDQ) {
          ag[k][0] = fmaT(u, dx, ag[k][0]);
          ag[k][1] = fmaT(u, dy, ag[k][1]);
          if constexpr (DIM == 3) ag[k][2] = fmaT(u, dz, ag[k][2]);
        }
        if constexpr (NDX) {
          const T v = a * u;
          sx[0] = (k == 0) ? v * dx : fmaT(v, dx, sx[0]);
          sx[1] = (k == 0) ? v * dy : fmaT(v, dy, sx[1]);
          if constexpr (DIM == 3) sx[2] = (k == 0) ? v * dz : fmaT(v, dz, sx[2]);
        }
      }
      sz = (k == 0) ? a * w : fmaT(a, w, sz);
    }
    acc = rotate_in(acc) + sz;
    if constexpr (NDX) {
#pragma unroll
      for (int e = 0; e < DIM; ++e) ax[e] = rotate_in(ax[e]) + sx[e];
    }
  }
  return acc;
}

// Coordinate given to queries that are left out of a sweep (flagged for the FP64 fix-up):
// far from every scaled data point, yet with r2 (< 3 * 2^120) and every product of the
// pair terms finite, so that their zero factors a = 0 give exact zeros.
constexpr float kFarF = 0x1p60f;

// The FP64 adjoint (the FP64 one-step and table forms of the weights).
template <typename T, int DIM, int L, int PM, int Q, bool NDP, bool NDQ, bool NDX, int UNR = 2, int WPE = 2,
          int NT = kFNT64>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(WPE, 8))) void k_bwd_fused(
    DevPts data, int64_t n, DevPts query, int64_t m, int64_t chunk, int groups, T nhp, unsigned flags,
    const double* __restrict__ hdr, const T* __restrict__ saved_z, const T* __restrict__ grad_out,
    const double* __restrict__ saved_den, double4* __restrict__ part_q, double* __restrict__ part_z,
    double* __restrict__ part_x, const uint8_t* __restrict__ route) {
  constexpr int kFTile = kFTile64;
  constexpr int kFBatches = kFTile / kBatch;
  __shared__ P4<T> tile[2][2 * kFTile];   // batches stored twice in a row
  constexpr int PPT = kFTile / NT;        // tile points staged per thread
  static_assert(PPT >= 1, "a tile holds at least one point per thread");
  __shared__ T zred[NT / 64][kFTile];     // per-wave dz sums of the current tile
  __shared__ T xred[NDX ? NT / 64 : 1][NDX ? DIM * kFTile : 1];  // per-wave X sums
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int qg = blockIdx.x;
  const int64_t jb = static_cast<int64_t>(blockIdx.y) * chunk;
  const int64_t je = (jb + chunk < n) ? jb + chunk : n;
  const T s = static_cast<T>(hdr[H_SCALE]);
  const double unit = hdr[H_DEN_UNIT];
  const bool excl = (flags & 1u) != 0;
  // FP64 tables (synchronised below); with dx the pow tables cost too much occupancy.
  constexpr bool kPow = PowTab<T, PM, NDP || NDX>::on;
  if constexpr (kPow) pow_table_init(NDQ ? nhp - 1.0 : nhp);
  if constexpr (sizeof(T) == 8 && !kPow && (NDP || PM == PM_GEN)) log2_table_init();
  if constexpr (sizeof(T) == 8 && !kPow && PM == PM_GEN) exp2_table_init();
  const int64_t qpb = static_cast<int64_t>(NT) * Q;
  const int64_t nqb = (m + qpb - 1) / qpb;
  const int ntiles = static_cast<int>((je - jb + kFTile - 1) / kFTile);
  double* zrow = part_z + static_cast<int64_t>(qg) * n;
  double* xrow = NDX ? part_x + static_cast<int64_t>(qg) * n * DIM : nullptr;

  T rc[PPT][3], rv[PPT];
  auto fetch = [&](int t) {
#pragma unroll
    for (int u = 0; u < PPT; ++u) {
      const int64_t j = jb + static_cast<int64_t>(t) * kFTile + u * NT + tid;
      rc[u][0] = rc[u][1] = rc[u][2] = T(0);
      rv[u] = T(0);
      if (j < je) Loader<T, DIM, L>::data(data, j, rc[u], rv[u]);
    }
  };
  auto put = [&](int b) {
#pragma unroll
    for (int u = 0; u < PPT; ++u) {
      const int p = u * NT + tid;                        // point within the tile
      const int at = (p / kBatch) * (2 * kBatch) + (p % kBatch);
      const P4<T> r = stage<T, DIM>(rc[u], rv[u], s);
      tile[b][at] = r;
      tile[b][at + kBatch] = r;
    }
  };

  int first = 1;
  for (int64_t qb = qg; qb < nqb; qb += groups, first = 0) {
    const int64_t q0 = qb * qpb;
    T qc[Q][3], zq[Q], aq[Q];
    int64_t qi[Q];
#pragma unroll
    for (int k = 0; k < Q; ++k) {
      qi[k] = q0 + tid + static_cast<int64_t>(k) * NT;
      T c[3] = {T(0), T(0), T(0)};
      bool ok = false;
      zq[k] = T(0);
      aq[k] = T(0);
      if (qi[k] < m) {
        ok = route[qi[k]] == F_FP32;  // the others are left to the FP64 fix-up
        if (ok) {
          const double D = saved_den[qi[k]];
          Loader<T, DIM, L>::query(query, qi[k], c);
          zq[k] = saved_z[qi[k]];
          const double g = static_cast<double>(grad_out[qi[k]]);
          aq[k] = static_cast<T>(g / (D / unit));
        }
      }
#pragma unroll
      for (int d = 0; d < 3; ++d) qc[k][d] = ok ? c[d] * s : static_cast<T>(kFarF);
    }
    BlockSum<T> P[Q], G[Q][3];
#pragma unroll
    for (int k = 0; k < Q; ++k) {
      P[k].zero();
#pragma unroll
      for (int d = 0; d < 3; ++d) G[k][d].zero();
    }

    fetch(0);
    put(0);
    __syncthreads();
    for (int t = 0; t < ntiles; ++t) {
      if (t + 1 < ntiles) fetch(t + 1);
      const int64_t jt = jb + static_cast<int64_t>(t) * kFTile;
      const bool diag = excl && jt < q0 + qpb && q0 < jt + kFTile;
      const bool tail = jt + kFTile > je;
#pragma unroll 1
      for (int b = 0; b < kFBatches; ++b) {
        T ap[Q], ag[Q][3];
#pragma unroll
        for (int k = 0; k < Q; ++k) {
          ap[k] = T(0);
          ag[k][0] = ag[k][1] = ag[k][2] = T(0);
        }
        const P4<T>* rec = tile[t & 1] + b * (2 * kBatch);
        const int64_t jbat = jt + b * kBatch;
        T zs, ax[3];
        if (diag || tail)
          zs = bwdf_batch<T, DIM, PM, Q, NDP, NDQ, NDX, true, 1>(rec, lane, jbat, je, excl, qc, zq, aq, qi, nhp, ap, ag, ax);
        else
          zs = bwdf_batch<T, DIM, PM, Q, NDP, NDQ, NDX, false, UNR>(rec, lane, jbat, je, excl, qc, zq, aq, qi, nhp, ap, ag, ax);
        const int at = b * kBatch + ((lane + kBatch - 1) & (kBatch - 1));
        zred[wave][at] = zs;
        if constexpr (NDX) {
#pragma unroll
          for (int e = 0; e < DIM; ++e) xred[wave][e * kFTile + at] = ax[e];
        }
#pragma unroll
        for (int k = 0; k < Q; ++k) {
          if constexpr (NDP) P[k].add(ap[k]);
          if constexpr (NDQ) {
#pragma unroll
            for (int d = 0; d < DIM; ++d) G[k][d].add(ag[k][d]);
          }
        }
      }
      __syncthreads();  // zred complete; tile t fully consumed
      // dz: sum the waves' partials in wave order and fold into this group's row
#pragma unroll
      for (int u = 0; u < PPT; ++u) {
        const int p = u * NT + tid;
        const int64_t j = jt + p;
        if (j < je) {
          double v = static_cast<double>(zred[0][p]);
#pragma unroll
          for (int w = 1; w < NT / 64; ++w) v += static_cast<double>(zred[w][p]);
          zrow[j] = first ? v : zrow[j] + v;
          if constexpr (NDX) {
#pragma unroll
            for (int e = 0; e < DIM; ++e) {
              double x = static_cast<double>(xred[0][e * kFTile + p]);
#pragma unroll
              for (int w = 1; w < NT / 64; ++w) x += static_cast<double>(xred[w][e * kFTile + p]);
              xrow[j * DIM + e] = first ? x : xrow[j * DIM + e] + x;
            }
          }
        }
      }
      if (t + 1 < ntiles) put((t + 1) & 1);
      __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < Q; ++k) {
      if (qi[k] < m) {
        double4 r;
        r.x = P[k].value();
        r.y = G[k][0].value();
        r.z = G[k][1].value();
        r.w = G[k][2].value();
        part_q[static_cast<int64_t>(blockIdx.y) * m + qi[k]] = r;
      }
    }
  }
  // A group without any query block still owns a partial row: make it zero.
  if (first) {
    for (int64_t j = jb + tid; j < je; j += NT) {
      zrow[j] = 0.0;
      if constexpr (NDX) {
#pragma unroll
        for (int e = 0; e < DIM; ++e) xrow[j * DIM + e] = 0.0;
      }
    }
  }
}

// ---------------------------------------------------------------------------------------
// FP32 form.  Lanes own data points, waves own queries: a wave holds R queries as uniform
// (scalar) values and sweeps the data range 64 points at a time.  The data-direction sums of
// a lane's point are then plain per-lane sums over the R queries, and the query-direction
// sums are kept per lane and query (R (1 + DIM) registers) and added over the 64 lanes only
// every kFlush points.  Nothing crosses lanes per pair: the rotation of the FP64 form costs
// half a DPP add per pair, which also puts the SIMD's waves out of step (idw_phase.hpp;
// measured 10 cycles per pair).  2-D p = 2 with dz, dp and dq: 11 plain instructions and two
// transcendentals, 39.2 cycles per pair and wave at best, 41.7 for the loop body alone, 44.2
// for the kernel; 1M x 1M: 350 ms with lanes owning queries and the rotation, 308 ms now; with
// dx 462 -> 389, p = 1.5 404 -> 335, p = 8 (relative weights) 458 -> 403.
// ---------------------------------------------------------------------------------------

// Queries per wave: as many as the registers of 4 waves per SIMD hold.  16 in 2-D (48 sums) and
// in 3-D (64 sums; 131,072 x 1M points, p = 2: 47.0 ms against 49.0 with 8); 8 where the scales
// of the relative weights would make 16 spill, which for dz alone, without query sums and X sums,
// they do not (65,536 x 65,536, p = 8: 1.18 ms against 1.28 with 8).  With the 3-D X sums 16 fit
// once the FP64 sums over lanes are left in memory (GSUM), and the staging, folding and row
// traffic of a tile are shared by twice the queries (131,072 x 262,144, p = 2 with dx: 83 cycles
// per pair and wave with 8 queries, 80 with 12, 74 with 16).
template <bool SUMS, bool NDX, bool REL>
struct FusedRows {
  static constexpr int R = REL && (SUMS || NDX) ? 8 : 16;
};
constexpr int kFusedWaves = 8;
constexpr int kFlush = 4096;  // data points between the sums over lanes (64 per lane)

__device__ __forceinline__ float read_lane(float v, int l) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}
__device__ __forceinline__ double shfl_xor64(double v, int x) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const int lo = __shfl_xor(static_cast<int>(static_cast<unsigned int>(b)), x);
  const int hi = __shfl_xor(static_cast<int>(static_cast<unsigned int>(b >> 32)), x);
  return __builtin_bit_cast(double, (static_cast<unsigned long long>(static_cast<unsigned int>(hi)) << 32) |
                                        static_cast<unsigned int>(lo));
}

template <int DIM, int L, int PM, bool NDP, bool NDQ, bool NDX, bool REL, bool EXCL,
          int R = FusedRows<NDP || NDQ, NDX, REL>::R>
__global__ __launch_bounds__(64 * kFusedWaves) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_bwd_fused32(
    DevPts data, int64_t n, DevPts query, int64_t m, int64_t chunk, int groups, float nhp, unsigned,
    const double* __restrict__ hdr, const float* __restrict__ saved_z, const float* __restrict__ grad_out,
    const double* __restrict__ saved_den, double4* __restrict__ part_q, double* __restrict__ part_z,
    double* __restrict__ part_x, const uint8_t* __restrict__ route, double pd) {
  constexpr int NT = 64 * kFusedWaves;
  constexpr int TILE = NT;                      // one point staged and folded per thread
  constexpr int NB = TILE / 64;                 // 64-point batches per tile
  constexpr int GQ = 4;                         // queries whose weights are taken in one run
  constexpr int NC = (NDP ? 1 : 0) + (NDQ ? DIM : 0);  // query-direction sums per query
  constexpr int NR = (R * NC + 7) / 8;          // rounds of 8 sums in the addition over lanes
  static_assert(R % 8 == 0 && R <= 64 && (NB & (NB - 1)) == 0, "whole runs of queries");
  __shared__ RecTile<float, 3, TILE> tile[2];
  alignas(16) __shared__ float zred[kFusedWaves][TILE];  // per-wave dz sums; rows of the addition over lanes
  static_assert(__alignof__(zred) >= alignof(P4<float>), "flush reads four values at a time");
  __shared__ float xred[NDX ? kFusedWaves : 1][NDX ? DIM * TILE : 1];  // per-wave X sums
  // The FP64 sums over lanes: in LDS, or, where the X sums take it, in registers, or, where 16
  // queries with X sums leave none (3-D), in the query's partial itself.
  constexpr bool LSUM = !NDX && NR > 0;
  constexpr bool GSUM = NDX && DIM == 3 && !REL;
  __shared__ double lsum[LSUM ? kFusedWaves : 1][LSUM ? NR : 1][LSUM ? 64 : 1];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qg = blockIdx.x;
  const int64_t jb = static_cast<int64_t>(blockIdx.y) * chunk;
  const int64_t je = (jb + chunk < n) ? jb + chunk : n;
  const float s = static_cast<float>(hdr[H_SCALE]);
  const double unit = hdr[H_DEN_UNIT];
  constexpr int64_t qpb = kFusedWaves * R;
  const int64_t nqb = (m + qpb - 1) / qpb;
  const int ntiles = static_cast<int>((je - jb + TILE - 1) / TILE);
  double* zrow = part_z + static_cast<int64_t>(qg) * n;
  double* xrow = NDX ? part_x + static_cast<int64_t>(qg) * n * DIM : nullptr;

  float rc[3], rv;
  auto fetch = [&](int t) {
    const int64_t j = jb + static_cast<int64_t>(t) * TILE + tid;
    rc[0] = rc[1] = rc[2] = rv = 0.f;
    if (j < je) Loader<float, DIM, L>::data(data, j, rc, rv);
  };
  auto put = [&](int b) {
    tile[b].put(tid, P4<float>{rc[0] * s, rc[1] * s, DIM == 3 ? rc[2] * s : 0.f, rv});
  };

  int first = 1;
  for (int64_t qb = qg; qb < nqb; qb += groups, first = 0) {
    const int64_t q0 = qb * qpb;
    const int64_t qw = q0 + static_cast<int64_t>(wave) * R;  // this wave's first query
    // lane r prepares query r, then every lane reads it as a uniform value
    auto prepare = [&](float (&vq)[3], float& vz, float& va, float& vs, float& vk, float& vx) {
      const int64_t i = qw + lane;
      float c[3] = {0.f, 0.f, 0.f};
      bool ok = false;
      vz = va = vk = vx = 0.f;
      vs = 1.f;
      if (lane < R && i < m) {
        ok = route[i] == F_FP32;  // the others are left to the FP64 fix-up
        if (ok) {
          const double D = saved_den[i];
          Loader<float, DIM, L>::query(query, i, c);
          vz = saved_z[i];
          const double g = static_cast<double>(grad_out[i]);
          if constexpr (REL) {
            double E = 1.0;
            rel_from_den(D / unit, pd, vs, vk, E);
            va = static_cast<float>(g / E);
            vx = static_cast<float>(g / E * static_cast<double>(vs));
          } else {
            vx = va = static_cast<float>(g / (D / unit));
          }
        }
      }
#pragma unroll
      for (int d = 0; d < 3; ++d) vq[d] = ok ? c[d] * s : kFarF;
    };
    float vq[3], vz, va, vs, vk, vx;
    prepare(vq, vz, va, vs, vk, vx);
    float qc[R][3], zq[R], aq[R], sg[R], kq[R], axq[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
      for (int d = 0; d < DIM; ++d) qc[r][d] = read_lane(vq[d], r);
      zq[r] = read_lane(vz, r);
      aq[r] = read_lane(va, r);
      if constexpr (REL) {
        sg[r] = read_lane(vs, r);
        if constexpr (NDP) kq[r] = read_lane(vk, r);
        if constexpr (NDX) axq[r] = read_lane(vx, r);
      }
    }
    constexpr int NA = NC > 0 ? NC : 1;
    float acc[NA][R];           // P, then G per coordinate
    float own[NA];              // EXCL, lane r: query r's sums over its leave-one-out block
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      own[c] = 0.f;
#pragma unroll
      for (int r = 0; r < R; ++r) acc[c][r] = 0.f;
    }
    double sums[LSUM || GSUM || NR == 0 ? 1 : NR];
    if constexpr (!GSUM) {
#pragma unroll
      for (int k = 0; k < NR; ++k) {
        if constexpr (LSUM)
          lsum[wave][k][lane] = 0.0;
        else
          sums[k] = 0.0;
      }
    }

    // The lane's point against the wave's queries.  Every layer of GQ independent operations
    // is kept together: an operation on the result of the one before it would not issue
    // beside the other wave's.
    auto batch = [&](const P4<float>& d, float& zs, float (&xs)[3]) {
#define IDW_LAYER(expr)                      \
  __builtin_amdgcn_sched_barrier(0);         \
  _Pragma("unroll") for (int i = 0; i < GQ; ++i) { expr; }
#pragma unroll
      for (int r0 = 0; r0 < R; r0 += GQ) {
        float dx[GQ], dy[GQ], dz[GQ], r2[GQ], w[GQ], f[GQ], lg[GQ], c[GQ];
        IDW_LAYER(dx[i] = qc[r0 + i][0] - d.x)
        IDW_LAYER(dy[i] = qc[r0 + i][1] - d.y)
        IDW_LAYER(r2[i] = dx[i] * dx[i])
        if constexpr (DIM == 3) { IDW_LAYER(dz[i] = qc[r0 + i][2] - d.z) }
        IDW_LAYER(r2[i] = fmaf(dy[i], dy[i], r2[i]))
        if constexpr (DIM == 3) { IDW_LAYER(r2[i] = fmaf(dz[i], dz[i], r2[i])) }
        if constexpr (REL) { IDW_LAYER(r2[i] *= sg[r0 + i]) }
        wterms_run<PM, NDQ || NDX, NDP, GQ>(r2, nhp, w, f, lg);
        IDW_LAYER(c[i] = d.w - zq[r0 + i])
        if constexpr (REL && NDP) { IDW_LAYER(lg[i] -= kq[r0 + i]) }
#pragma unroll
        for (int i = 0; i < GQ; ++i) zs = fmaf(aq[r0 + i], w[i], zs);
        if constexpr (NDP || PM != PM_GEN) { IDW_LAYER(w[i] = w[i] * c[i]) }
        if constexpr (NDP) { IDW_LAYER(acc[0][r0 + i] = fmaf(w[i], lg[i], acc[0][r0 + i])) }
        if constexpr (NDQ || NDX) {
          IDW_LAYER(f[i] = wr_times<PM>(w[i], c[i], f[i]))  // (w / r2)(z - Z)
          if constexpr (NDQ) {
            constexpr int G0 = NDP ? 1 : 0;
            IDW_LAYER(acc[G0][r0 + i] = fmaf(f[i], dx[i], acc[G0][r0 + i]))
            IDW_LAYER(acc[G0 + 1][r0 + i] = fmaf(f[i], dy[i], acc[G0 + 1][r0 + i]))
            if constexpr (DIM == 3) { IDW_LAYER(acc[G0 + 2][r0 + i] = fmaf(f[i], dz[i], acc[G0 + 2][r0 + i])) }
          }
          if constexpr (NDX) {
            IDW_LAYER(f[i] = (REL ? axq[r0 + i] : aq[r0 + i]) * f[i])
#pragma unroll
            for (int i = 0; i < GQ; ++i) {
              xs[0] = fmaf(f[i], dx[i], xs[0]);
              xs[1] = fmaf(f[i], dy[i], xs[1]);
              if constexpr (DIM == 3) xs[2] = fmaf(f[i], dz[i], xs[2]);
            }
          }
        }
      }
#undef IDW_LAYER
    };

    // Leave-one-out: the lanes whose points are the wave's own queries against those queries,
    // one query at a time, the self pair left out (at most R - 1 terms, added over the lanes in
    // FP32 and then with the other sums in FP64).
    auto near_self = [&](const P4<float>& d, int self, float& zs, float (&xs)[3]) {
      float vq[3], vz, va, vs, vk, vx;
      prepare(vq, vz, va, vs, vk, vx);
#pragma unroll 1
      for (int r = 0; r < R; ++r) {
        const float o[8] = {read_lane(vq[0], r), read_lane(vq[1], r), read_lane(vq[2], r), read_lane(vz, r),
                            read_lane(va, r),    read_lane(vs, r),    read_lane(vk, r),    read_lane(vx, r)};
        float p[NA];
#pragma unroll
        for (int c = 0; c < NA; ++c) p[c] = 0.f;
        if (self >= 0 && self != r) {
          float dx = o[0] - d.x, dy = o[1] - d.y, dz = 0.f;
          float r2 = dx * dx;
          r2 = fmaf(dy, dy, r2);
          if constexpr (DIM == 3) {
            dz = o[2] - d.z;
            r2 = fmaf(dz, dz, r2);
          }
          if constexpr (REL) r2 *= o[5];
          float w, f = 0.f, lg = 0.f;
          wterms<PM, NDQ || NDX, NDP>(r2, nhp, w, f, lg);
          if constexpr (REL && NDP) lg -= o[6];
          const float c = d.w - o[3];
          const float t = w * c;
          const float u = wr_times<PM>(t, c, f);
          zs = fmaf(o[4], w, zs);
          if constexpr (NDP) p[0] = t * lg;
          if constexpr (NDQ) {
            constexpr int G0 = NDP ? 1 : 0;
            p[G0] = u * dx;
            p[G0 + 1] = u * dy;
            if constexpr (DIM == 3) p[G0 + 2] = u * dz;
          }
          if constexpr (NDX) {
            const float v = (REL ? o[7] : o[4]) * u;
            xs[0] = fmaf(v, dx, xs[0]);
            xs[1] = fmaf(v, dy, xs[1]);
            if constexpr (DIM == 3) xs[2] = fmaf(v, dz, xs[2]);
          }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          float v = p[c];
#pragma unroll
          for (int x = 1; x < 64; x <<= 1) v += __shfl_xor(v, x);
          own[c] += lane == r ? v : 0.f;
        }
      }
    };

    // Adds the per-lane sums over the lanes: 8 of them at a time go through this wave's row of
    // zred as 8 rows of 64, of which lane l adds 8 values of row l / 8 into its FP64 sum.  They
    // are widened before they are added, so that at most 64 FP32 terms lie between two FP64
    // additions (0.2-0.8% of the sweep: 131,072 x 131,072, p = 2, 4.94 -> 4.95 ms).
    // With GSUM, lanes 8 i .. 8 i + 7 add theirs together and lane 8 i adds that to its query's
    // partial (component c of query 8 h + i in round k = (c R) / 8 + h).
    auto flush = [&](bool start, bool last) {
      float* row = zred[wave];
#pragma unroll
      for (int k = 0; k < NR; ++k) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int e = 8 * k + i;
          if (e < R * NC) {
            row[i * 64 + lane] = acc[e / R][e % R];
            acc[e / R][e % R] = 0.f;
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const P4<float> a = *reinterpret_cast<const P4<float>*>(&row[lane * 8]);
        const P4<float> b = *reinterpret_cast<const P4<float>*>(&row[lane * 8 + 4]);
        const double v = ((static_cast<double>(a.x) + a.y) + (static_cast<double>(a.z) + a.w)) +
                         ((static_cast<double>(b.x) + b.y) + (static_cast<double>(b.z) + b.w));
        if constexpr (LSUM)
          lsum[wave][k][lane] += v;  // this lane's own element
        else if constexpr (!GSUM)
          sums[k] += v;
        else {
          const int c = 8 * k / R, r = 8 * k % R + lane / 8;
          double t = v;
#pragma unroll
          for (int x = 1; x < 8; x <<= 1) t += shfl_xor64(t, x);
          if constexpr (EXCL) {
            if (last) t += static_cast<double>(__shfl(own[c], r));
          }
          if ((lane & 7) == 0 && qw + r < m) {
            double* o = &part_q[static_cast<int64_t>(blockIdx.y) * m + qw + r].x + (NDP ? c : c + 1);
            *o = start ? t : *o + t;
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
    };

    fetch(0);
    put(0);
    __syncthreads();
    for (int t = 0; t < ntiles; ++t) {
      if (t + 1 < ntiles) fetch(t + 1);
      const int64_t jt = jb + static_cast<int64_t>(t) * TILE;
      const auto& tl = tile[t & 1];
      const int cnt = static_cast<int>(je - jt < TILE ? je - jt : TILE);  // points of the tile
      // where the wave's own queries lie among them (leave-one-out)
      const int64_t at = qw - jt;
      const bool diag = EXCL && at < TILE && at > -R;
      const int selfat = diag ? static_cast<int>(at) : TILE;
      const bool plain = cnt == TILE && !diag;
      const int64_t j = jt + tid;
      double zold = 0.0;  // this thread's element of the dz row, loaded ahead
      if (!first && j < je) zold = zrow[j];
      P4<float> d = tl.get(lane);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const P4<float> dn = tl.get(((b + 1) & (NB - 1)) * 64 + lane);
        const int pt = b * 64 + lane;
        float zs = 0.f, xs[3] = {0.f, 0.f, 0.f};
        uint64_t on = ~uint64_t(0);  // the lanes that take part
        if (!plain)
          on = __ballot(pt < cnt && static_cast<unsigned>(pt - selfat) >= static_cast<unsigned>(R));
        if (__builtin_amdgcn_inverse_ballot_w64(on)) batch(d, zs, xs);
        zred[wave][pt] = zs;
        if constexpr (NDX) {
#pragma unroll
          for (int e = 0; e < DIM; ++e) xred[wave][e * TILE + pt] = xs[e];
        }
        d = dn;
      }
      if (EXCL && diag) {  // the points that the loop left out
#pragma unroll 1
        for (int b = 0; b < NB; ++b) {
          const int pt = b * 64 + lane;
          const int self = static_cast<unsigned>(pt - selfat) < static_cast<unsigned>(R) && pt < cnt ? pt - selfat : -1;
          if (!__any(self >= 0)) continue;
          float zs = 0.f, xs[3] = {0.f, 0.f, 0.f};
          near_self(tl.get(pt), self, zs, xs);
          if (self >= 0) {
            zred[wave][pt] = zs;
            if constexpr (NDX) {
#pragma unroll
              for (int e = 0; e < DIM; ++e) xred[wave][e * TILE + pt] = xs[e];
            }
          }
        }
      }
      double xold[3] = {0.0, 0.0, 0.0};  // loaded here, where the batches' registers are free
      if constexpr (GSUM) {
        if (!first && j < je) {
#pragma unroll
          for (int e = 0; e < DIM; ++e) xold[e] = xrow[j * DIM + e];
        }
      }
      __syncthreads();  // zred complete; tile t fully consumed
      // dz: add the waves' sums in a fixed order and fold into this group's row.  FP32: 16 terms
      // a wave and three additions over the waves, 19 roundings at most (in FP64 the additions
      // cost 0.5% with dz alone, but 12% with the 3-D X sums, whose registers then spill).  The stores
      // come after the next tile has been put: a wait for its loads, which were issued before
      // them, would otherwise wait for the stores too.
      auto waves = [&](const float* v, int stride) {
        return static_cast<double>(((v[0] + v[stride]) + (v[2 * stride] + v[3 * stride])) +
                                   ((v[4 * stride] + v[5 * stride]) + (v[6 * stride] + v[7 * stride])));
      };
      zold += waves(&zred[0][tid], TILE);
      double xv[3];
      if constexpr (NDX) {
#pragma unroll
        for (int e = 0; e < DIM; ++e) xv[e] = xold[e] + waves(&xred[0][e * TILE + tid], DIM * TILE);
      }
      if (t + 1 < ntiles) put((t + 1) & 1);
      __syncthreads();
      if (j < je) {
        zrow[j] = zold;
        if constexpr (NDX) {
#pragma unroll
          for (int e = 0; e < DIM; ++e) xrow[j * DIM + e] = GSUM || first ? xv[e] : xrow[j * DIM + e] + xv[e];
        }
      }
      if constexpr (NC > 0) {
        if ((t + 1) % (kFlush / TILE) == 0 || t + 1 == ntiles)
          flush(t < kFlush / TILE, t + 1 == ntiles);  // own row of zred only
      }
    }
    if constexpr (NC > 0 && !GSUM) {
      // lanes 8 i .. 8 i + 7 hold sum 8 k + i: query r = 8 h + i of component c at k = (c R + 8 h) / 8
#pragma unroll
      for (int h = 0; h < R / 8; ++h) {
        const int64_t i = qw + 8 * h + lane / 8;
        double v[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          double t;
          if constexpr (LSUM)
            t = lsum[wave][(c * R) / 8 + h][lane];
          else
            t = sums[(c * R) / 8 + h];
#pragma unroll
          for (int x = 1; x < 8; x <<= 1) t += shfl_xor64(t, x);
          if constexpr (EXCL) t += static_cast<double>(__shfl(own[c], 8 * h + lane / 8));
          v[NDP ? c : c + 1] = t;
        }
        if ((lane & 7) == 0 && i < m) {
          const double4 o = make_double4(v[0], v[1], v[2], v[3]);
          part_q[static_cast<int64_t>(blockIdx.y) * m + i] = o;
        }
      }
    }
  }
  // A group without any query block still owns a partial row: make it zero.
  if (first) {
    for (int64_t j = jb + tid; j < je; j += NT) {
      zrow[j] = 0.0;
      if constexpr (NDX) {
#pragma unroll
        for (int e = 0; e < DIM; ++e) xrow[j * DIM + e] = 0.0;
      }
    }
  }
}

template <typename T, int DIM, int L, int PM, bool REL = false>
hipError_t launch_bwd_fused_t(const BwdArgs& a, int groups, int ranges, int64_t chunk, hipStream_t st) {
  const bool ndp = (a.flags & 0x4u) != 0, ndq = (a.flags & 0x8u) != 0, ndx = a.part_x != nullptr;
  dim3 grid(static_cast<unsigned>(groups), static_cast<unsigned>(ranges));
  const T nhp = static_cast<T>(-0.5 * a.p);
  const T* sz = static_cast<const T*>(a.saved_z);
  const T* go = static_cast<const T*>(a.grad_out);
#define IDW_BF_ARGS                                                                                       \
  a.data, a.n, a.query, a.m, chunk, groups, nhp, a.flags, a.hdr, sz, go, a.saved_den, a.part_q, a.part_z, \
      a.part_x, a.route
#define IDW_BF(DP, DQ, DX)                                                                                  \
  do {                                                                                                      \
    if constexpr (sizeof(T) == 8)                                                                           \
      hipLaunchKernelGGL((k_bwd_fused<T, DIM, L, PM, 2, DP, DQ, DX>), grid, dim3(kFNT64), 0, st,            \
                         IDW_BF_ARGS);                                                                      \
    else if (a.flags & 1u)                                                                                  \
      hipLaunchKernelGGL((k_bwd_fused32<DIM, L, PM, DP, DQ, DX, REL, true>), grid, dim3(64 * kFusedWaves),  \
                         0, st, IDW_BF_ARGS, a.p);                                                          \
    else                                                                                                    \
      hipLaunchKernelGGL((k_bwd_fused32<DIM, L, PM, DP, DQ, DX, REL, false>), grid, dim3(64 * kFusedWaves), \
                         0, st, IDW_BF_ARGS, a.p);                                                          \
  } while (0)
  // The data-coordinate gradient is instantiated with both query-direction sums (they share
  // its per-pair factors); merges write only what was requested.  With relative weights
  // every request runs here, dz alone included.
  if (ndx)
    IDW_BF(true, true, true);
  else if (ndp && ndq)
    IDW_BF(true, true, false);
  else if (ndp)
    IDW_BF(true, false, false);
  else if (ndq)
    IDW_BF(false, true, false);
  else if constexpr (REL)
    IDW_BF(false, false, false);
  else
    return hipErrorInvalidValue;
#undef IDW_BF
#undef IDW_BF_ARGS
  return hipGetLastError();
}

template <typename T, int DIM, int L>
hipError_t bwd_fused_pm(const BwdArgs& a, int groups, int ranges, int64_t chunk, hipStream_t st) {
  if constexpr (sizeof(T) == 4) {
    if (a.rel)
      return a.pmode == PM_GEN ? launch_bwd_fused_t<T, DIM, L, PM_GEN, true>(a, groups, ranges, chunk, st)
                               : hipErrorInvalidValue;
  } else {
    if (a.rel) return hipErrorInvalidValue;
  }
  switch (a.pmode) {
    case PM_1: return launch_bwd_fused_t<T, DIM, L, PM_1>(a, groups, ranges, chunk, st);
    case PM_2: return launch_bwd_fused_t<T, DIM, L, PM_2>(a, groups, ranges, chunk, st);
    case PM_3: return launch_bwd_fused_t<T, DIM, L, PM_3>(a, groups, ranges, chunk, st);
    case PM_4: return launch_bwd_fused_t<T, DIM, L, PM_4>(a, groups, ranges, chunk, st);
    default: return launch_bwd_fused_t<T, DIM, L, PM_GEN>(a, groups, ranges, chunk, st);
  }
}

}  // namespace idw
