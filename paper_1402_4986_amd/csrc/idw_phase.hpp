// Phased evaluation of the FP32 sweeps (gfx950): the transcendentals of several pairs are
// issued as one run, between the plain arithmetic of those pairs.
//
// A SIMD issues plain FP32 instructions (add, mul, fma, mov on VGPRs) of two of its waves
// together, 2.1 cycles each instead of 4.2, as long as the two waves stay in step.  A
// transcendental takes 8.2 cycles, runs alone, and puts the waves out of step: with one
// reciprocal among six plain instructions every one of them costs 4.2 again (32.4 cycles per
// pair and wave, measured with register-only loops at 2 or 4 waves per SIMD).  Raising the
// wave's priority around a run of transcendentals lets each wave finish its run without
// being interleaved, after which the waves are in step again: 20.7 cycles for the same seven
// instructions at 4 waves per SIMD with runs of 8 or more (20.9 with runs of 4, 24.5 with
// single ones), 22.4 at 2 waves, 25 at 3, where one wave has no partner.  So the sweeps work
// on groups of pairs whose transcendentals form one run, and their register budgets are set
// for an even number of waves per SIMD.
//
// Records in LDS: a broadcast ds_read_b128 takes 4 cycles of the CU's LDS, a ds_read_b96 or
// ds_read2_b64 8, so 2-D records of FP32 are kept as a coordinate pair array and a value array,
// read four records at a time (three ds_read_b128), the others as four values.
#pragma once

#include "idw_device.hpp"

namespace idw {

// N records {x, y, (z), v} of the working type in LDS.
template <typename T, int DIM, int N>
struct RecTile {
  P4<T> r[N];
  __device__ __forceinline__ void put(int j, const P4<T>& d) { r[j] = d; }
  __device__ __forceinline__ P4<T> get(int j) const { return r[j]; }
};
// FP64 keeps the whole record: as a pair and a value its forward at
// p = 1 took 6.78 ms against 6.70 (131,072 points), at p = 3 7.95 against 7.79.
template <int N>
struct RecTile<float, 2, N> {
  using T = float;
  alignas(32) P2<T> xy[N];
  alignas(32) T v[N];
  __device__ __forceinline__ void put(int j, const P4<T>& d) {
    xy[j] = P2<T>{d.x, d.y};
    v[j] = d.z;
  }
  __device__ __forceinline__ P4<T> get(int j) const {
    const P2<T> c = xy[j];
    return P4<T>{c.x, c.y, v[j], T(0)};
  }
};

// G consecutive records (j a multiple of 4) in registers, as {x, y, z, v}.
template <int DIM, int G>
struct RecGroup {
  static_assert(G % 4 == 0, "groups are read four records at a time");
  float x[G], y[G], z[G], v[G];
  template <int N>
  __device__ __forceinline__ void load(const RecTile<float, DIM, N>& t, int j) {
    if constexpr (DIM == 2) {
#pragma unroll
      for (int g = 0; g < G; g += 4) {
        const P4<float> a = *reinterpret_cast<const P4<float>*>(&t.xy[j + g]);
        const P4<float> b = *reinterpret_cast<const P4<float>*>(&t.xy[j + g + 2]);
        const P4<float> c = *reinterpret_cast<const P4<float>*>(&t.v[j + g]);
        x[g] = a.x, y[g] = a.y, x[g + 1] = a.z, y[g + 1] = a.w;
        x[g + 2] = b.x, y[g + 2] = b.y, x[g + 3] = b.z, y[g + 3] = b.w;
        v[g] = c.x, v[g + 1] = c.y, v[g + 2] = c.z, v[g + 3] = c.w;
      }
    } else {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const P4<float> d = t.r[j + g];
        x[g] = d.x, y[g] = d.y, z[g] = d.z, v[g] = d.w;
      }
    }
  }
  // Squared distance of record g from q, in the order of sqdist.
  template <typename Q3>
  __device__ __forceinline__ float r2(const Q3& q, int g) const {
    const float dx = q[0] - x[g];
    const float dy = q[1] - y[g];
    float s = dx * dx;
    s = fmaf(dy, dy, s);
    if constexpr (DIM == 3) {
      const float dz = q[2] - z[g];
      s = fmaf(dz, dz, s);
    }
    return s;
  }
};

// Nothing is scheduled across the ends of a run.
__device__ __forceinline__ void run_begin() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_setprio(1);
}
__device__ __forceinline__ void run_end() {
  __builtin_amdgcn_s_setprio(0);
  __builtin_amdgcn_sched_barrier(0);
}

// The weights of N pairs from their squared distances, in place; the same operations per
// pair as weight<PM>.
template <int PM, int N>
__device__ __forceinline__ void weight_run(float (&r2)[N], float nhp) {
  float u[N];
  run_begin();
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if constexpr (PM == PM_2 || PM == PM_4)
      r2[i] = __builtin_amdgcn_rcpf(r2[i]);
    else if constexpr (PM == PM_GEN)
      r2[i] = __builtin_amdgcn_logf(r2[i]);
    else
      r2[i] = __builtin_amdgcn_rsqf(r2[i]);
  }
  if constexpr (PM == PM_25) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < N; ++i) u[i] = __builtin_amdgcn_sqrtf(r2[i]);
  }
  if constexpr (PM == PM_GEN) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < N; ++i) r2[i] *= nhp;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < N; ++i) r2[i] = __builtin_amdgcn_exp2f(r2[i]);
  }
  run_end();
  if constexpr (PM == PM_3) {
#pragma unroll
    for (int i = 0; i < N; ++i) r2[i] = r2[i] * r2[i] * r2[i];
  } else if constexpr (PM == PM_4) {
#pragma unroll
    for (int i = 0; i < N; ++i) r2[i] = r2[i] * r2[i];
  } else if constexpr (PM == PM_25) {
#pragma unroll
    for (int i = 0; i < N; ++i) r2[i] = r2[i] * r2[i] * u[i];
  }
}

}  // namespace idw
