// Wavefront reductions of float64 sums without LDS traffic.
//
// __shfl_xor of a double is two ds_bpermute operations on the CU's one LDS
// pipe, and a chain of six of them per value; an Arnoldi pass that reduces up
// to 32 values per wavefront spent more time there than in its loads on small
// grids.  Here lanes exchange through the VALU: v_permlane32_swap /
// v_permlane16_swap across halves and rows, DPP inside a 16-lane row.  Every
// function sums in a fixed order (bitwise reproducible).  Measured against the
// shuffles: a 32^2 Euler step 27.0 -> 23.3 ms, two 512^2 midpoint steps 11.0 ->
// 9.9 ms, a 48^3 solve 7.1 -> 6.5 ms; 128^3 and 256^3 (HBM bound) unchanged.
#pragma once
#include <hip/hip_runtime.h>

namespace llg {

// DPP controls whose lane pairs differ in lane bit 3, 2, 1, 0: rotation of a
// 16-lane row by 8, mirror inside 8 lanes (flips bits 2..0), xor 2, xor 1.
constexpr int kDppBit3 = 0x128, kDppBit2 = 0x141, kDppBit1 = 0x4E, kDppBit0 = 0xB1;

template <int CTRL>
__device__ __forceinline__ double dpp_get(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}

// One halving step across lane bit BIT (5 or 4): on return the lanes with the
// bit clear hold a's sum over the lane pair, those with it set hold b's.
template <int BIT>
__device__ __forceinline__ double swap_add(double a, double b) {
  unsigned lo0, lo1, hi0, hi1;
  if constexpr (BIT == 5) {
    const auto l = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
    lo0 = l[0]; lo1 = l[1]; hi0 = h[0]; hi1 = h[1];
  } else {
    const auto l = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
    lo0 = l[0]; lo1 = l[1]; hi0 = h[0]; hi1 = h[1];
  }
  return __hiloint2double(int(hi0), int(lo0)) + __hiloint2double(int(hi1), int(lo1));
}

// The same across lane bit 3..0 with the DPP control CTRL of that bit.
template <int CTRL>
__device__ __forceinline__ double dpp_halve(double a, double b, bool set) {
  const double keep = set ? b : a, send = set ? a : b;
  return keep + dpp_get<CTRL>(send);
}

// Sum of v over the wavefront, in every lane.
__device__ __forceinline__ double wave_sum(double v) {
  v = swap_add<5>(v, v);
  v = swap_add<4>(v, v);
  v += dpp_get<kDppBit3>(v);
  v += dpp_get<kDppBit2>(v);
  v += dpp_get<kDppBit1>(v);
  v += dpp_get<kDppBit0>(v);
  return v;
}

// Number of values (a power of two, at most 32) of one multi-value reduction.
__host__ __device__ constexpr int wave_pow2(int n) {
  return n <= 1 ? 1 : n <= 2 ? 2 : n <= 4 ? 4 : n <= 8 ? 8 : n <= 16 ? 16 : 32;
}
// Index of the value that a lane holds after wave_sums<N> (its high bits).
template <int N>
__device__ __forceinline__ int wave_sums_index(int lane) {
  return (lane * wave_pow2(N)) >> 6;
}

// Sums of N <= 32 values over the wavefront: lane l returns the sum of v[i],
// i = wave_sums_index<N>(l) (0 for i >= N).  Each step halves the values a
// lane holds, so N values take about N exchanges instead of 6 N.
template <int N>
__device__ __forceinline__ double wave_sums(const double (&v)[N]) {
  constexpr int M = wave_pow2(N);
  static_assert(N >= 1 && N <= 32, "at most 32 values");
  const int lane = threadIdx.x & 63;
  double a[M];
#pragma unroll
  for (int i = 0; i < M; ++i) a[i] = i < N ? v[i] : 0.0;
  if constexpr (M >= 2) {
#pragma unroll
    for (int i = 0; i < M / 2; ++i) a[i] = swap_add<5>(a[i], a[i + M / 2]);
  } else {
    a[0] = swap_add<5>(a[0], a[0]);
  }
  if constexpr (M >= 4) {
#pragma unroll
    for (int i = 0; i < M / 4; ++i) a[i] = swap_add<4>(a[i], a[i + M / 4]);
  } else {
    a[0] = swap_add<4>(a[0], a[0]);
  }
  if constexpr (M >= 8) {
#pragma unroll
    for (int i = 0; i < M / 8; ++i) a[i] = dpp_halve<kDppBit3>(a[i], a[i + M / 8], lane & 8);
  } else {
    a[0] += dpp_get<kDppBit3>(a[0]);
  }
  if constexpr (M >= 16) {
#pragma unroll
    for (int i = 0; i < M / 16; ++i) a[i] = dpp_halve<kDppBit2>(a[i], a[i + M / 16], lane & 4);
  } else {
    a[0] += dpp_get<kDppBit2>(a[0]);
  }
  if constexpr (M >= 32) a[0] = dpp_halve<kDppBit1>(a[0], a[1], lane & 2);
  else a[0] += dpp_get<kDppBit1>(a[0]);
  a[0] += dpp_get<kDppBit0>(a[0]);
  return a[0];
}

// Sums of N values over the wavefront into dst[0 .. N) (LDS), 32 at a time.
template <int N>
__device__ __forceinline__ void wave_sums_store(const double (&v)[N], double* __restrict__ dst) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int i0 = 0; i0 < N; i0 += 32) {
    constexpr int FULL = N < 32 ? N : 32;
    constexpr int REST = N % 32 ? N % 32 : FULL;
    if (i0 + 32 <= N || N < 32) {
      double c[FULL];
#pragma unroll
      for (int i = 0; i < FULL; ++i) c[i] = v[i0 + i < N ? i0 + i : 0];
      const double s = wave_sums<FULL>(c);
      const int q = wave_sums_index<FULL>(lane);
      if ((lane & (64 / wave_pow2(FULL) - 1)) == 0 && q < FULL) dst[i0 + q] = s;
    } else {
      double c[REST];
#pragma unroll
      for (int i = 0; i < REST; ++i) c[i] = v[i0 + i < N ? i0 + i : 0];
      const double s = wave_sums<REST>(c);
      const int q = wave_sums_index<REST>(lane);
      if ((lane & (64 / wave_pow2(REST) - 1)) == 0 && q < REST) dst[i0 + q] = s;
    }
  }
}

// Sums of nv rows of nb values (value-major) by the first NW wavefronts of a
// block, four rows at a time per wavefront; dst(q, sum) on one lane per row.
template <int NW, class F>
__device__ __forceinline__ void rows_sum(const double* __restrict__ part, int nb, int nv, F&& dst) {
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int q0 = wv; q0 < nv; q0 += 4 * NW) {
    const double* r[4];
    double t[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      r[k] = part + (long long)(q0 + k * NW < nv ? q0 + k * NW : q0) * nb;
      t[k] = 0.0;
    }
#pragma unroll 4
    for (int b = lane; b < nb; b += 64) {
#pragma unroll
      for (int k = 0; k < 4; ++k) t[k] += r[k][b];
    }
    const double s = wave_sums<4>(t);
    const int q = q0 + wave_sums_index<4>(lane) * NW;
    if ((lane & 15) == 0 && q < nv) dst(q, s);
  }
}

}  // namespace llg
