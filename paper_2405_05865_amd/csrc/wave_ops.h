// Wavefront sums of doubles without LDS: every exchange is a register move inside the
// vector unit (row permutations within 16 lanes, lane-half swaps across them), about a
// quarter of the latency of the LDS permute that a general shuffle takes. The order of the
// additions is fixed.
#pragma once
#include <hip/hip_runtime.h>

namespace wave_ops {

// row permutations that reach every lane of a 16-lane row: within quads, quad against quad,
// half row against half row
constexpr int kXor1 = 0xB1;        // quad_perm [1, 0, 3, 2]
constexpr int kXor2 = 0x4E;        // quad_perm [2, 3, 0, 1]
constexpr int kHalfMirror = 0x141; // lane i of each 8 takes lane 7 - i
constexpr int kRor8 = 0x128;       // lane i of each 16 takes lane i xor 8

template <int CTRL>
__device__ __forceinline__ double row_move(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}

template <int CTRL>
__device__ __forceinline__ float row_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

// sum over the 16 lanes of a row, valid in all of them
template <class T>
__device__ __forceinline__ T row_sum(T v) {
  v += row_move<kXor1>(v);
  v += row_move<kXor2>(v);
  v += row_move<kHalfMirror>(v);
  v += row_move<kRor8>(v);
  return v;
}

// a and b with the odd 16-lane rows of a exchanged for the even rows of b: the sum of the
// two results is a's pairs of rows in the even rows and b's in the odd ones
__device__ __forceinline__ double swap16_add(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
// the same with the 32-lane halves
__device__ __forceinline__ double swap32_add(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}

__device__ __forceinline__ float swap16_add(float a, float b) {
  const auto v = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(v[0]) + __uint_as_float(v[1]);
}
__device__ __forceinline__ float swap32_add(float a, float b) {
  const auto v = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(v[0]) + __uint_as_float(v[1]);
}

// sum over the 64 lanes, valid in every lane
__device__ __forceinline__ double wave_sum(double v) {
  v = row_sum(v);
  v = swap16_add(v, v);
  return swap32_add(v, v);
}

constexpr int log2i(int x) { return x <= 1 ? 0 : 1 + log2i(x / 2); }

template <int CTRL>
__device__ __forceinline__ double halve_row(double lower, double upper, bool up) {
  return (up ? upper : lower) + row_move<CTRL>(up ? lower : upper);
}

// one halving exchange: of the 2H values, the lanes with lane bit MSK set keep the upper H
template <int H, int MSK, int NV>
__device__ __forceinline__ void halve_step(double (&v)[NV], int lane) {
  const bool up = (lane & MSK) != 0;
#pragma unroll
  for (int q = 0; q < H; ++q) {
    if constexpr (MSK == 32) v[q] = swap32_add(v[q], v[q + H]);
    else if constexpr (MSK == 16) v[q] = swap16_add(v[q], v[q + H]);
    else if constexpr (MSK == 8) v[q] = halve_row<kRor8>(v[q], v[q + H], up);
    else if constexpr (MSK == 4) v[q] = halve_row<kHalfMirror>(v[q], v[q + H], up);
    else if constexpr (MSK == 2) v[q] = halve_row<kXor2>(v[q], v[q + H], up);
    else v[q] = halve_row<kXor1>(v[q], v[q + H], up);
  }
}

template <int MSK>
__device__ __forceinline__ double full_step(double v) {
  if constexpr (MSK == 32) return swap32_add(v, v);
  else if constexpr (MSK == 16) return swap16_add(v, v);
  else if constexpr (MSK == 8) return v + row_move<kRor8>(v);
  else if constexpr (MSK == 4) return v + row_move<kHalfMirror>(v);
  else if constexpr (MSK == 2) return v + row_move<kXor2>(v);
  else return v + row_move<kXor1>(v);
}

template <int H, int MSK, int NV>
__device__ __forceinline__ void scatter_steps(double (&v)[NV], int lane) {
  if constexpr (MSK >= 1) {
    if constexpr (H >= 1) halve_step<H, MSK, NV>(v, lane);
    else v[0] = full_step<MSK>(v[0]);
    scatter_steps<H / 2, MSK / 2, NV>(v, lane);
  }
}

// sums over the 64 lanes of NV values per lane (NV a power of two, at most 64): lane l
// returns the total of value l >> log2(64 / NV)
template <int NV>
__device__ __forceinline__ double scatter_sums(double (&v)[NV]) {
  static_assert(NV >= 1 && NV <= 64 && (NV & (NV - 1)) == 0, "a power of two up to the wavefront");
  scatter_steps<NV / 2, 32, NV>(v, (int)(threadIdx.x & 63));
  return v[0];
}

}  // namespace wave_ops
