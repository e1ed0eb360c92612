// Device helpers shared by the librsv kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "rsv_internal.h"

namespace rsv {

template <class R> struct CxT;
template <> struct CxT<double> { using T = double2; };
template <> struct CxT<float> { using T = float2; };
template <class R> using Cx = typename CxT<R>::T;

// The hardware hands workgroup w to XCD w % 8.  Give every XCD one contiguous range of tile
// indices, so that neighbouring tiles (which share cache lines in the strided passes) are
// scheduled back to back on the same XCD and its L2.
__device__ __forceinline__ uint32_t xcd_remap(uint32_t bid, uint32_t nblk) {
  if (nblk < 8 || (nblk & 7u) != 0) return bid;
  return (bid & 7u) * (nblk >> 3) + (bid >> 3);
}

// ------------------------------------------------------------------ sums inside a wave (DPP)
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0u, (uint32_t)b, CTRL, 0xF, 0xF, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0u, (uint32_t)(b >> 32), CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, (uint32_t)__builtin_amdgcn_update_dpp(
                                       0u, __builtin_bit_cast(uint32_t, v), CTRL, 0xF, 0xF, true));
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppXor3 = 0x1B, kDppHalfMirror = 0x141, kDppMirror = 0x140;
constexpr int kDppFromBelow = 0x138, kDppFromAbove = 0x130;  // lane i takes lane i - 1 / i + 1

__device__ __forceinline__ double lane_value(double v, int lane) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), lane);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

struct OpAdd { __device__ double operator()(double a, double b) const { return a + b; } };
struct OpMin { __device__ double operator()(double a, double b) const { return fmin(a, b); } };
struct OpMax { __device__ double operator()(double a, double b) const { return fmax(a, b); } };

// Reduction over rows of 16 lanes, the same value in all of a row's lanes.
template <class Op>
__device__ __forceinline__ double row_reduce(double v, Op op) {
  v = op(v, dpp<kDppXor1>(v));
  v = op(v, dpp<kDppXor2>(v));
  v = op(v, dpp<kDppHalfMirror>(v));
  return op(v, dpp<kDppMirror>(v));
}
// Over the wave, uniform.  Every lane must be active.
template <class Op>
__device__ __forceinline__ double wave_reduce(double v, Op op) {
  v = row_reduce(v, op);
  return op(op(lane_value(v, 0), lane_value(v, 16)), op(lane_value(v, 32), lane_value(v, 48)));
}
__device__ __forceinline__ double wave_total(double v) { return wave_reduce(v, OpAdd()); }

// Sum of a double over a 256-thread workgroup; the result is valid in thread 0.  Fixed
// reduction tree, so the result is bitwise reproducible.
__device__ __forceinline__ double block_sum_256(double v, double* red /* >= 4 doubles */) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) red[wave] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0) r = (red[0] + red[1]) + (red[2] + red[3]);
  __syncthreads();
  return r;
}

// acc + (x^2 + y^2) with every product and sum rounded separately, so that every kernel
// that accumulates a squared norm of the same values gets the same bits.  The pragma keeps
// the operations out of FMA contraction after inlining (the _rn intrinsics alone do not).
__device__ __forceinline__ double norm_add(double acc, double x, double y) {
#pragma clang fp contract(off)
  return acc + (x * x + y * y);
}

// Fixed grid for the streaming vector kernels: 8 workgroups per CU on 256 CUs at most.
inline uint32_t stream_grid(size_t count, int per_thread) {
  size_t per_wg = (size_t)kBlock * per_thread;
  size_t g = (count + per_wg - 1) / per_wg;
  if (g > 2048) g = 2048;
  if (g < 1) g = 1;
  return (uint32_t)g;
}

}  // namespace rsv
