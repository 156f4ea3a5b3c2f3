// Wavefront lane shifts, buffer words and order points of the generated row
// code (include before generated/stencils.inc).
#pragma once
#include <hip/hip_runtime.h>

namespace hhg {
namespace gen {
// DPP wave_shr:1 / wave_shl:1: the value held by lane L - 1 (from_prev) or
// L + 1 (from_next); the end lanes receive 0.
template <int CTRL>
__device__ __forceinline__ int lane_shift(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ __forceinline__ float lane_shift(float v) {
  return __int_as_float(lane_shift<CTRL>(__float_as_int(v)));
}
template <int CTRL>
__device__ __forceinline__ double lane_shift(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const int lo = lane_shift<CTRL>((int)(unsigned)(b & 0xffffffffull));
  const int hi = lane_shift<CTRL>((int)(unsigned)(b >> 32));
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
template <typename T>
__device__ __forceinline__ T from_prev(T v) {
  return lane_shift<0x138>(v);
}
template <typename T>
__device__ __forceinline__ T from_next(T v) {
  return lane_shift<0x130>(v);
}
}  // namespace gen
}  // namespace hhg

namespace hhg {
namespace gen {
// One word of a buffer (raw buffer load, bounds-checked by the resource: an
// offset outside it reads 0).
template <typename T>
__device__ __forceinline__ T buffer_word(__amdgpu_buffer_rsrc_t r, int voff, int soff);
template <>
__device__ __forceinline__ double buffer_word<double>(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}
template <>
__device__ __forceinline__ float buffer_word<float>(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
// Buffer resource over n bytes from p (gfx9 word 3: 32-bit data format).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, unsigned n) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)n, 0x00020000);
}
}  // namespace gen
}  // namespace hhg

namespace hhg {
namespace gen {
// Order points of the k-marching plane step.  The compiler otherwise makes
// the lane-shifted copies of every loaded word right after the loads and the
// multiply-adds much later, holding all copies at once (about 40 registers).
// An empty volatile asm that takes the accumulators (zm_order) and the next
// word (zm_word) as in/out register operands fixes the order word by word:
// it emits no instruction and touches no memory.
template <typename T, int R>
__device__ __forceinline__ void zm_order(T (&acc)[3][R]) {
#pragma unroll
  for (int s = 0; s < 3; ++s)
#pragma unroll
    for (int r = 0; r < R; ++r) asm volatile("" : "+v"(acc[s][r]));
}
template <typename T>
__device__ __forceinline__ T zm_word(T v) {
  asm volatile("" : "+v"(v));
  return v;
}
}  // namespace gen
}  // namespace hhg
