// device.hpp -- device-side helpers shared by the kernel sources.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>
#include <type_traits>

namespace huge2 {

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;

constexpr int cmax(int a, int b) { return a > b ? a : b; }
constexpr int gcd_c(int a, int b) { return b == 0 ? a : gcd_c(b, a % b); }
constexpr int lcm3(int a, int b, int c) {
  return (a / gcd_c(a, b) * b) / gcd_c(a / gcd_c(a, b) * b, c) * c;
}
// f(integral_constant<int, u>) for u = 0 .. N-1, unrolled at compile time.
template <int N, int I = 0, typename F>
__device__ __forceinline__ void unroll_stages(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>());
    unroll_stages<N, I + 1>(f);
  }
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// 16-byte store of output data that nothing in the kernel reads back, with
// the non-temporal (streaming) cache policy.
__device__ __forceinline__ void store_stream16(void* p, uint4 v) {
  const u32x4 t = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(t, (u32x4*)p);
}

// Workgroups are dealt to the 8 XCDs round-robin (id mod 8).  Map them so
// that each XCD runs one contiguous run of the work list: neighbouring
// tiles share input rows and weight blocks, which then stay in that XCD's L2.
__device__ __forceinline__ int xcd_remap(int b, int g) {
  const int g8 = (g + 7) >> 3, r = g & 7, x = b & 7, y = b >> 3;
  if (r == 0 || x < r) return x * g8 + y;
  return r * g8 + (x - r) * (g8 - 1) + y;
}

// The epilogue's elementwise function (huge2_activation): 0 none, 1 max(v, 0),
// 2 tanh(v).  act is uniform over the launch.
__device__ __forceinline__ float activate(float v, int act) {
  return act == 1 ? fmaxf(v, 0.f) : act == 2 ? tanhf(v) : v;
}

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
  // v_cvt_pk_bf16_f32: round to nearest even, NaN stays a (quiet) NaN
  return __builtin_bit_cast(uint16_t, (__bf16)f);
}

// Two floats to bf16 (round to nearest even) in one 32-bit word, lo in the
// low half: one v_cvt_pk_bf16_f32 with both sources.
__device__ __forceinline__ uint32_t pack_bf16x2_rne(float lo, float hi) {
  typedef float f2_t __attribute__((ext_vector_type(2)));
  typedef __bf16 b2_t __attribute__((ext_vector_type(2)));
  const f2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, b2_t));
}

__device__ __forceinline__ uint32_t fast_div(uint32_t v, uint32_t mul, uint32_t shift) {
  return (uint32_t)(((uint64_t)v * mul) >> shift);
}
template <typename T>
__device__ __forceinline__ float to_f32(T v) {
  if constexpr (std::is_same<T, uint16_t>::value)
    return __uint_as_float((uint32_t)v << 16);
  else
    return __uint_as_float(v);
}

}  // namespace huge2
