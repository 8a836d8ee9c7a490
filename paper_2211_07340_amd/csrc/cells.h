// The cell update of Eq. 1 in both number formats, shared by the alignment
// kernels.  Costs travel as uint32 bit patterns: every DP value is a sum of
// absolute differences (>= +0) or +inf, and IEEE encodings of non-negative
// floats order like their values, so one unsigned min3 serves both formats.
#pragma once
#include <type_traits>

#include "common.h"

namespace sdtw {
namespace {

struct FmtI16 {
  using qin = int16_t;
  using xlds = uint16_t;  // biased copy of the query in LDS
  static constexpr uint32_t kInf = 0xFFFFFFFFu;
  __device__ static __forceinline__ xlds to_lds(int16_t v) {
    return (uint16_t)((int32_t)v + (int32_t)kI16Bias);
  }
  __device__ static __forceinline__ uint32_t cell(uint32_t x, uint32_t y, uint32_t m) {
    const uint32_t d = x > y ? x - y : y - x;  // with the add: v_sad_u32
    return d + m;
  }
  __device__ static __forceinline__ void store_cost(void* cost, int32_t r, uint32_t v) {
    ((int32_t*)cost)[r] = (int32_t)v;
  }
  __device__ static __forceinline__ float value(uint32_t v) { return (float)v; }
};

struct FmtF32 {
  using qin = float;
  using xlds = uint32_t;
  static constexpr uint32_t kInf = 0x7F800000u;
  __device__ static __forceinline__ xlds to_lds(float v) { return __float_as_uint(v); }
  __device__ static __forceinline__ uint32_t cell(uint32_t x, uint32_t y, uint32_t m) {
    return __float_as_uint(fabsf(__uint_as_float(x) - __uint_as_float(y)) + __uint_as_float(m));
  }
  __device__ static __forceinline__ void store_cost(void* cost, int32_t r, uint32_t v) {
    ((float*)cost)[r] = __uint_as_float(v);
  }
  __device__ static __forceinline__ float value(uint32_t v) { return __uint_as_float(v); }
};

// f(integral_constant<int, I>) for I in [B, E), unrolled at compile time
template <int B, int E, class Fn>
__device__ __forceinline__ void static_for(Fn&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

__device__ __forceinline__ uint32_t min3u(uint32_t a, uint32_t b, uint32_t c) {
  return min(min(a, b), c);
}

__device__ __forceinline__ void wave_argmin(uint32_t& best, int32_t& bestj) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const uint32_t ob = (uint32_t)__shfl_xor((int)best, off);
    const int32_t oj = __shfl_xor(bestj, off);
    if (ob < best || (ob == best && oj < bestj)) {
      best = ob;
      bestj = oj;
    }
  }
}

}  // namespace
}  // namespace sdtw
