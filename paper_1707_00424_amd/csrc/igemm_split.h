// fp32 values as sums of three bf16 values (igemm_f32.hip has the arithmetic and its error).
#pragma once
#include "common.h"

namespace igemm_dev {

// V values -> three parts, two consecutive values per packed word (an odd last value beside a zero)
template <int V>
__device__ __forceinline__ void split_words(const float *v, uint32_t (&p)[3][(V + 1) / 2]) {
#pragma unroll
  for (int w = 0; w < (V + 1) / 2; ++w) {
    float a = v[2 * w], b = 2 * w + 1 < V ? v[2 * w + 1] : 0.f;
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      p[s][w] = f32x2_to_bf16x2(a, b);
      if (s < 2) a -= __uint_as_float(p[s][w] << 16), b -= __uint_as_float(p[s][w] & 0xffff0000u);
    }
  }
}

// Results of split products that plain fp32 has to give instead: infinite and NaN ones, and nonzero ones below 2^-64.  A part
// that would lie below bf16's smallest denormal is lost, up to 2^-134 of either operand: of a sum of 4096 products with
// values below 2^33, less than 2^-88, which is within an fp32 rounding of any result from 2^-64 up.  A result of exactly
// zero is kept (rows of zeros are common): its products all underflow in fp32 as well.
constexpr uint32_t kLeastTwice = 0x3f000000u;  // the bits of 2^-64, without the sign, times two
__device__ __forceinline__ bool out_of_split_range(float v) {
  const uint32_t u = __float_as_uint(v) << 1;
  return u >= 0xff000000u || u - 1 < kLeastTwice - 1;
}
// A quick look at many results: one and a half instructions each, and it also stops at zeros.
struct SplitRange {
  uint32_t least = ~0u;
  __device__ __forceinline__ void add(float v) { least = min(least, (__float_as_uint(v) << 1) + 0x01000000u); }
  __device__ __forceinline__ bool in_doubt() const { return __builtin_expect(__any(least < kLeastTwice + 0x01000000u), 0); }
};

}  // namespace igemm_dev
