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

}  // namespace igemm_dev
