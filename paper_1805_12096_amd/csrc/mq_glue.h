// Device functions of the float glue that more than one translation unit evaluates: one definition, one rounding.
#pragma once

#include <hip/hip_runtime.h>

#include "mq_internal.h"

namespace mq {

// Sum over the 64 lanes, the same in every lane.
__device__ __forceinline__ float wave_sum_f(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

// Sum of the CH x 4 elements of a row that a lane holds, in pairs: as short a chain of additions as with a thread per
// element.  Layer normalisation of 2048 rows of 256 / 512 / 768 / 1024, relative error against 64 bits: 7.10 / 7.10 / 7.11 /
// 7.13e-8 (k_layer_norm, a thread per element: 7.12 / 7.13 / 7.23 / 7.06e-8; 300 x 512 with a running sum 7.04e-8, so 6.98).
template <int CH>
__device__ __forceinline__ float lane_sum_f(const float (&x)[CH][4]) {
  static_assert(CH <= 4, "pieces of a row per lane");
  float p[4] = {};
#pragma unroll
  for (int c = 0; c < CH; ++c) p[c] = (x[c][0] + x[c][1]) + (x[c][2] + x[c][3]);
  return (p[0] + p[1]) + (p[2] + p[3]);
}

__device__ __forceinline__ float sigmoidf_(float z) { return __fdiv_rn(1.0f, 1.0f + expf(-z)); }

}  // namespace mq
