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

__device__ __forceinline__ float sigmoidf_(float z) { return __fdiv_rn(1.0f, 1.0f + expf(-z)); }

}  // namespace mq
