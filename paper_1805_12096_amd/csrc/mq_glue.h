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

// Value of lane (l - N) mod 16 (row_ror) or of another lane of the quad, of the same row of 16 lanes.
template <int CTRL>
__device__ __forceinline__ float dpp16_f(float x) {
  return __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, 0xF, 0xF, true));
}

// Sum of a row of 256 CH floats, lane l of the wave holding elements 256 c + 4 l + t as x[c][t]; the same in every lane.
// The additions are those of k_layer_norm, a thread per element of a piece and four waves, in the same order -- element
// by element over the pieces, a tree over 64 neighbours, four of those one after the other -- so that the rows come out the
// same whichever kernel normalises them: a last bit decides on which side of a half an integer falls further on, and in a
// decoder layer of one sentence that can move a tensor's maximum with it.
template <int CH>
__device__ __forceinline__ float row_sum_f(const float (&x)[CH][4]) {
  float p[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    p[t] = x[0][t];
#pragma unroll
    for (int c = 1; c < CH; ++c) p[t] += x[c][t];
    // element 64 w + e sits in lane 16 w + e / 4 as t = e % 4: the tree's steps 32, 16, 8, 4 are lanes 8, 4, 2, 1 apart
    p[t] += dpp16_f<0x128>(p[t]);      // row_ror:8
    p[t] += dpp16_f<0x124>(p[t]);      // row_ror:4 (lanes 8 apart hold the same value by now)
    p[t] += dpp16_f<0x4E>(p[t]);       // quad_perm [2,3,0,1]
    p[t] += dpp16_f<0xB1>(p[t]);       // quad_perm [1,0,3,2]
  }
  const unsigned s = __float_as_uint((p[0] + p[2]) + (p[1] + p[3]));
  auto part = [&](int w) { return __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)s, 16 * w)); };
  return ((part(0) + part(1)) + part(2)) + part(3);
}

__device__ __forceinline__ float sigmoidf_(float z) { return __fdiv_rn(1.0f, 1.0f + expf(-z)); }

}  // namespace mq
