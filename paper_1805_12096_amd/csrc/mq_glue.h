// Device functions of the float glue that more than one translation unit evaluates: one definition, one rounding.
#pragma once

#include <hip/hip_runtime.h>

#include "mq_internal.h"

namespace mq {

// Value of lane (l - N) mod 16 (row_ror) or of another lane of the quad, of the same row of 16 lanes.
template <int CTRL>
__device__ __forceinline__ float dpp16_f(float x) {
  return __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, 0xF, 0xF, true));
}

// op(own, lane ^ 32's) and op(own, lane ^ 16's) value: the swap of two copies leaves one operand in each.
template <typename Op>
__device__ __forceinline__ float across32_f(float v, Op op) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <typename Op>
__device__ __forceinline__ float across16_f(float v, Op op) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// The butterfly over the 64 lanes, distances 32, 16, .. 1; the same in every lane.
template <typename Op>
__device__ __forceinline__ float wave_reduce_f(float v, Op op) {
  v = across32_f(v, op);
  v = across16_f(v, op);
  v = op(v, dpp16_f<0x128>(v));        // row_ror:8
  v = op(v, dpp16_f<0x124>(v));        // row_ror:4 (lanes 8 apart hold the same value by now)
  v = op(v, dpp16_f<0x4E>(v));         // quad_perm [2,3,0,1]
  return op(v, dpp16_f<0xB1>(v));      // quad_perm [1,0,3,2]
}
__device__ __forceinline__ float wave_sum_f(float v) {
  return wave_reduce_f(v, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ float wave_max_f(float v) {
  return wave_reduce_f(v, [](float a, float b) { return fmaxf(a, b); });
}

// Butterfly sums over groups of `grp` neighbouring lanes (a power of two up to 64), distances grp / 2 .. 1, of several values
// a step (one after the other they are serial chains).
template <int U, int C>
__device__ __forceinline__ void group_sums_f(float (&a)[U][C], unsigned grp) {
  auto add = [](float x, float y) { return x + y; };
  auto all = [&](auto step) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int c = 0; c < C; ++c) a[u][c] = step(a[u][c]);
  };
  if (grp >= 64) all([&](float v) { return across32_f(v, add); });
  if (grp >= 32) all([&](float v) { return across16_f(v, add); });
  if (grp >= 16) {
    all([&](float v) { return v + dpp16_f<0x128>(v); });
    all([&](float v) { return v + dpp16_f<0x124>(v); });
  } else if (grp == 8) {
    all([&](float v) { return v + __shfl_xor(v, 4, kWave); });
  }
  if (grp >= 4) all([&](float v) { return v + dpp16_f<0x4E>(v); });
  if (grp >= 2) all([&](float v) { return v + dpp16_f<0xB1>(v); });
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
