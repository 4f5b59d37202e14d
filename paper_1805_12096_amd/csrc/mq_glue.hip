// Floating-point glue between the integer products of one greedy decode step of the averaging
// attention decoder (arxiv 1805.12096, Section 3.2: the decoder's self-attention is replaced by a
// cumulative uniform average that is updated from the last step only, followed by a feed-forward
// network and a gate; Section 3.1: source attention and the position-wise feed-forward block; every
// sub-layer ends in residual + layer normalisation).  All tensors are binary32, a decode step has a
// few hundred rows of model width, so every kernel here is one short pass over a few 100 KB: rows of up
// to 1024 floats in whole pieces of 256 are normalised by one wave in registers, other widths and the
// source attention take one workgroup per sentence with the row or the scores in LDS.
#include <type_traits>

#include "mq_glue.h"
#include "mq_grid_max.h"
#include "mq_internal.h"

namespace mq {

namespace {

constexpr int kT = 256;              // threads per workgroup
constexpr int kMaxRow = 8192;        // floats of a row kept in LDS (32 KB)
constexpr int kMaxScores = 4096;     // heads x source positions kept in LDS

// sum over the workgroup; every thread gets the result.  `red` holds kT / 64 floats.
__device__ __forceinline__ float block_sum(float v, float* red) {
  v = wave_sum_f(v);
  __syncthreads();                               // `red` may still be read from the call before
  if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = v;
  __syncthreads();
  float r = red[0];
#pragma unroll
  for (int k = 1; k < kT / kWave; ++k) r += red[k];
  return r;
}

// max over the workgroup of a non-negative value, to partial[blockIdx.x] (for the abs-max of the tensor
// this kernel writes, so that the quantizer of the next product needs no pass of its own)
__device__ __forceinline__ void block_absmax_out(float v, float* red, float* __restrict__ partial) {
  v = wave_max_f(v);
  __syncthreads();
  if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    float r = red[0];
#pragma unroll
    for (int k = 1; k < kT / kWave; ++k) r = fmaxf(r, red[k]);
    partial[blockIdx.x] = r;
  }
}

__global__ __launch_bounds__(kT) void k_running_average(const float* __restrict__ g_prev, const float* __restrict__ x,
                                                        size_t n, float tm1, float t, float* __restrict__ g,
                                                        float* __restrict__ partial, unsigned* __restrict__ clear,
                                                        unsigned nclear, float* __restrict__ partial_x) {
  __shared__ float red[kT / kWave];
  const size_t i = (size_t)blockIdx.x * kT + threadIdx.x;
  float v = 0.f, xv = 0.f;
  if (i < n) {
    xv = x[i];
    v = __fdiv_rn(__fmaf_rn(tm1, g_prev[i], xv), t);
    g[i] = v;
  }
  if (clear != nullptr && blockIdx.x == 0 && threadIdx.x < nclear) clear[threadIdx.x] = 0u;   // later kernels' maxima
  if (partial != nullptr) block_absmax_out(fabsf(v), red, partial);       // fmaxf drops NaN
  // max|x| as well (the gate's product takes [x, f] as its input and needs the maximum of both halves)
  if (partial_x != nullptr) block_absmax_out(fabsf(xv), red, partial_x);
}

// The same, four elements per thread, for 16-byte aligned tensors of a multiple of 4 elements: a quarter of the workgroups
// and of the partial maxima the next kernel has to read.
__global__ __launch_bounds__(kT) void k_running_average4(const float4* __restrict__ g_prev, const float4* __restrict__ x,
                                                         size_t n4, float tm1, float t, float4* __restrict__ g,
                                                         float* __restrict__ partial, unsigned* __restrict__ clear,
                                                         unsigned nclear, float* __restrict__ partial_x) {
  __shared__ float red[2][kT / kWave];
  const size_t i = (size_t)blockIdx.x * kT + threadIdx.x, ic = i < n4 ? i : n4 - 1;
  const float4 xv = x[ic], gv = g_prev[ic];
  const float4 v = make_float4(__fdiv_rn(__fmaf_rn(tm1, gv.x, xv.x), t), __fdiv_rn(__fmaf_rn(tm1, gv.y, xv.y), t),
                               __fdiv_rn(__fmaf_rn(tm1, gv.z, xv.z), t), __fdiv_rn(__fmaf_rn(tm1, gv.w, xv.w), t));
  if (i < n4) g[i] = v;
  if (clear != nullptr && blockIdx.x == 0 && threadIdx.x < nclear) clear[threadIdx.x] = 0u;
  if (partial == nullptr) return;
  // maxima of |g| and |x| (fmaxf drops NaN; non-negative floats order like their bits).  Threads past the end loaded the
  // last vector, which with g = g_prev another wave may have averaged already: their average counts for nothing.
  const float mg = i < n4 ? fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))) : 0.f;
  const float mx = fmaxf(fmaxf(fabsf(xv.x), fabsf(xv.y)), fmaxf(fabsf(xv.z), fabsf(xv.w)));
  const float wg = __uint_as_float(wave_max_u32(__float_as_uint(fmaxf(mg, 0.f))));
  const float wx = __uint_as_float(wave_max_u32(__float_as_uint(fmaxf(mx, 0.f))));
  if (threadIdx.x % kWave == 0) {
    red[0][threadIdx.x / kWave] = wg;
    red[1][threadIdx.x / kWave] = wx;
  }
  __syncthreads();
  if (threadIdx.x < 2 && (threadIdx.x == 0 || partial_x != nullptr)) {
    float r = red[threadIdx.x][0];
#pragma unroll
    for (int k = 1; k < kT / kWave; ++k) r = fmaxf(r, red[threadIdx.x][k]);
    (threadIdx.x == 0 ? partial : partial_x)[blockIdx.x] = r;
  }
}

__global__ __launch_bounds__(kT) void k_concat2(const float* __restrict__ a, unsigned da, const float* __restrict__ b,
                                                unsigned db, float* __restrict__ out, float* __restrict__ partial) {
  __shared__ float red[kT / kWave];
  const size_t m = blockIdx.x;
  float mx = 0.f;
  for (unsigned j = threadIdx.x; j < da + db; j += kT) {
    const float v = j < da ? a[m * da + j] : b[m * db + (j - da)];
    out[m * (da + db) + j] = v;
    mx = fmaxf(mx, fabsf(v));
  }
  if (partial != nullptr) block_absmax_out(mx, red, partial);
}

// One workgroup per row: h = GATED ? sigmoid(z[:d]) x + sigmoid(z[d:]) f : a;  y = LN(h + r) gamma + beta with
// the biased variance, mean and variance as two passes over the row held in LDS.
template <bool GATED>
__global__ __launch_bounds__(kT) void k_layer_norm(const float* __restrict__ a, const float* __restrict__ f,
                                                   const float* __restrict__ z, const float* __restrict__ r,
                                                   const float* __restrict__ gamma, const float* __restrict__ beta,
                                                   unsigned d, float eps, float* __restrict__ y,
                                                   float* __restrict__ partial) {
  __shared__ float row[kMaxRow];
  __shared__ float red[kT / kWave];
  const size_t m = blockIdx.x;
  float s = 0.f;
  for (unsigned j = threadIdx.x; j < d; j += kT) {
    float h;
    if (GATED) {
      const float x = a[m * d + j];
      h = sigmoidf_(z[m * 2 * d + j]) * x + sigmoidf_(z[m * 2 * d + d + j]) * f[m * d + j];
    } else {
      h = a[m * d + j];
    }
    h += r[m * d + j];
    row[j] = h;
    s += h;
  }
  const float mu = block_sum(s, red) / (float)d;
  float q = 0.f;
  for (unsigned j = threadIdx.x; j < d; j += kT) {
    const float c = row[j] - mu;
    q += c * c;
  }
  const float var = block_sum(q, red) / (float)d;
  const float inv = __fdiv_rn(1.0f, sqrtf(var + eps));
  float mx = 0.f;
  for (unsigned j = threadIdx.x; j < d; j += kT) {
    const float v = (row[j] - mu) * inv * gamma[j] + beta[j];
    y[m * d + j] = v;
    mx = fmaxf(mx, fabsf(v));
  }
  if (partial != nullptr) block_absmax_out(mx, red, partial);
}

// The same for rows of 256 CH floats (CH <= 4) with 16-byte alignment: one wave per row, the row in registers, everything
// the row needs asked for at once (gamma and beta included), reductions by lane moves -- no LDS, no barrier, and no
// second round trip to memory.
// The two kernels of a decoder layer (300 x 512) together with the averaging above: 65.3 -> 62.1 us per layer.
template <bool GATED, int CH>
__global__ __launch_bounds__(kWave) void k_layer_norm_wave(const float* __restrict__ a, const float* __restrict__ f,
                                                           const float* __restrict__ z, const float* __restrict__ r,
                                                           const float* __restrict__ gamma,
                                                           const float* __restrict__ beta, float eps,
                                                           float* __restrict__ y, float* __restrict__ partial) {
  constexpr unsigned d = 256u * CH;
  const size_t m = blockIdx.x;
  const unsigned lane = threadIdx.x;
  auto load = [&](const float* base, int c) { return reinterpret_cast<const float4*>(base)[c * 64 + lane]; };
  float4 av[CH], rv[CH], fv[CH], z1[CH], z2[CH], gv[CH], bv[CH];
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    av[c] = load(a + m * d, c);
    if constexpr (GATED) {
      fv[c] = load(f + m * d, c);
      z1[c] = load(z + m * 2 * d, c);
      z2[c] = load(z + m * 2 * d + d, c);
    }
    rv[c] = load(r + m * d, c);
  }
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    gv[c] = load(gamma, c);
    bv[c] = load(beta, c);
  }
  float h[CH][4], sq[CH][4];
#pragma unroll
  for (int c = 0; c < CH; ++c)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      auto at = [&](const float4& v) { return t == 0 ? v.x : t == 1 ? v.y : t == 2 ? v.z : v.w; };
      float v = at(av[c]);
      if constexpr (GATED) v = sigmoidf_(at(z1[c])) * v + sigmoidf_(at(z2[c])) * at(fv[c]);
      h[c][t] = v + at(rv[c]);
    }
  const float mu = row_sum_f(h) / (float)d;
#pragma unroll
  for (int c = 0; c < CH; ++c)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      h[c][t] -= mu;
      sq[c][t] = h[c][t] * h[c][t];
    }
  const float var = row_sum_f(sq) / (float)d;
  const float inv = __fdiv_rn(1.0f, sqrtf(var + eps));
  float mx = 0.f;
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const float4 v = make_float4(h[c][0] * inv * gv[c].x + bv[c].x, h[c][1] * inv * gv[c].y + bv[c].y,
                                 h[c][2] * inv * gv[c].z + bv[c].z, h[c][3] * inv * gv[c].w + bv[c].w);
    reinterpret_cast<float4*>(y + m * d)[c * 64 + lane] = v;
    mx = fmaxf(mx, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
  }
  if (partial != nullptr) {
    mx = __uint_as_float(wave_max_u32(__float_as_uint(mx)));
    if (lane == 0) partial[m] = mx;
  }
}

// One workgroup per sentence.  Scores of all heads and source positions into LDS (one wave per (head,
// position) pair, lanes over the head's width, four pairs per trip so that four rows of K are in flight
// per wave instead of one: the loop is bound by memory latency, not by arithmetic), softmax per head, then
// the context: thread j of the model width sums p[s] V[s][j] over the source positions.
constexpr int kTA = 512;             // threads of the attention kernel

__global__ __launch_bounds__(kTA) void k_cross_attention(const float* __restrict__ q, const float* __restrict__ K,
                                                         const float* __restrict__ V, unsigned S, unsigned d,
                                                         unsigned heads, float* __restrict__ ctx,
                                                         float* __restrict__ partial) {
  __shared__ float sc[kMaxScores];
  __shared__ float red[kTA / kWave];
  constexpr unsigned NWV = kTA / kWave;
  const size_t m = blockIdx.x;
  const unsigned dh = d / heads;
  const unsigned lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const float scale = __fdiv_rn(1.0f, sqrtf((float)dh));
  const float* qm = q + m * d;
  const float* Km = K + m * S * d;
  const float* Vm = V + m * S * d;
  const unsigned pairs = heads * S;
  for (unsigned p0 = wave; p0 < pairs; p0 += 4 * NWV) {
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    for (unsigned j = lane; j < dh; j += kWave) {
      float kv[4], qv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const unsigned p = p0 + u * NWV;
        const unsigned pc = p < pairs ? p : p0;                 // past the end: a valid pair again, result unused
        const unsigned h = pc / S, s = pc % S;
        kv[u] = Km[(size_t)s * d + h * dh + j];
        qv[u] = qm[h * dh + j];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[u] = fmaf(qv[u], kv[u], acc[u]);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float t = wave_sum_f(acc[u]);
      const unsigned p = p0 + u * NWV;
      if (lane == 0 && p < pairs) sc[p] = t * scale;
    }
  }
  __syncthreads();
  // softmax over the S positions of each head: one wave per head at a time
  for (unsigned h = wave; h < heads; h += NWV) {
    float mx = -INFINITY;
    for (unsigned s = lane; s < S; s += kWave) mx = fmaxf(mx, sc[h * S + s]);
    mx = wave_max_f(mx);
    float sum = 0.f;
    for (unsigned s = lane; s < S; s += kWave) {
      const float e = expf(sc[h * S + s] - mx);
      sc[h * S + s] = e;
      sum += e;
    }
    sum = wave_sum_f(sum);
    const float inv = __fdiv_rn(1.0f, sum);
    for (unsigned s = lane; s < S; s += kWave) sc[h * S + s] *= inv;
  }
  __syncthreads();
  float mx = 0.f;
  for (unsigned j = threadIdx.x; j < d; j += kTA) {
    const unsigned h = j / dh;
    float acc = 0.f;
    unsigned s = 0;
    for (; s + 4 <= S; s += 4) {                                   // four rows of V in flight
      const float v0 = Vm[(size_t)s * d + j], v1 = Vm[(size_t)(s + 1) * d + j], v2 = Vm[(size_t)(s + 2) * d + j],
                  v3 = Vm[(size_t)(s + 3) * d + j];
      acc = fmaf(sc[h * S + s], v0, acc);
      acc = fmaf(sc[h * S + s + 1], v1, acc);
      acc = fmaf(sc[h * S + s + 2], v2, acc);
      acc = fmaf(sc[h * S + s + 3], v3, acc);
    }
    for (; s < S; ++s) acc = fmaf(sc[h * S + s], Vm[(size_t)s * d + j], acc);
    ctx[m * d + j] = acc;
    mx = fmaxf(mx, fabsf(acc));
  }
  if (partial != nullptr) {
    // (the helper is written for kT threads; here the workgroup is kTA wide)
    mx = wave_max_f(mx);
    __syncthreads();
    if (lane == 0) red[wave] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
      float r = red[0];
#pragma unroll
      for (unsigned k = 1; k < NWV; ++k) r = fmaxf(r, red[k]);
      partial[blockIdx.x] = r;
    }
  }
}

// The same for the usual shapes (model width a multiple of 256, head width a power of two between 4 and 256):
// every load is a float4, a wave reads whole 1 KB pieces of a K row and all heads' partial dot products of one
// source position come out of one pass; the context phase splits the source positions over thread groups so
// that every thread has several rows of V in flight.
// Bound by memory latency (one sentence) and bytes in flight (hundreds): the lanes' dot products of a trip share the steps of
// the exchange between lanes, and up to 64 scores of a head are normalised in registers.
// AHEAD: K and the first rows of V are asked for together and without branches between the loads (past the end: the last row
// again), so that V's round trip is over when the scores are: for at most one workgroup per compute unit, where neither the
// registers (70 / 94 / 132 for d = 256 / 512 / 1024) nor the surplus loads are in anybody's way.  Otherwise nothing is asked
// for that is not needed, and 36 / 54 / 96 registers let four, four and two workgroups share a compute unit.  In us, K and V
// from the last-level cache, with and without AHEAD: d = 512, 100 sentences x 25 words 5.6, 6.2; x 8 4.9, 4.5; 300 x 25 9.1,
// 8.5; 600 x 1 8.2, 6.3; d = 1024, 100 x 14 6.9, 7.6; 300 x 25 19.0, 14.7.  Before the exchange was shared 300 x 25, d = 512
// took 8.5 us in the L2s, now 7.2 (4.3 TB/s), one sentence 6.0 and 4.7.
template <int CH, bool AHEAD>      // CH = d / 256: float4 pieces of a row per lane
__global__ __launch_bounds__(kTA) void k_cross_attention_fast(const float* __restrict__ q, const float* __restrict__ K,
                                                              const float* __restrict__ V, unsigned S, unsigned heads,
                                                              float* __restrict__ ctx, float* __restrict__ partial) {
  constexpr unsigned d = 256u * CH;
  constexpr unsigned NWV = kTA / kWave;
  constexpr unsigned COLS = d / 4;                 // float4 columns of a row
  constexpr unsigned SG = kTA / COLS;              // groups of threads that share the source positions
  static_assert(kTA % COLS == 0 && SG >= 1, "context phase layout");
  constexpr int kAhead = AHEAD ? 8 : 0;            // rows of V in registers: 32 source positions at d = 512
  __shared__ float sc[kMaxScores];
  __shared__ float4 part[SG > 1 ? kTA : 1];
  __shared__ float red[NWV];
  const size_t m = blockIdx.x;
  const unsigned dh = d / heads, grp = dh / 4;     // lanes per head inside a 256-float piece
  const unsigned lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const float scale = __fdiv_rn(1.0f, sqrtf((float)dh));
  const float4* q4 = reinterpret_cast<const float4*>(q + m * d);
  const float4* K4 = reinterpret_cast<const float4*>(K + m * S * d);
  const float4* V4 = reinterpret_cast<const float4*>(V + m * S * d);
  float4 qr[CH];
#pragma unroll
  for (int c = 0; c < CH; ++c) qr[c] = q4[c * 64 + lane];
  const unsigned col = threadIdx.x % COLS, sg = threadIdx.x / COLS;
  float4 va[AHEAD ? kAhead : 1];
  auto scores = [&](unsigned s0, auto first) {
    float4 kr[4][CH];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const unsigned s = s0 + u * NWV;
      if (AHEAD || s < S) {
#pragma unroll
        for (int c = 0; c < CH; ++c) kr[u][c] = K4[(size_t)(!AHEAD || s < S ? s : S - 1) * COLS + c * 64 + lane];
      } else {
#pragma unroll
        for (int c = 0; c < CH; ++c) kr[u][c] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
    if constexpr (AHEAD && decltype(first)::value) {
#pragma unroll
      for (int j = 0; j < kAhead; ++j) va[j] = V4[(size_t)(sg + j * SG < S ? sg + j * SG : S - 1) * COLS + col];
      __builtin_amdgcn_sched_barrier(0);
    }
    float a[4][CH];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int c = 0; c < CH; ++c)
        a[u][c] = fmaf(qr[c].x, kr[u][c].x, fmaf(qr[c].y, kr[u][c].y, fmaf(qr[c].z, kr[u][c].z, qr[c].w * kr[u][c].w)));
    group_sums_f(a, grp);
    if (lane % grp == 0)
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int c = 0; c < CH; ++c)
          if (s0 + u * NWV < S) sc[(c * 256 + 4 * lane) / dh * S + s0 + u * NWV] = a[u][c] * scale;
  };
  if (AHEAD || wave < S) scores(wave, std::true_type{});
  for (unsigned s0 = wave + 4 * NWV; s0 < S; s0 += 4 * NWV) scores(s0, std::false_type{});
  __syncthreads();
  for (unsigned h = wave; h < heads; h += NWV) {
    if (S <= kWave) {                                // the scores stay in a register
      const bool in = lane < S;
      const float x = in ? sc[h * S + lane] : -INFINITY;
      float mx = x;
      mx = wave_max_f(mx);
      const float e = in ? expf(x - mx) : 0.f;
      const float inv = __fdiv_rn(1.0f, wave_sum_f(e));
      if (in) sc[h * S + lane] = e * inv;
      continue;
    }
    float mx = -INFINITY;
    for (unsigned s = lane; s < S; s += kWave) mx = fmaxf(mx, sc[h * S + s]);
    mx = wave_max_f(mx);
    float sum = 0.f;
    for (unsigned s = lane; s < S; s += kWave) {
      const float e = expf(sc[h * S + s] - mx);
      sc[h * S + s] = e;
      sum += e;
    }
    sum = wave_sum_f(sum);
    const float inv = __fdiv_rn(1.0f, sum);
    for (unsigned s = lane; s < S; s += kWave) sc[h * S + s] *= inv;
  }
  __syncthreads();
  const unsigned h = (4 * col) / dh;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int j = 0; j < kAhead; ++j)
    if (sg + j * SG < S) {
      const float p0 = sc[h * S + sg + j * SG];
      acc.x = fmaf(p0, va[j].x, acc.x);
      acc.y = fmaf(p0, va[j].y, acc.y);
      acc.z = fmaf(p0, va[j].z, acc.z);
      acc.w = fmaf(p0, va[j].w, acc.w);
    }
  unsigned s = sg + kAhead * SG;
  for (; s + 3 * SG < S; s += 4 * SG) {
    const float4 v0 = V4[(size_t)s * COLS + col], v1 = V4[(size_t)(s + SG) * COLS + col],
                 v2 = V4[(size_t)(s + 2 * SG) * COLS + col], v3 = V4[(size_t)(s + 3 * SG) * COLS + col];
    const float p0 = sc[h * S + s], p1 = sc[h * S + s + SG], p2 = sc[h * S + s + 2 * SG], p3 = sc[h * S + s + 3 * SG];
    acc.x = fmaf(p3, v3.x, fmaf(p2, v2.x, fmaf(p1, v1.x, fmaf(p0, v0.x, acc.x))));
    acc.y = fmaf(p3, v3.y, fmaf(p2, v2.y, fmaf(p1, v1.y, fmaf(p0, v0.y, acc.y))));
    acc.z = fmaf(p3, v3.z, fmaf(p2, v2.z, fmaf(p1, v1.z, fmaf(p0, v0.z, acc.z))));
    acc.w = fmaf(p3, v3.w, fmaf(p2, v2.w, fmaf(p1, v1.w, fmaf(p0, v0.w, acc.w))));
  }
  for (; s < S; s += SG) {
    const float4 v0 = V4[(size_t)s * COLS + col];
    const float p0 = sc[h * S + s];
    acc.x = fmaf(p0, v0.x, acc.x);
    acc.y = fmaf(p0, v0.y, acc.y);
    acc.z = fmaf(p0, v0.z, acc.z);
    acc.w = fmaf(p0, v0.w, acc.w);
  }
  float mx = 0.f;
  if constexpr (SG > 1) {
    part[threadIdx.x] = acc;
    __syncthreads();
    if (sg == 0) {
#pragma unroll
      for (unsigned g = 1; g < SG; ++g) {
        const float4 o = part[g * COLS + col];
        acc.x += o.x; acc.y += o.y; acc.z += o.z; acc.w += o.w;
      }
    }
  }
  if (sg == 0) {
    reinterpret_cast<float4*>(ctx + m * d)[col] = acc;
    mx = fmaxf(fmaxf(fabsf(acc.x), fabsf(acc.y)), fmaxf(fabsf(acc.z), fabsf(acc.w)));
  }
  if (partial != nullptr) {
    mx = wave_max_f(mx);
    __syncthreads();
    if (lane == 0) red[wave] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
      float r = red[0];
#pragma unroll
      for (unsigned k = 1; k < NWV; ++k) r = fmaxf(r, red[k]);
      partial[blockIdx.x] = r;
    }
  }
}

}  // namespace

// The launchers' optional `partial` receives one max|output| per workgroup (glue_partials(...) of them).
size_t running_average_partials(size_t n) { return (n + kT - 1) / kT; }

static bool aligned16(const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }

int launch_running_average(const float* g_prev, const float* x, size_t n, int t, float* g, hipStream_t s, float* partial,
                           unsigned* clear, unsigned nclear, float* partial_x, unsigned* npartial) {
  const bool vec = n % 4 == 0 && aligned16(g_prev) && aligned16(x) && aligned16(g);
  const size_t blocks = vec ? (n / 4 + kT - 1) / kT : (n + kT - 1) / kT;
  if (blocks > 0x7FFFFFFFull || nclear > (unsigned)kT) return MQ_ERR_SHAPE;
  if (npartial != nullptr) *npartial = (unsigned)blocks;
  if (vec)
    hipLaunchKernelGGL(k_running_average4, dim3((unsigned)blocks), dim3(kT), 0, s, reinterpret_cast<const float4*>(g_prev),
                       reinterpret_cast<const float4*>(x), n / 4, (float)(t - 1), (float)t, reinterpret_cast<float4*>(g),
                       partial, clear, nclear, partial_x);
  else
    hipLaunchKernelGGL(k_running_average, dim3((unsigned)blocks), dim3(kT), 0, s, g_prev, x, n, (float)(t - 1), (float)t, g,
                       partial, clear, nclear, partial_x);
  return check_hip(hipGetLastError());
}

int launch_concat2(const float* a, size_t da, const float* b, size_t db, size_t M, float* out, hipStream_t s,
                   float* partial) {
  hipLaunchKernelGGL(k_concat2, dim3((unsigned)M), dim3(kT), 0, s, a, (unsigned)da, b, (unsigned)db, out, partial);
  return check_hip(hipGetLastError());
}

// the wave-per-row kernel where the row fits it; false = not launched
template <bool GATED>
static bool launch_layer_norm_wave(const float* a, const float* f, const float* z, const float* r, const float* gamma,
                                   const float* beta, size_t M, size_t d, float eps, float* y, hipStream_t s, float* partial) {
  if (d % 256 != 0 || d > 1024) return false;
  if (!aligned16(a) || !aligned16(r) || !aligned16(gamma) || !aligned16(beta) || !aligned16(y)) return false;
  if (GATED && (!aligned16(f) || !aligned16(z))) return false;
  auto go = [&](auto kern) { hipLaunchKernelGGL(kern, dim3((unsigned)M), dim3(kWave), 0, s, a, f, z, r, gamma, beta, eps, y, partial); };
  switch (d / 256) {
    case 1: go(k_layer_norm_wave<GATED, 1>); break;
    case 2: go(k_layer_norm_wave<GATED, 2>); break;
    case 3: go(k_layer_norm_wave<GATED, 3>); break;
    default: go(k_layer_norm_wave<GATED, 4>); break;
  }
  return true;
}

int launch_add_layer_norm(const float* a, const float* r, const float* gamma, const float* beta, size_t M, size_t d,
                          float eps, float* y, hipStream_t s, float* partial) {
  if (d > (size_t)kMaxRow) return MQ_ERR_UNSUPPORTED;
  if (!launch_layer_norm_wave<false>(a, nullptr, nullptr, r, gamma, beta, M, d, eps, y, s, partial))
    hipLaunchKernelGGL((k_layer_norm<false>), dim3((unsigned)M), dim3(kT), 0, s, a, (const float*)nullptr,
                       (const float*)nullptr, r, gamma, beta, (unsigned)d, eps, y, partial);
  return check_hip(hipGetLastError());
}

int launch_gate_mix_layer_norm(const float* x, const float* f, const float* z, const float* gamma, const float* beta,
                               size_t M, size_t d, float eps, float* y, hipStream_t s, float* partial) {
  if (d > (size_t)kMaxRow) return MQ_ERR_UNSUPPORTED;
  if (!launch_layer_norm_wave<true>(x, f, z, x, gamma, beta, M, d, eps, y, s, partial))
    hipLaunchKernelGGL((k_layer_norm<true>), dim3((unsigned)M), dim3(kT), 0, s, x, f, z, x, gamma, beta, (unsigned)d, eps, y,
                       partial);
  return check_hip(hipGetLastError());
}

int launch_cross_attention(const float* q, const float* K, const float* V, size_t M, size_t S, size_t d, int heads,
                           float* ctx, hipStream_t s, float* partial) {
  if ((size_t)heads * S > (size_t)kMaxScores) return MQ_ERR_UNSUPPORTED;
  const size_t dh = d / (size_t)heads;
  const bool pow2 = (dh & (dh - 1)) == 0;
  const bool vec_ok = (reinterpret_cast<uintptr_t>(q) | reinterpret_cast<uintptr_t>(K) | reinterpret_cast<uintptr_t>(V) |
                       reinterpret_cast<uintptr_t>(ctx)) % 16 == 0;
  if (vec_ok && pow2 && dh >= 4 && dh <= 256 && (d == 256 || d == 512 || d == 1024)) {
    auto go = [&](auto kern) {
      hipLaunchKernelGGL(kern, dim3((unsigned)M), dim3(kTA), 0, s, q, K, V, (unsigned)S, (unsigned)heads, ctx, partial);
    };
    // up to 8 words asking ahead reads rows again for nothing (d = 512: 0.87 - 0.98 of the time without), from 14 on it wins
    // while every sentence has a compute unit to itself (1.02 - 1.14)
    const bool ahead = M <= 256 && S > 12;
    if (d == 256) ahead ? go(k_cross_attention_fast<1, true>) : go(k_cross_attention_fast<1, false>);
    else if (d == 512) ahead ? go(k_cross_attention_fast<2, true>) : go(k_cross_attention_fast<2, false>);
    else ahead ? go(k_cross_attention_fast<4, true>) : go(k_cross_attention_fast<4, false>);
    return check_hip(hipGetLastError());
  }
  hipLaunchKernelGGL(k_cross_attention, dim3((unsigned)M), dim3(kTA), 0, s, q, K, V, (unsigned)S, (unsigned)d,
                     (unsigned)heads, ctx, partial);
  return check_hip(hipGetLastError());
}

}  // namespace mq
