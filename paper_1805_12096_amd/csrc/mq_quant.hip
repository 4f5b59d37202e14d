// quant_int on gfx950: per-tensor abs-max, multiplier, and the float -> int8 /
// int16 conversion (arxiv 1805.12096, Section 4.2).  All three are bound by HBM
// traffic: wide coalesced loads, one pass each.
#include <type_traits>

#include "mq_grid_max.h"
#include "mq_internal.h"
#include "mq_tiles.h"

namespace mq {

namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, kWave));
  return v;
}

__device__ __forceinline__ int wave_sum(int v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

__global__ void k_fill_u32(uint32_t* p, uint32_t v) { *p = v; }
// Pseudo-random bytes (a hash of the word index): operand contents for timing runs.  The matrix units draw more
// power on varied operands than on constant ones and clock lower, so constant fill ranks tile variants wrongly.
__global__ void k_fill_pattern(uint32_t* p, size_t nwords, uint32_t seed) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < nwords; i += stride) {
    uint32_t x = (uint32_t)i * 2654435761u + seed;
    x ^= x >> 15; x *= 2246822519u; x ^= x >> 13; x *= 3266489917u; x ^= x >> 16;
    p[i] = x;
  }
}

__global__ void k_clear_words(uint32_t* p, unsigned n) {
  const unsigned i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}

// |x| of a non-NaN float orders like its bit pattern, so the grid-wide maximum
// is an integer atomicMax.  fmaxf drops NaN operands.
// Workgroups of 1024 threads, at most 512 of them: every workgroup may end in one atomic on the same word,
// and those are served one after the other (2048 small workgroups ending together took 25 us for that alone).
constexpr int kAbsmaxThreads = 1024;
__global__ __launch_bounds__(kAbsmaxThreads) void k_absmax(const float* __restrict__ x, size_t n,
                                                           uint32_t* __restrict__ amax_bits) {
  constexpr int kThreads = kAbsmaxThreads;
  const size_t tid = (size_t)blockIdx.x * kThreads + threadIdx.x;
  const size_t nthreads = (size_t)gridDim.x * kThreads;
  const size_t nvec = n / 4;
  const float4* xv = reinterpret_cast<const float4*>(x);
  float m0 = 0.f, m1 = 0.f, m2 = 0.f, m3 = 0.f;
  size_t i = tid;
  for (; i + 3 * nthreads < nvec; i += 4 * nthreads) {
    float4 a = xv[i], b = xv[i + nthreads], c = xv[i + 2 * nthreads], d = xv[i + 3 * nthreads];
    m0 = fmaxf(m0, fmaxf(fmaxf(fabsf(a.x), fabsf(a.y)), fmaxf(fabsf(a.z), fabsf(a.w))));
    m1 = fmaxf(m1, fmaxf(fmaxf(fabsf(b.x), fabsf(b.y)), fmaxf(fabsf(b.z), fabsf(b.w))));
    m2 = fmaxf(m2, fmaxf(fmaxf(fabsf(c.x), fabsf(c.y)), fmaxf(fabsf(c.z), fabsf(c.w))));
    m3 = fmaxf(m3, fmaxf(fmaxf(fabsf(d.x), fabsf(d.y)), fmaxf(fabsf(d.z), fabsf(d.w))));
  }
  for (; i < nvec; i += nthreads) {
    float4 a = xv[i];
    m0 = fmaxf(m0, fmaxf(fmaxf(fabsf(a.x), fabsf(a.y)), fmaxf(fabsf(a.z), fabsf(a.w))));
  }
  for (size_t j = nvec * 4 + tid; j < n; j += nthreads) m1 = fmaxf(m1, fabsf(x[j]));
  float m = wave_max(fmaxf(fmaxf(m0, m1), fmaxf(m2, m3)));
  __shared__ float part[kThreads / kWave];
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
  if (lane == 0) part[w] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    float r = part[0];
#pragma unroll
    for (int k = 1; k < kThreads / kWave; ++k) r = fmaxf(r, part[k]);
    // the running maximum only grows: a block that cannot raise it skips the (serialising) atomic
    const uint32_t bits = __float_as_uint(r);
    if (bits > __hip_atomic_load(amax_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(amax_bits, bits);
  }
}

__global__ void k_scale(const float* __restrict__ amax, float qmax, float* __restrict__ scale) {
  const float a = *amax;
  *scale = (a > 0.0f) ? __fdiv_rn(qmax, a) : 1.0f;
}

// One element of quant_int: binary32 multiply, round half to even, symmetric
// clamp; NaN becomes 0.  Four instructions: the conversion saturates and takes NaN
// to 0 by itself, so the clamp is one on integers.
__device__ __forceinline__ int quant1(float x, float s, int lim) {
  const float r = rintf(__fmul_rn(x, s));
  int i;
  asm("v_cvt_i32_f32 %0, %1" : "=v"(i) : "v"(r));
  return min(max(i, -lim), lim);
}

// Byte BYTE of four words: two byte permutes and an or (0x0c selects zero).
template <unsigned BYTE>
__device__ __forceinline__ uint32_t pack4_bytes(int a, int b, int c, int d) {
  return __builtin_amdgcn_perm((uint32_t)b, (uint32_t)a, 0x0c0c0000u | (4u + BYTE) << 8 | BYTE) |
         __builtin_amdgcn_perm((uint32_t)d, (uint32_t)c, (4u + BYTE) << 24 | BYTE << 16 | 0x0c0cu);
}
__device__ __forceinline__ uint32_t pack4_i8(int a, int b, int c, int d) { return pack4_bytes<0>(a, b, c, d); }
__device__ __forceinline__ uint32_t pack2_i16(int a, int b) {
  return (uint32_t)(a & 0xFFFF) | ((uint32_t)(b & 0xFFFF) << 16);
}

// Flat conversion, 8 elements per thread and step: two 16-byte loads, one 8-byte
// (int8) or 16-byte (int16) store.
template <int BITS>
__global__ __launch_bounds__(kThreads) void k_quantize_flat(const float* __restrict__ x, size_t n,
                                                            const float* __restrict__ scale,
                                                            void* __restrict__ qv) {
  const float s = *scale;
  const int lim = BITS == 8 ? 127 : 32767;
  const size_t tid = (size_t)blockIdx.x * kThreads + threadIdx.x;
  const size_t nthreads = (size_t)gridDim.x * kThreads;
  const size_t nvec = n / 8;
  const float4* xv = reinterpret_cast<const float4*>(x);
  for (size_t i = tid; i < nvec; i += nthreads) {
    const float4 a = xv[2 * i], b = xv[2 * i + 1];
    const int q0 = quant1(a.x, s, lim), q1 = quant1(a.y, s, lim), q2 = quant1(a.z, s, lim),
              q3 = quant1(a.w, s, lim), q4 = quant1(b.x, s, lim), q5 = quant1(b.y, s, lim),
              q6 = quant1(b.z, s, lim), q7 = quant1(b.w, s, lim);
    if (BITS == 8) {
      uint2 o;
      o.x = pack4_i8(q0, q1, q2, q3);
      o.y = pack4_i8(q4, q5, q6, q7);
      reinterpret_cast<uint2*>(qv)[i] = o;
    } else {
      uint4 o;
      o.x = pack2_i16(q0, q1);
      o.y = pack2_i16(q2, q3);
      o.z = pack2_i16(q4, q5);
      o.w = pack2_i16(q6, q7);
      reinterpret_cast<uint4*>(qv)[i] = o;
    }
  }
  for (size_t j = nvec * 8 + tid; j < n; j += nthreads) {
    const int q = quant1(x[j], s, lim);
    if (BITS == 8) reinterpret_cast<int8_t*>(qv)[j] = (int8_t)q;
    else reinterpret_cast<int16_t*>(qv)[j] = (int16_t)q;
  }
}

// Row-wise conversion that also produces sum_c q[r][c]: one wavefront per row.
template <int BITS, bool VEC>
__global__ __launch_bounds__(kThreads) void k_quantize_rows(const float* __restrict__ x, size_t rows,
                                                            size_t cols, const float* __restrict__ scale,
                                                            void* __restrict__ qv,
                                                            int32_t* __restrict__ rowsum) {
  const float s = *scale;
  const int lim = BITS == 8 ? 127 : 32767;
  const int lane = threadIdx.x % kWave;
  const size_t wave = (size_t)blockIdx.x * (kThreads / kWave) + threadIdx.x / kWave;
  const size_t nwaves = (size_t)gridDim.x * (kThreads / kWave);
  for (size_t r = wave; r < rows; r += nwaves) {
    const float* xr = x + r * cols;
    int sum = 0;
    if (VEC) {  // cols % 8 == 0 and 16-byte aligned rows
      const float4* xv = reinterpret_cast<const float4*>(xr);
      for (size_t i = lane; i < cols / 8; i += kWave) {
        const float4 a = xv[2 * i], b = xv[2 * i + 1];
        const int q0 = quant1(a.x, s, lim), q1 = quant1(a.y, s, lim), q2 = quant1(a.z, s, lim),
                  q3 = quant1(a.w, s, lim), q4 = quant1(b.x, s, lim), q5 = quant1(b.y, s, lim),
                  q6 = quant1(b.z, s, lim), q7 = quant1(b.w, s, lim);
        sum += q0 + q1 + q2 + q3 + q4 + q5 + q6 + q7;
        if (BITS == 8) {
          uint2 o;
          o.x = pack4_i8(q0, q1, q2, q3);
          o.y = pack4_i8(q4, q5, q6, q7);
          reinterpret_cast<uint2*>(reinterpret_cast<int8_t*>(qv) + r * cols)[i] = o;
        } else {
          uint4 o;
          o.x = pack2_i16(q0, q1);
          o.y = pack2_i16(q2, q3);
          o.z = pack2_i16(q4, q5);
          o.w = pack2_i16(q6, q7);
          reinterpret_cast<uint4*>(reinterpret_cast<int16_t*>(qv) + r * cols)[i] = o;
        }
      }
    } else {
      for (size_t c = lane; c < cols; c += kWave) {
        const int q = quant1(xr[c], s, lim);
        sum += q;
        if (BITS == 8) reinterpret_cast<int8_t*>(qv)[r * cols + c] = (int8_t)q;
        else reinterpret_cast<int16_t*>(qv)[r * cols + c] = (int16_t)q;
      }
    }
    sum = wave_sum(sum);
    if (lane == 0) rowsum[r] = sum;
  }
}

unsigned grid_for(size_t work_items, size_t per_block, unsigned cap) {
  size_t g = (work_items + per_block - 1) / per_block;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (unsigned)g;
}

}  // namespace

int launch_absmax(const float* x, size_t n, float* amax, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(1), 0, s, reinterpret_cast<uint32_t*>(amax), 0u);
  // 16 floats per thread and pass; at most two workgroups per compute unit
  const unsigned grid = grid_for(n, (size_t)kAbsmaxThreads * 16, 512);
  hipLaunchKernelGGL(k_absmax, dim3(grid), dim3(kAbsmaxThreads), 0, s, x, n, reinterpret_cast<uint32_t*>(amax));
  return check_hip(hipGetLastError());
}

int launch_scale(const float* amax, int bits, float* scale, hipStream_t s) {
  hipLaunchKernelGGL(k_scale, dim3(1), dim3(1), 0, s, amax, (float)qmax_of(bits), scale);
  return check_hip(hipGetLastError());
}

int launch_quantize(const float* x, size_t rows, size_t cols, int bits, const float* scale,
                    void* q, int32_t* rowsum, hipStream_t s) {
  if (rowsum == nullptr) {
    const size_t n = rows * cols;
    const unsigned grid = grid_for(n, (size_t)kThreads * 8, 4096);
    if (bits == 8)
      hipLaunchKernelGGL(k_quantize_flat<8>, dim3(grid), dim3(kThreads), 0, s, x, n, scale, q);
    else
      hipLaunchKernelGGL(k_quantize_flat<16>, dim3(grid), dim3(kThreads), 0, s, x, n, scale, q);
  } else {
    const bool vec = (cols % 8 == 0);
    const unsigned grid = grid_for(rows, kThreads / kWave, 4096);
    if (bits == 8) {
      if (vec) hipLaunchKernelGGL((k_quantize_rows<8, true>), dim3(grid), dim3(kThreads), 0, s, x, rows, cols, scale, q, rowsum);
      else hipLaunchKernelGGL((k_quantize_rows<8, false>), dim3(grid), dim3(kThreads), 0, s, x, rows, cols, scale, q, rowsum);
    } else {
      if (vec) hipLaunchKernelGGL((k_quantize_rows<16, true>), dim3(grid), dim3(kThreads), 0, s, x, rows, cols, scale, q, rowsum);
      else hipLaunchKernelGGL((k_quantize_rows<16, false>), dim3(grid), dim3(kThreads), 0, s, x, rows, cols, scale, q, rowsum);
    }
  }
  return check_hip(hipGetLastError());
}

}  // namespace mq

// ---------------------------------------------------------------------------
// quant_int straight into the fragment order the product kernels read (the
// same layout as a prepared parameter, see PackedDims): the activations then
// reach LDS by plain linear copies.  Eight lanes share a row and walk along K
// four floats at a time, so reads are whole 128-byte lines and each store
// instruction writes two 128-byte runs.
namespace mq {
namespace {

// Abs-max without atomics or initialisation: block b writes its maximum to partial[b];
// the consumer reduces the few hundred values itself (block_max_of_partials).  The blocks walk through the tensor together, one
// piece of 256 vectors after the other; BY_XCD (see by_eighths) every block takes one run of `share` vectors and every XCD an
// eighth of the tensor.  Instances of their own, here and in the quantizer: with the order as an argument and the runs' ends
// formed by 64-bit products in front of the first load, calls that deal nothing were 0.4 - 1 % slower (captured, 1001 x 1536 x 512
// in 16 bit 14.96 us, now 14.83; 700 x 1024 x 1024 in 8 bit 10.81, now 10.76; 300 x 512 x 512 6.01, now 5.97).
constexpr int kAbsmaxFlight = 4;
template <bool BY_XCD>
__global__ __launch_bounds__(kThreads) void k_absmax_partial(const float* __restrict__ x, size_t n,
                                                             float* __restrict__ partial, unsigned* clear, unsigned nclear,
                                                             size_t share) {
  // (all arguments at once: the condition below would split their loads, a trip to memory each)
  if constexpr (BY_XCD) asm volatile("" ::"s"(x), "s"(n), "s"(share), "s"(gridDim.x));
  if (clear != nullptr && blockIdx.x == 0)                 // a later kernel's counters
    for (unsigned i = threadIdx.x; i < nclear; i += kThreads) clear[i] = 0u;
  const size_t nvec = n / 4;
  const unsigned block = BY_XCD ? xcd_remap(blockIdx.x, gridDim.x) : blockIdx.x;
  const size_t first = block * (BY_XCD ? share : (size_t)kThreads), step = BY_XCD ? (size_t)kThreads : (size_t)gridDim.x * kThreads;
  const size_t end = BY_XCD && first + share < nvec ? first + share : nvec;
  const float4* xv = reinterpret_cast<const float4*>(x);
  float m0 = 0.f;
  // kAbsmaxFlight loads in flight per thread (past the end: the last vector again, which changes nothing)
  for (size_t i = first + threadIdx.x; i < end; i += kAbsmaxFlight * step) {
    float4 a[kAbsmaxFlight];
#pragma unroll
    for (int t = 0; t < kAbsmaxFlight; ++t) a[t] = xv[i + t * step < end ? i + t * step : end - 1];
#pragma unroll
    for (int t = 0; t < kAbsmaxFlight; ++t)
      m0 = fmaxf(m0, fmaxf(fmaxf(fabsf(a[t].x), fabsf(a[t].y)), fmaxf(fabsf(a[t].z), fabsf(a[t].w))));
  }
  if (blockIdx.x == 0 && nvec * 4 + threadIdx.x < n) m0 = fmaxf(m0, fabsf(x[nvec * 4 + threadIdx.x]));      // n % 4 elements
  const float m = __uint_as_float(wave_max_u32(__float_as_uint(m0)));
  __shared__ float part[kThreads / kWave];
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
  if (lane == 0) part[w] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    float r = part[0];
#pragma unroll
    for (int k = 1; k < kThreads / kWave; ++k) r = fmaxf(r, part[k]);
    partial[blockIdx.x] = r;
  }
}

// Maximum of `count` partial maxima, computed redundantly by every block of W waves that needs it.
template <int W>
__device__ __forceinline__ float block_max_of_partials(const float* __restrict__ partial, unsigned count) {
  constexpr unsigned kT = W * kWave, kFlight = kAbsmaxPartials / kT;      // kAbsmaxPartials of them: one trip
  float m = 0.f;
  for (unsigned i0 = 0; i0 < count; i0 += kFlight * kT) {
    float v[kFlight];
#pragma unroll
    for (unsigned t = 0; t < kFlight; ++t) v[t] = partial[min(i0 + t * kT + threadIdx.x, count - 1)];
#pragma unroll
    for (unsigned t = 0; t < kFlight; ++t) m = fmaxf(m, v[t]);
  }
  m = __uint_as_float(wave_max_u32(__float_as_uint(m)));      // non-negative: ordered like its bits
  __shared__ float red[W];
  if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = m;
  __syncthreads();
  float r = red[0];
#pragma unroll
  for (int k = 1; k < W; ++k) r = fmaxf(r, red[k]);
  return r;
}

// Four consecutive elements of a row from column k on, always from addresses inside the tensor: a load under a condition of
// its own is a branch with a wait of its own behind it, which makes the loads of a trip follow one another instead of being
// in flight together (quantizing kernel of a 5003 x 1024 product 7.4 -> 6.4 us = 4.0 TB/s, of 8192 x 4096 to 16 bit 35.7 ->
// 34.3 us = 5.9 TB/s; one-kernel form, 300 x 512, 4.8 -> 4.6 us).  What lies past the row's end is taken out of the
// converted bytes by place4.  Rows of any length are read in vectors, too: one element at a time, each with its own clamp,
// 1001 x 2050 took 5.4 us where it now takes 4.0 (16 bit 8.0, now 6.3; with abs-max in one kernel 12.1, now 8.9).
enum Cols {
  kColsVec,       // a multiple of 4: rows are 16-byte aligned
  kColsAny,       // at least 4: rows are 4-byte aligned; the last vector of a row ends at its end
  kColsFew,       // 1 .. 3
};
inline Cols cols_kind(size_t cols) { return cols % 4 == 0 ? kColsVec : cols > 4 ? kColsAny : kColsFew; }

template <Cols COLS>
__device__ __forceinline__ float4 load4_clamped(const float* __restrict__ row, unsigned k, unsigned cols) {
  if constexpr (COLS == kColsFew) {
    const unsigned last = cols - 1;
    return make_float4(row[min(k, last)], row[min(k + 1, last)], row[min(k + 2, last)], row[min(k + 3, last)]);
  } else {
    float4 v;
    const float* src = row + min(k, cols - 4);
    if constexpr (COLS == kColsVec) v = *reinterpret_cast<const float4*>(src);
    else __builtin_memcpy(&v, src, sizeof(v));
    return v;
  }
}
// The bytes of what load4_clamped read, as elements k .. k + 3 of the row: zero past the row's end, and past the last row.
template <Cols COLS>
__device__ __forceinline__ uint32_t place4(uint32_t bytes, bool row_ok, unsigned k, unsigned cols) {
  if (!row_ok || k >= cols) return 0u;
  if constexpr (COLS == kColsVec) return bytes;
  if constexpr (COLS == kColsAny) return bytes >> (8 * (k - min(k, cols - 4)));      // read up to three elements early
  return bytes & (0xFFFFFFFFu >> (8 * (4 - min(cols - k, 4u))));
}

// Converts four elements and stores their bytes at dst (16 bit: two planes; q = 256 h + l + 128, high bytes and low
// bytes with the top bit flipped).  Returns the sum of the four quantized values (16 bit).
template <int BITS, Cols COLS>
__device__ __forceinline__ int store4(uint8_t* dst, float4 v, float s, int lim, bool row_ok, unsigned k, unsigned cols) {
  const int q0 = quant1(v.x, s, lim), q1 = quant1(v.y, s, lim), q2 = quant1(v.z, s, lim), q3 = quant1(v.w, s, lim);
  const uint32_t lo = place4<COLS>(pack4_i8(q0, q1, q2, q3), row_ok, k, cols);
  if constexpr (BITS == 8) {
    *reinterpret_cast<uint32_t*>(dst) = lo;
    return 0;
  } else {
    const uint32_t hi = place4<COLS>(pack4_bytes<1>(q0, q1, q2, q3), row_ok, k, cols);
    *reinterpret_cast<uint32_t*>(dst) = hi;
    *reinterpret_cast<uint32_t*>(dst + kFragBytes) = lo ^ 0x80808080u;
    // sum of the values = sum of the low bytes (unsigned) + 256 x sum of the high bytes (signed)
    return (int)__builtin_amdgcn_udot4(lo, 0x01010101u, 0u, false) + 256 * __builtin_amdgcn_sdot4((int)hi, 0x01010101, 0, false);
  }
}

// FROM_PARTIALS: `scale` holds `npartial` partial abs-maxima instead of the multiplier; the
// multiplier Qmax / max is formed here (one correctly rounded division) and block 0 also
// publishes it in scale_out[0] for the product kernels that follow.
// A work item is `per` fragments along K of a group of eight rows, kQuantFlight of them loaded at a time; the first item's
// first loads go out before the partial maxima are asked for, so that the two round trips to memory are one.
constexpr int kQuantFlight = 4;
template <int BITS, Cols COLS, bool FROM_PARTIALS, int W, bool BY_XCD>
__global__ __launch_bounds__(W * kWave) void k_quantize_pack(const float* __restrict__ x, size_t rows,
                                                            size_t cols, const float* __restrict__ scale,
                                                            uint8_t* __restrict__ packed, unsigned ksplit,
                                                            unsigned npartial, float* __restrict__ scale_out,
                                                            unsigned* __restrict__ clear, unsigned nclear) {
  constexpr unsigned kT = W * kWave;
  // (all arguments at once: the loop's condition would split their loads, a trip to memory each)
  if constexpr (BY_XCD) asm volatile("" ::"s"(x), "s"(rows), "s"(cols), "s"(ksplit), "s"(gridDim.x));
  // words a later kernel wants zero (spread over the grid: one workgroup walking through them is a serial tail)
  for (unsigned i = blockIdx.x * kT + threadIdx.x; i < nclear; i += gridDim.x * kT) clear[i] = 0u;
  const PackedDims d(BITS, rows, cols);
  const int lim = BITS == 8 ? 127 : 32767;
  const int lane = threadIdx.x % kWave;
  const int sub = lane % 8;                       // which 4 floats of a 32-element fragment row
  // (indexes of fragments, row groups and items fit 32 bits: rows and columns are below 2^31, items below 2^29 x 16)
  const unsigned kfrags = (unsigned)d.kfrags, row_groups = (unsigned)(d.Np / 8);
  const unsigned wave_in = threadIdx.x / kWave;
  const unsigned block = BY_XCD ? xcd_remap(blockIdx.x, gridDim.x) : blockIdx.x, wave = block * W + wave_in;
  const unsigned nwaves = gridDim.x * W;
  const unsigned shift = 31 - __builtin_clz(ksplit);     // (a power of two)
  const unsigned per = (kfrags + ksplit - 1) >> shift;   // fragments along K per work item
  // 16 bit, long rows: the workgroup's waves share a row group, each takes its part of K (W times the loads in
  // flight of one wave per row group, which leaves a chip with a thousand row groups at four waves per compute
  // unit), and the rows' sums meet in LDS.  ksplit is the number of waves of the workgroup then (see pack_split).
  const bool shared_rows = BITS == 16 && ksplit > 1;
  unsigned rg = shared_rows ? block : wave >> shift, part = shared_rows ? wave_in : wave & (ksplit - 1);
  const unsigned ncols = (unsigned)cols, nrows = (unsigned)rows;
  float4 v[kQuantFlight];
  auto load = [&](unsigned kb0) {
    const float* xr = x + (size_t)min(rg * 8 + lane / 8, nrows - 1) * cols;
#pragma unroll
    for (int j = 0; j < kQuantFlight; ++j) v[j] = load4_clamped<COLS>(xr, (kb0 + j) * kFragK + 4 * sub, ncols);
  };
  if (rg < row_groups) load(part * per);
  float s;
  if (FROM_PARTIALS) {
    const float amax = block_max_of_partials<W>(scale, npartial);
    s = (amax > 0.0f) ? __fdiv_rn(BITS == 8 ? 127.0f : 32767.0f, amax) : 1.0f;
    if (blockIdx.x == 0 && threadIdx.x == 0) *scale_out = s;
  } else {
    s = *scale;
  }
  // the item (rg, part), whose first loads are in v; returns the lane's share of the rows' sums (16 bit)
  auto convert = [&]() -> int {
    const unsigned row = rg * 8 + lane / 8;
    const unsigned kb_end = (part + 1) * per < kfrags ? (part + 1) * per : kfrags;
    uint8_t* out = packed + d.frag_offset(row / kFragRows, 0) + (row % kFragRows + 32 * (sub / 4)) * 16 + 4 * (sub % 4);
    int sum = 0;
    for (unsigned kb0 = part * per; kb0 < kb_end; kb0 += kQuantFlight) {
      if (kb0 != part * per) load(kb0);
#pragma unroll
      for (int j = 0; j < kQuantFlight; ++j) {
        if (kb0 + j >= kb_end) break;
        sum += store4<BITS, COLS>(out + (size_t)(kb0 + j) * (kFragBytes * (BITS == 16 ? 2 : 1)), v[j], s, lim, row < nrows,
                                  (kb0 + j) * kFragK + 4 * sub, ncols);
      }
    }
    if (BITS == 16) {
      sum += __shfl_xor(sum, 1, kWave);
      sum += __shfl_xor(sum, 2, kWave);
      sum += __shfl_xor(sum, 4, kWave);
    }
    return sum;
  };
  if (shared_rows) {
    __shared__ int s_part[W][8];
    for (; rg < row_groups; rg += gridDim.x) {
      if (rg != block) load(part * per);
      const int sum = convert();
      if (sub == 0) s_part[part][lane / 8] = sum;
      __syncthreads();
      if (part == 0 && sub == 0) {
        int total = 0;
#pragma unroll
        for (int k = 0; k < W; ++k) total += s_part[k][lane / 8];
        reinterpret_cast<int32_t*>(packed + d.plane_bytes())[(size_t)rg * 8 + lane / 8] = total;
      }
      __syncthreads();
    }
    return;
  }
  for (unsigned item = wave; item < row_groups * ksplit; item += nwaves) {
    if (item != wave) {
      rg = item >> shift;
      part = item & (ksplit - 1);
      load(part * per);
    }
    const int sum = convert();
    // 16 bit here: one wave owns whole rows
    if (BITS == 16 && sub == 0) reinterpret_cast<int32_t*>(packed + d.plane_bytes())[rg * 8 + lane / 8] = sum;
  }
}


// abs-max + quant_int in ONE launch for tensors whose elements all fit the registers of one resident
// grid: every wave loads its share (8 rows x 4 NI fragments), the workgroups agree on max|x| (see
// mq_grid_max.h), and the share is converted from registers.  Same work split, rounding and layout as
// k_quantize_pack; x is read once instead of twice and one kernel boundary disappears.
template <int BITS, Cols COLS, int NI>
__global__ __launch_bounds__(512) void k_absmax_quantize_pack(const float* __restrict__ x, size_t rows, size_t cols,
                                                              uint8_t* __restrict__ packed, unsigned ksplit,
                                                              unsigned* barrier, unsigned long long ticks,
                                                              float* __restrict__ scale_out, unsigned* clear_words,
                                                              unsigned nclear, int self_clean) {
  constexpr int kW = 512 / kWave;
  // words a LATER kernel's agreement wants zero (not the ones used below): a caller that keeps its agreement
  // areas clean from call to call has this kernel and the next one clear each other's
  if (clear_words != nullptr && blockIdx.x == 0)
    for (unsigned i = threadIdx.x; i < nclear; i += 512) clear_words[i] = 0u;
  const PackedDims d(BITS, rows, cols);
  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);      // scalar, as the item
  const int sub = lane % 8;                       // which 4 floats of a 32-element fragment row
  // (a resident grid's items and the tensor's rows, columns and fragments all fit 32 bits)
  const unsigned kfrags = (unsigned)d.kfrags, row_groups = (unsigned)(d.Np / 8), ncols = (unsigned)cols, nrows = (unsigned)rows;
  const unsigned shift = 31 - __builtin_clz(ksplit);     // (a power of two)
  const unsigned per = (kfrags + ksplit - 1) >> shift;   // fragments along K per wave, at most 4 NI
  const unsigned item = blockIdx.x * kW + wave;
  const bool active = item < row_groups * ksplit;
  const unsigned rg = item >> shift, part = item & (ksplit - 1);
  const unsigned row = rg * 8 + lane / 8;
  const unsigned kb_begin = part * per, kb_end = min(kb_begin + per, kfrags);
  // every load from inside the tensor and without a condition of its own (see load4_clamped); fragments past this wave's
  // part, rows past the end and inactive waves read elements that other lanes hold as well, so the maximum needs no mask
  const float* xr = x + (size_t)min(row, nrows - 1) * cols;
  float4 v[NI][4];
  float m = 0.f;
#pragma unroll
  for (int t = 0; t < NI; ++t) {
    if (t == 0 || kb_begin + 4 * t < kb_end) {      // scalar: trips past this wave's part are left out
#pragma unroll
      for (int j = 0; j < 4; ++j) v[t][j] = load4_clamped<COLS>(xr, (kb_begin + 4 * t + j) * kFragK + 4 * sub, ncols);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) v[t][j] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
#pragma unroll
  for (int t = 0; t < NI; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      m = fmaxf(m, fmaxf(fmaxf(fabsf(v[t][j].x), fabsf(v[t][j].y)), fmaxf(fabsf(v[t][j].z), fabsf(v[t][j].w))));
  m = __uint_as_float(wave_max_u32(__float_as_uint(m)));      // m >= 0 and never NaN (fmaxf drops NaN operands)
  __shared__ float red[kW];
  if (lane == 0) red[wave] = m;
  __syncthreads();
  if (wave == 0) {
    float b = red[0];
#pragma unroll
    for (int w = 1; w < kW; ++w) b = fmaxf(b, red[w]);
    if (lane == 0) grid_max_publish(barrier, b);
    const float amax = grid_max_collect(barrier, ticks);
    if (lane == 0) red[0] = amax;
  }
  __syncthreads();
  const float amax = red[0];
  // self_clean: the agreement area is left all zero.  Every workgroup but the first is done with it here (its
  // count goes out now and is looked at after the stores); the first still has to look at the sticky word.
  unsigned retired_before = 0u;
  if (self_clean && blockIdx.x != 0 && threadIdx.x == 0) retired_before = grid_max_retire(barrier);
  const int lim = BITS == 8 ? 127 : 32767;
  const float s = (amax > 0.0f) ? __fdiv_rn((float)lim, amax) : 1.0f;
  int sum = 0;
  if (active) {
    uint8_t* out = packed + d.frag_offset(row / kFragRows, 0) + (row % kFragRows + 32 * (sub / 4)) * 16 + 4 * (sub % 4);
#pragma unroll
    for (int t = 0; t < NI; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const unsigned kb = kb_begin + 4 * t + j;
        if (kb < kb_end)
          sum += store4<BITS, COLS>(out + (size_t)kb * (kFragBytes * (BITS == 16 ? 2 : 1)), v[t][j], s, lim, row < nrows,
                                    kb * kFragK + 4 * sub, ncols);
      }
  }
  if (BITS == 16) {
    sum += __shfl_xor(sum, 1, kWave);
    sum += __shfl_xor(sum, 2, kWave);
    sum += __shfl_xor(sum, 4, kWave);
    if (ksplit > 1) {
      // the ksplit waves that share a row group sit side by side in the workgroup (ksplit divides its eight waves):
      // their parts of the rows' sums meet in LDS
      __shared__ int s_rowpart[kW][8];
      if (sub == 0) s_rowpart[wave][lane / 8] = sum;
      __syncthreads();
      if (active && part == 0 && sub == 0) {
        int total = 0;
        for (unsigned j = 0; j < ksplit; ++j) total += s_rowpart[wave + j][lane / 8];
        reinterpret_cast<int32_t*>(packed + d.plane_bytes())[row] = total;
      }
    } else if (active && sub == 0) {
      reinterpret_cast<int32_t*>(packed + d.plane_bytes())[row] = sum;
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    *scale_out = grid_max_failed(barrier) ? __builtin_nanf("") : s;
    if (self_clean) retired_before = grid_max_retire(barrier);
  }
  if (self_clean) {
    __shared__ unsigned last;
    if (threadIdx.x == 0) last = retired_before == gridDim.x - 1 ? 1u : 0u;
    __syncthreads();
    if (last != 0u)
      for (unsigned i = threadIdx.x; i < kBarrierWords; i += 512) barrier[i] = 0u;
  }
}

}  // namespace

namespace {
// Whether abs-max and the quantizer behind it take a tensor in eighths, one to an XCD: what the abs-max launch has read on the
// same XCD then comes from its L2 (20 MB in 2.2 us instead of 4.4).  Captured calls of mq_linear_f32 with abs-max, 300 to 4096
// columns in and out, 600 to 8192 rows, eighths against row groups that go round the XCDs (mean, least and largest ratio by
// millions of 2^20 elements):
//   8 bit   below 1  0.986 (0.956 - 1.015)   1 - 2  0.974 (0.942 - 1.008)   2 - 4  0.961 (0.934 - 0.994)   4 - 12  0.947 (0.912 -
//           0.987)   12 - 16  0.985 (0.950 - 1.045)   above  0.994 (0.952 - 1.013)
//   16 bit  below 1  0.994 (0.982 - 1.012)   1 - 2  0.982 (0.951 - 0.995)   2 - 4  0.971 (0.938 - 0.993)   4 - 12  0.970 (0.945 -
//           0.994)   12 - 16  0.993 (0.969 - 1.023)   above  1.003 (0.995 - 1.013)
// (8192 x 1024 x 1024 in 8 bit 30.5 -> 28.5 us, 8192 x 512 x 512 in 16 bit 23.0 -> 22.0).  Below a million the gain is small and the
// first products of the blocks lose (8-bit block of 1001 rows, 512 / 2048, 17.7 and 17.9; first product of the 16-bit block of 300
// rows 6.6 and 7.4).  The products behind it matter less: those that split K and share rows between XCDs gain as well.
// Only behind an abs-max launch: with the multiplier given nobody has read the tensor before (106 calls a width of 1 to 14
// million elements: 8 bit 0.998, 0.940 - 1.029, 16 bit 1.002, 0.981 - 1.014), and an input that some product has written lies on
// the XCDs that held its columns (the 16-bit block of 3000 rows, 512 / 2048, 54.8 and 55.7).
bool by_eighths(int bits, size_t n) { return n >= ((size_t)1 << 20) && (bits == 8 || n <= ((size_t)12 << 20)); }
}  // namespace

namespace {
// How many waves share a row group along K and, for 16 bit, how many a workgroup has.  8 bit: split K so that even a 300-row
// batch fills the chip.  16 bit: the rows' sums have to meet in one workgroup, rows of 512 elements or more are shared by its
// waves, shorter ones stay whole.  Four waves leave a batch of a few hundred rows with one wave per SIMD on a part of the
// compute units, each with a long chain of trips along K, so up to 128 row groups take 16 waves and up to 256 eight, as long
// as a wave keeps eight fragments (quantizer and product of 300 x 4096, given multiplier, 25.4 -> 22.7 us, 1001 x 4096 38.1 ->
// 36.0, 500 x 2048 13.6 -> 12.9; shorter runs than that gain nothing).  Beyond, the chip is full and larger workgroups only
// meet more often: eight waves for 4000 rows of 2050 elements 30.1 -> 31.1 us, sixteen 32.2.
struct PackSplit {
  unsigned ksplit, waves;
};
PackSplit pack_split(int bits, const PackedDims& d) {
  const size_t row_groups = d.Np / 8;
  unsigned ksplit = 1;
  if (bits == 8) {
    while (row_groups * ksplit < 2048 && ksplit * 4 <= d.kfrags) ksplit *= 2;
    return {ksplit, kThreads / kWave};
  }
  if (d.kfrags < 16) return {1, kThreads / kWave};
  unsigned waves = kThreads / kWave;
  while (waves < 16 && row_groups * waves < 1024u && waves * 8 <= d.kfrags) waves *= 2;
  return {waves, waves};
}

// FROM_PARTIALS: `scale` holds `npartial` partial maxima and scale_out receives the multiplier (see the kernel).
// by_xcd: rows go to the XCDs in eighths (by_eighths), as k_absmax_partial has dealt them; otherwise row groups go round the XCDs.
template <bool FROM_PARTIALS>
int launch_pack(const float* x, size_t rows, size_t cols, int bits, const float* scale, unsigned npartial, float* scale_out,
                void* packed, unsigned* clear, unsigned nclear, bool by_xcd, hipStream_t s) {
  const PackedDims d(bits, rows, cols);
  const size_t row_groups = d.Np / 8;
  const PackSplit sp = pack_split(bits, d);
  const unsigned grid = bits == 16 && sp.ksplit > 1 ? grid_for(row_groups, 1, 8192) : grid_for(row_groups * sp.ksplit, sp.waves, 8192);
  const Cols kind = cols_kind(cols);
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(grid), dim3(sp.waves * kWave), 0, s, x, rows, cols, scale, static_cast<uint8_t*>(packed),
                       sp.ksplit, npartial, scale_out, clear, nclear);
  };
  auto by_kind = [&](auto bits_tag, auto waves_tag, auto xcd_tag) {
    constexpr int B = decltype(bits_tag)::value, W = decltype(waves_tag)::value;
    constexpr bool X = decltype(xcd_tag)::value;
    if (kind == kColsVec) go(k_quantize_pack<B, kColsVec, FROM_PARTIALS, W, X>);
    else if (kind == kColsAny) go(k_quantize_pack<B, kColsAny, FROM_PARTIALS, W, X>);
    else if constexpr (W == 4) go(k_quantize_pack<B, kColsFew, FROM_PARTIALS, W, X>);      // (two fragments along K)
  };
  auto by_waves = [&](auto xcd_tag) {
    if (bits == 8) by_kind(std::integral_constant<int, 8>{}, std::integral_constant<int, 4>{}, xcd_tag);
    else if (sp.waves == 4) by_kind(std::integral_constant<int, 16>{}, std::integral_constant<int, 4>{}, xcd_tag);
    else if (sp.waves == 8) by_kind(std::integral_constant<int, 16>{}, std::integral_constant<int, 8>{}, xcd_tag);
    else by_kind(std::integral_constant<int, 16>{}, std::integral_constant<int, 16>{}, xcd_tag);
  };
  if constexpr (FROM_PARTIALS) by_xcd ? by_waves(std::true_type{}) : by_waves(std::false_type{});
  else by_waves(std::false_type{});
  return check_hip(hipGetLastError());
}
}  // namespace

int launch_quantize_pack(const float* x, size_t rows, size_t cols, int bits, const float* scale,
                         void* packed, hipStream_t s, unsigned* clear, unsigned nclear) {
  return launch_pack<false>(x, rows, cols, bits, scale, 0u, nullptr, packed, clear, nclear, false, s);
}

int launch_fill_pattern(void* p, size_t bytes, unsigned seed, hipStream_t s) {
  const size_t nwords = bytes / 4;
  if (nwords == 0) return MQ_OK;
  const unsigned grid = grid_for(nwords, 256 * 8, 2048);
  hipLaunchKernelGGL(k_fill_pattern, dim3(grid), dim3(256), 0, s, static_cast<uint32_t*>(p), nwords, seed);
  return check_hip(hipGetLastError());
}

int launch_clear_words(unsigned* p, unsigned n, hipStream_t s) {
  if (n == 0) return MQ_OK;
  hipLaunchKernelGGL(k_clear_words, dim3((n + 255) / 256), dim3(256), 0, s, reinterpret_cast<uint32_t*>(p), n);
  return check_hip(hipGetLastError());
}

// quant_int into the packed layout with the multiplier formed in the kernel from `npartials` partial
// maxima (one is enough: a single max|x| in device memory); scale_out[0] receives the multiplier.
int launch_quantize_pack_partials(const float* x, size_t rows, size_t cols, int bits, const float* partials,
                                  unsigned npartials, float* scale_out, void* packed, hipStream_t s) {
  return launch_pack<true>(x, rows, cols, bits, partials, npartials, scale_out, packed, nullptr, 0u, false, s);
}

namespace {
template <int BITS, Cols COLS, int NI>
int launch_fused_one(const float* x, size_t rows, size_t cols, uint8_t* packed, unsigned ksplit, unsigned grid,
                     unsigned* barrier, float* scale_out, hipStream_t s, unsigned* clear_words, unsigned nclear,
                     int self_clean) {
  auto kern = k_absmax_quantize_pack<BITS, COLS, NI>;
  static int max_blocks = -1;       // workgroups the device can hold at once, asked once
  if (max_blocks < 0) {
    int per_cu = 0, dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(kern), 512, 0) != hipSuccess)
      return MQ_ERR_HIP;
    max_blocks = per_cu * cus;
  }
  if (grid > (unsigned)max_blocks) return MQ_ERR_UNSUPPORTED;     // the grid-wide wait needs every workgroup resident
  hipLaunchKernelGGL(kern, dim3(grid), dim3(512), 0, s, x, rows, cols, packed, ksplit, barrier, barrier_timeout_ticks(),
                     scale_out, clear_words, nclear, self_clean);
  return check_hip(hipGetLastError());
}

template <int BITS, Cols COLS>
int launch_fused_ni(int ni, const float* x, size_t rows, size_t cols, uint8_t* packed, unsigned ksplit, unsigned grid,
                    unsigned* barrier, float* scale_out, hipStream_t s, unsigned* clear_words, unsigned nclear,
                    int self_clean) {
  switch (ni) {
    case 1: return launch_fused_one<BITS, COLS, 1>(x, rows, cols, packed, ksplit, grid, barrier, scale_out, s, clear_words, nclear, self_clean);
    case 2: return launch_fused_one<BITS, COLS, 2>(x, rows, cols, packed, ksplit, grid, barrier, scale_out, s, clear_words, nclear, self_clean);
    case 4: return launch_fused_one<BITS, COLS, 4>(x, rows, cols, packed, ksplit, grid, barrier, scale_out, s, clear_words, nclear, self_clean);
    default: return launch_fused_one<BITS, COLS, 8>(x, rows, cols, packed, ksplit, grid, barrier, scale_out, s, clear_words, nclear, self_clean);
  }
}
}  // namespace

// abs-max + quant_int into the packed layout in ONE launch, for tensors small enough to sit in the
// registers of one resident grid (at most 256 workgroups of 8 waves, at most 32 fragments along K per
// wave): MQ_ERR_UNSUPPORTED otherwise, nothing launched.  The kBarrierWords words at `barrier` must be
// zero when the kernel starts.  scale_out[0] receives the multiplier (NaN if the grid-wide wait failed).
int launch_absmax_quantize_pack_fused(const float* x, size_t rows, size_t cols, int bits, unsigned* barrier,
                                      float* scale_out, void* packed, hipStream_t s, unsigned* clear_words,
                                      unsigned nclear, int self_clean) {
  const PackedDims d(bits, rows, cols);
  const size_t row_groups = d.Np / 8;
  const size_t max_waves = (size_t)kBarrierSlots * (512 / kWave);
  if (row_groups > max_waves) return MQ_ERR_UNSUPPORTED;
  // split K as far as one trip of four fragments per wave allows while the waves still fit; 16 bit: at most over
  // the eight waves of a workgroup, where the parts of a row's sum meet in LDS
  unsigned ksplit = 1;
  while (row_groups * ksplit * 2 <= max_waves && (d.kfrags + 2 * ksplit - 1) / (2 * ksplit) >= 4 &&
         (bits == 8 || ksplit * 2 <= 512 / kWave))
    ksplit *= 2;
  const size_t per = (d.kfrags + ksplit - 1) / ksplit;
  if (per > 32) return MQ_ERR_UNSUPPORTED;
  const int ni = per <= 4 ? 1 : per <= 8 ? 2 : per <= 16 ? 4 : 8;
  const unsigned grid = (unsigned)((row_groups * ksplit + 512 / kWave - 1) / (512 / kWave));
  uint8_t* p = static_cast<uint8_t*>(packed);
  const Cols kind = cols_kind(cols);
  auto go = [&](auto bits_tag) {
    constexpr int B = decltype(bits_tag)::value;
    // (1 .. 3 columns are two fragments along K)
    if (kind == kColsFew) return launch_fused_one<B, kColsFew, 1>(x, rows, cols, p, ksplit, grid, barrier, scale_out, s, clear_words, nclear, self_clean);
    return kind == kColsVec ? launch_fused_ni<B, kColsVec>(ni, x, rows, cols, p, ksplit, grid, barrier, scale_out, s, clear_words, nclear, self_clean)
                            : launch_fused_ni<B, kColsAny>(ni, x, rows, cols, p, ksplit, grid, barrier, scale_out, s, clear_words, nclear, self_clean);
  };
  return bits == 8 ? go(std::integral_constant<int, 8>{}) : go(std::integral_constant<int, 16>{});
}

namespace {
unsigned launch_absmax_blocks(const float* x, size_t n, float* partials, unsigned* clear, unsigned nclear, bool by_xcd, hipStream_t s) {
  const unsigned g1 = grid_for(n, (size_t)kThreads * 8, kAbsmaxPartials);
  const size_t share = (n / 4 + g1 - 1) / g1;
  auto kern = by_xcd ? k_absmax_partial<true> : k_absmax_partial<false>;
  hipLaunchKernelGGL(kern, dim3(g1), dim3(kThreads), 0, s, x, n, partials, clear, nclear, share);
  return g1;
}
}  // namespace
// Partial maxima of |x| only (at most kAbsmaxPartials of them); *count receives how many were written.
int launch_absmax_partials(const float* x, size_t n, float* partials, unsigned* count, hipStream_t s) {
  *count = launch_absmax_blocks(x, n, partials, nullptr, 0u, false, s);
  return check_hip(hipGetLastError());
}

// abs-max + quant_int into the packed layout in two launches, no atomics, no fill:
// partial maxima to `partials` (kAbsmaxPartials floats), then quantization with the multiplier
// formed from them; scale_out[0] receives the multiplier.
int launch_absmax_quantize_pack(const float* x, size_t rows, size_t cols, int bits, float* partials,
                                float* scale_out, void* packed, hipStream_t s, unsigned* clear, unsigned nclear) {
  const size_t n = rows * cols;
  const bool by_xcd = by_eighths(bits, n);
  const unsigned g1 = launch_absmax_blocks(x, n, partials, clear, nclear, by_xcd, s);
  return launch_pack<true>(x, rows, cols, bits, partials, g1, scale_out, packed, nullptr, 0u, by_xcd, s);
}

}  // namespace mq
