// Products of at most 32 rows with everything in front of them in one launch (arxiv 1805.12096, Section 4.2: every
// activation is quantized on each call; Section 3.2: a decoder step of a few sentences).
//
// With one block of rows every workgroup can afford to look at the WHOLE input: it loads all rows, applies the float
// operation that produces them (running average, residual + layer normalisation, or nothing), takes their abs-max,
// quantizes them into operand fragments in LDS and multiplies them with its own 32 columns.  Nothing has to be agreed
// between workgroups, so the glue kernel, the abs-max pass and the quantizer that stood in front of the product
// disappear: at these sizes each of them is a launch (2.4 us on the host, 2 - 4 us on the device) around a few hundred
// nanoseconds of work.  The price is that the input is read and converted once per 32 columns.
// Measured: decoder layer of one sentence (512 / 2048) 53.3 -> 35.6 us, nine launches for fourteen.  32 rows are what one
// workgroup's matrix instructions take; at 32 rows and K = 2048 it converts 64 K elements for 32 columns and is still ahead
// with abs-max (7.7 against 9.1 us), no longer with a given multiplier: see gemm_rows_ahead_given.
#include "mq_gemm_common.h"
#include "mq_glue.h"
#include "mq_grid_max.h"

namespace mq {

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

enum RowsIn {
  kRowsPlain = 0,      // A = a
  kRowsAverage = 1,    // A = (tm1 a + b) / t, also written to `side`
  kRowsPairGate = 2,   // A = [a | b] (K1 and K - K1 columns); result: sigmoid(y[:K1]) a + sigmoid(y[K1:]) b, N = 2 K1 = K
  kRowsNorm = 3,       // A = LN(a + b) gamma + beta, also written to `side`
};

// Two cache lines: every line of arguments is a miss of its own on each launch.  (RowsFill is a third, which only the form with
// the average reads; the others take the same time with it and without, 0.994 to 0.998 in seven calls.)
struct RowsParams {
  const float* a;
  const float* b;
  const float *gamma, *beta;
  const uint8_t* packedW;
  const float* scale;        // multiplier, or NULL: Qmax / max|A|
  unsigned M, N, K, K1;
  const float* sW;
  const float* bias;
  float* side;               // [M x K]
  float* Y;                  // [M x N]; with the gate [M x K1]
  float* out_amax;
  float* partial_out;        // optional: max|y| of every workgroup
  float tm1, t, eps;
  int relu;
};
static_assert(sizeof(RowsParams) <= 128, "two cache lines");

// Four integers |q| <= 127 as bytes: two byte permutes and an or (0x0c selects zero).
__device__ __forceinline__ uint32_t bytes_of4(const int (&q)[4], unsigned byte) {
  const uint32_t lo = 0x0c0c0000u | (4u + byte) << 8 | byte, hi = (4u + byte) << 24 | byte << 16 | 0x0c0cu;
  return __builtin_amdgcn_perm((uint32_t)q[1], (uint32_t)q[0], lo) | __builtin_amdgcn_perm((uint32_t)q[3], (uint32_t)q[2], hi);
}

// KS: waves; CH: 256-element pieces of a row (K <= 256 CH); NR: rows per wave (M <= KS NR).
// First phase: wave w holds rows w, w + KS, ... whole, lane l the elements 256 c + 4 l + 0 .. 3 of piece c -- the layout of
// k_layer_norm_wave, so that both normalise with the same order of additions.  Second phase: wave w multiplies fragments
// w KW .. of K for all 32 rows, and the partial sums meet in LDS (see k_gemm_small).  Rows past M repeat row M - 1 (their
// results are never stored), K elements past K are zero bytes as in a packed operand.
template <int BITS, int IN, int KS, int CH, int NR>
__global__ __launch_bounds__(KS * 64) void k_gemm_rows(const RowsParams p, const RowsFill fill) {
  constexpr int NPL = BITS == 16 ? 2 : 1, NACC = BITS == 16 ? 3 : 1;
  constexpr int NB = IN == kRowsPairGate ? 2 : 1;           // column blocks per workgroup: z1 and z2 of the same columns
  constexpr int KW = (CH * 8 + KS - 1) / KS;                // fragments of K per wave
  // fragment f of the input: plane 0 (and 1), K half h, row r, 16 bytes; the paddings spread one row's 4-byte writes
  // over all banks
  constexpr int kHalf = 512 + 16, kPitch = 2 * kHalf;
  constexpr int kStage = CH * 8 * NPL * kPitch, kPart = KS * NB * 1024 * (int)sizeof(int);
  constexpr bool kShared = kStage + kPart > 150 * 1024;     // both do not fit: the sums take the fragments' place
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  uint8_t* stage = lds;
  int* part = reinterpret_cast<int*>(kShared ? lds : lds + kStage);
  __shared__ float red[KS];
  __shared__ int rowsum[BITS == 16 ? 32 : 1];
  const int tid = threadIdx.x, lane = tid % 64;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);      // scalar, see k_gemm_small
  const PackedDims dW(BITS, p.N, p.K);
  const unsigned kfrags = (unsigned)dW.kfrags;
  const unsigned M1 = p.M - 1;

  // everything this workgroup reads is asked for before anything is waited for, in the order of its use
  f4 v[NR][CH], w[IN == kRowsAverage || IN == kRowsNorm ? NR : 1][CH];
  f4 gv[IN == kRowsNorm ? CH : 1], bv[IN == kRowsNorm ? CH : 1];
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const size_t row = min((unsigned)(wave + i * KS), M1);
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const unsigned col = min(256u * c + 4u * lane, p.K - 4);
      if constexpr (IN == kRowsPairGate) {
        const bool second = col >= p.K1;                            // (K1 is a multiple of 4)
        v[i][c] = *reinterpret_cast<const f4*>((second ? p.b - p.K1 : p.a) + row * p.K1 + col);
      } else {
        v[i][c] = *reinterpret_cast<const f4*>(p.a + row * p.K + col);
        if constexpr (IN != kRowsPlain) w[i][c] = *reinterpret_cast<const f4*>(p.b + row * p.K + col);
      }
    }
  }
  if constexpr (IN == kRowsNorm) {
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const unsigned col = min(256u * c + 4u * lane, p.K - 4);
      gv[c] = *reinterpret_cast<const f4*>(p.gamma + col);
      bv[c] = *reinterpret_cast<const f4*>(p.beta + col);
    }
  }
  u4 fw[NB][KW][NPL];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int j = 0; j < KW; ++j) {
      const unsigned kb = min((unsigned)(wave * KW + j), kfrags - 1);
      const uint8_t* src = p.packedW + dW.frag_offset(blockIdx.x + (size_t)nb * (p.K1 / 32), kb) + lane * 16;
#pragma unroll
      for (int pl = 0; pl < NPL; ++pl) fw[nb][j][pl] = *reinterpret_cast<const u4*>(src + pl * kFragBytes);
    }
  // The epilogue's constants.  A thread finishes V rows of column n (of both blocks with the gate): vector tid of the
  // 1024 / V in a block.
  constexpr int V = 1024 / (KS * 64);
  static_assert(V >= 1 && V <= 4, "elements must divide over the threads");
  const int lj = lane % 32, lh = lane / 32;
  const unsigned n = blockIdx.x * 32 + lj;
  const int r0 = wave * V;                                          // of 16 accumulator registers
  const unsigned m0 = 8 * (r0 / 4) + 4 * lh + r0 % 4;
  const bool has_bias = p.bias != nullptr;
  const float s_w = *p.sW;
  float bias[NB], gate_in[NB][V];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) bias[nb] = (has_bias ? p.bias : p.sW)[has_bias ? min(n + nb * p.K1, p.N - 1) : 0u];
  if constexpr (IN == kRowsPairGate) {
#pragma unroll
    for (int t = 0; t < V; ++t) {
      gate_in[0][t] = p.a[(size_t)min(m0 + t, M1) * p.K1 + n];
      gate_in[1][t] = p.b[(size_t)min(m0 + t, M1) * p.K1 + n];
    }
  }
  uint32_t cs = 0;
  if constexpr (BITS == 16) cs = reinterpret_cast<const uint32_t*>(p.packedW + dW.plane_bytes())[n];   // (covers padded rows)
  const bool given = p.scale != nullptr;
  const float s_given = *(given ? p.scale : p.sW);
  __builtin_amdgcn_sched_barrier(0);

  if constexpr (IN == kRowsAverage) {
    const unsigned step = (p.N + 31) / 32 * KS * 64;
    const u4 unset = {kUnsetWord, kUnsetWord, kUnsetWord, kUnsetWord};
    for (unsigned i = blockIdx.x * KS * 64 + tid; i < fill.na; i += step) reinterpret_cast<u4*>(fill.a)[i] = unset;
    for (unsigned i = blockIdx.x * KS * 64 + tid; i < fill.nb; i += step) reinterpret_cast<u4*>(fill.b)[i] = unset;
  }

  // ---- the input's rows, their maximum
  float mx = 0.f;
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const unsigned row = wave + i * KS;
    if constexpr (IN == kRowsAverage) {
#pragma unroll
      for (int c = 0; c < CH; ++c)
#pragma unroll
        for (int t = 0; t < 4; ++t) v[i][c][t] = __fdiv_rn(__fmaf_rn(p.tm1, v[i][c][t], w[i][c][t]), p.t);
    }
    if constexpr (IN == kRowsNorm) {
      const float d = (float)p.K;
      float x[CH][4];
#pragma unroll
      for (int c = 0; c < CH; ++c)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const float h = v[i][c][t] + w[i][c][t];
          v[i][c][t] = h;
          x[c][t] = 256u * c < p.K ? h : 0.f;                       // (K is a multiple of 256)
        }
      const float mu = row_sum_f(x) / d;
#pragma unroll
      for (int c = 0; c < CH; ++c)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const float h = v[i][c][t] - mu;
          v[i][c][t] = h;
          x[c][t] = 256u * c < p.K ? h * h : 0.f;
        }
      const float inv = __fdiv_rn(1.0f, sqrtf(row_sum_f(x) / d + p.eps));
#pragma unroll
      for (int c = 0; c < CH; ++c)
#pragma unroll
        for (int t = 0; t < 4; ++t) v[i][c][t] = v[i][c][t] * inv * gv[c][t] + bv[c][t];
    }
    if constexpr (IN == kRowsAverage || IN == kRowsNorm) {
      // one of the workgroups writes the row
      if (row < p.M && row % gridDim.x == blockIdx.x)
#pragma unroll
        for (int c = 0; c < CH; ++c)
          if (256u * c + 4u * lane < p.K) *reinterpret_cast<f4*>(p.side + (size_t)row * p.K + 256u * c + 4u * lane) = v[i][c];
    }
#pragma unroll
    for (int c = 0; c < CH; ++c)                                    // (past K: element K - 4 .. K - 1 again)
#pragma unroll
      for (int t = 0; t < 4; ++t) mx = fmaxf(mx, fabsf(v[i][c][t]));       // drops NaN
  }
  mx = __uint_as_float(wave_max_u32(__float_as_uint(mx)));
  if (lane == 0) red[wave] = mx;
  __syncthreads();
  constexpr float kQmax = BITS == 16 ? 32767.0f : 127.0f;
  float amax = red[0];
#pragma unroll
  for (int k = 1; k < KS; ++k) amax = fmaxf(amax, red[k]);
  const float s = given ? s_given : (amax > 0.0f ? __fdiv_rn(kQmax, amax) : 1.0f);

  // ---- quant_int into fragments
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int row = wave + i * KS;
    int sum = 0;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const bool inside = 256u * c + 4u * lane < p.K;
      int q[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const float r = rintf(__fmul_rn(v[i][c][t], s));
        asm("v_cvt_i32_f32 %0, %1" : "=v"(q[t]) : "v"(r));          // saturates, NaN -> 0
        q[t] = min(max(q[t], -(int)kQmax), (int)kQmax);
      }
      uint8_t* dst = stage + (8 * c + lane / 8) * NPL * kPitch + ((lane / 4) % 2) * kHalf + row * 16 + 4 * (lane % 4);
      if constexpr (BITS == 8) {
        *reinterpret_cast<uint32_t*>(dst) = inside ? bytes_of4(q, 0) : 0u;
      } else {
        *reinterpret_cast<uint32_t*>(dst) = inside ? bytes_of4(q, 1) : 0u;
        *reinterpret_cast<uint32_t*>(dst + kPitch) = inside ? bytes_of4(q, 0) ^ 0x80808080u : 0u;
        sum += inside ? q[0] + q[1] + q[2] + q[3] : 0;
      }
    }
    if constexpr (BITS == 16) {
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, kWave);
      if (lane == 0) rowsum[row] = sum;
    }
  }
  __syncthreads();

  // ---- the product: this wave's fragments of K
  v16i acc[NB][NACC];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int c = 0; c < NACC; ++c)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[nb][c][r] = 0;
#pragma unroll
  for (int j = 0; j < KW; ++j) {
    const unsigned kb = wave * KW + j;
    if (kb < kfrags) {
      v4i a[NPL];
#pragma unroll
      for (int pl = 0; pl < NPL; ++pl)
        a[pl] = as_v4i(*reinterpret_cast<const u4*>(stage + (kb * NPL + pl) * kPitch + lh * kHalf + lj * 16));
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        acc[nb][0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[0], as_v4i(fw[nb][j][0]), acc[nb][0], 0, 0, 0);
        if constexpr (BITS == 16) {
          acc[nb][1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[0], as_v4i(fw[nb][j][1]), acc[nb][1], 0, 0, 0);
          acc[nb][2] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[1], as_v4i(fw[nb][j][1]), acc[nb][2], 0, 0, 0);
          acc[nb][1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[1], as_v4i(fw[nb][j][0]), acc[nb][1], 0, 0, 0);
        }
      }
    }
  }
  if constexpr (kShared) __syncthreads();
  typedef uint32_t Vec __attribute__((ext_vector_type(V)));
  Vec* mine = reinterpret_cast<Vec*>(part) + wave * (NB * 1024 / V);
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 16; r += V) {
      Vec x;
#pragma unroll
      for (int t = 0; t < V; ++t) {
        x[t] = (unsigned)acc[nb][0][r + t];
        if constexpr (BITS == 16) x[t] = (x[t] << 16) + ((unsigned)acc[nb][1][r + t] << 8) + (unsigned)acc[nb][2][r + t];
      }
      mine[(nb * 16 + r) / V * 64 + lane] = x;
    }
  __syncthreads();

  const float u = __fdiv_rn(1.0f, __fmul_rn(s, s_w));
  Vec sum[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
    for (int t = 0; t < V; ++t) sum[nb][t] = 0u;
#pragma unroll
    for (int k = 0; k < KS; ++k) sum[nb] += reinterpret_cast<const Vec*>(part)[(k * NB + nb) * (1024 / V) + tid];   // mod 2^32
    if (!has_bias) bias[nb] = 0.f;
  }
  float local_amax = 0.f;
#pragma unroll
  for (int t = 0; t < V; ++t) {
    const unsigned m = m0 + t;
    if (m > M1 || n >= (IN == kRowsPairGate ? p.K1 : p.N)) continue;
    if constexpr (BITS == 16) sum[0][t] += 128u * ((uint32_t)rowsum[m] + cs) - 16384u * p.K;
    float y = fmaf((float)(int)sum[0][t], u, bias[0]);
    if constexpr (IN == kRowsPairGate) {
      const float z2 = fmaf((float)(int)sum[NB - 1][t], u, bias[NB - 1]);
      y = sigmoidf_(y) * gate_in[0][t] + sigmoidf_(z2) * gate_in[NB - 1][t];
      p.Y[(size_t)m * p.K1 + n] = y;
    } else {
      if (p.relu) y = (y > 0.0f) ? y : 0.0f;
      p.Y[(size_t)m * p.N + n] = y;
      local_amax = fmaxf(local_amax, fabsf(y));
    }
  }
  if (p.out_amax != nullptr || p.partial_out != nullptr) {
    // as in k_gemm_small: one maximum per workgroup, without atomics, and/or the raised word.  (`red` was read before
    // the last two barriers.)
    local_amax = __uint_as_float(wave_max_u32(__float_as_uint(local_amax)));
    if (lane == 0) red[wave] = local_amax;
    __syncthreads();
    if (tid == 0) {
      float top = red[0];
#pragma unroll
      for (int k = 1; k < KS; ++k) top = fmaxf(top, red[k]);
      if (p.partial_out != nullptr) p.partial_out[blockIdx.x] = top;
      if (p.out_amax != nullptr) {
        unsigned* dst = reinterpret_cast<unsigned*>(p.out_amax);
        const unsigned bits = __float_as_uint(top);
        if (bits > __hip_atomic_load(dst, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(dst, bits);
      }
    }
  }
}

template <int BITS, int IN, int KS, int CH, int NR>
int launch_rows(const RowsParams& p, hipStream_t s, const RowsFill& fill) {
  constexpr int NPL = BITS == 16 ? 2 : 1, NB = IN == kRowsPairGate ? 2 : 1;
  constexpr size_t stage = (size_t)CH * 8 * NPL * 2 * (512 + 16), part = (size_t)KS * NB * 1024 * sizeof(int);
  constexpr size_t smem = stage + part > 150 * 1024 ? (stage > part ? stage : part) : stage + part;
  static_assert(smem <= 150 * 1024, "LDS budget");
  auto kern = k_gemm_rows<BITS, IN, KS, CH, NR>;
  static bool attr_done = false;
  if (!attr_done) {
    int rc = check_hip(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
    if (rc != MQ_OK) return rc;
    attr_done = true;
  }
  const unsigned grid = IN == kRowsPairGate ? p.K1 / 32 : (unsigned)PackedDims(BITS, p.N, p.K).nblocks;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(KS * 64), smem, s, p, fill);
  return check_hip(hipGetLastError());
}

// Eight waves up to K = 1024; sixteen beyond (64 registers of input per lane: two rows of 2048 or one of 4096).  Few rows
// take the form that holds one row per wave: the others would be converted for nothing.
template <int BITS, int IN>
int launch_rows_k(const RowsParams& p, hipStream_t s, const RowsFill& fill = {}) {
  auto by_rows = [&](auto few, auto many) { return p.M <= 8 ? few(p, s, fill) : many(p, s, fill); };
  if constexpr (IN != kRowsPairGate)
    if (p.K <= 256) return by_rows(launch_rows<BITS, IN, 8, 1, 1>, launch_rows<BITS, IN, 8, 1, 4>);
  if (p.K <= 512) return by_rows(launch_rows<BITS, IN, 8, 2, 1>, launch_rows<BITS, IN, 8, 2, 4>);
  if (p.K <= 1024) return by_rows(launch_rows<BITS, IN, 8, 4, 1>, launch_rows<BITS, IN, 8, 4, 4>);
  if constexpr (IN == kRowsPlain || IN == kRowsPairGate) {
    if (p.K <= 2048) return p.M <= 16 ? launch_rows<BITS, IN, 16, 8, 1>(p, s, fill) : launch_rows<BITS, IN, 16, 8, 2>(p, s, fill);
    if constexpr (BITS == 8 && IN == kRowsPlain)
      if (p.K <= 4096 && p.M <= 16) return launch_rows<8, IN, 16, 16, 1>(p, s, fill);
  }
  return MQ_ERR_UNSUPPORTED;
}

RowsParams rows_params(const GemmArgs& a) {
  RowsParams p{};
  p.packedW = static_cast<const uint8_t*>(a.packedW);
  p.M = (unsigned)a.M; p.N = (unsigned)a.N; p.K = (unsigned)a.K;
  p.sW = a.sW; p.bias = a.bias; p.relu = a.relu; p.Y = a.Y; p.out_amax = a.out_amax; p.partial_out = a.partial;
  return p;
}

}  // namespace

bool gemm_rows_supported(int bits, size_t M, size_t N, size_t K) {
  if (M < 1 || M > 32 || N < 1 || K < 4 || K % 4 != 0) return false;
  return K <= 2048 || (bits == 8 && K <= 4096 && M <= 16);
}
// With abs-max this form saves one launch at least and wins everywhere (K 4 .. 4096, 1 .. 32 rows, in us: 8 bit, K = 512 4.1
// against 7.3, K = 1024 5.2 against 8.1, K = 2048 17 rows 7.6 against 9.0, K = 4096 9.3 against 10.1; 16 bit, K = 2048 17
// rows 10.3 against 13.1).  With a given multiplier the others need one launch less and convert an element once, not once
// per 32 columns, so it depends on how much every workgroup here converts, all pieces of 256 elements of every row a wave
// holds (see launch_rows_k):
//   * 8 bit with quant_int in the operand fetch, K in 513 .. 1024, four rows per wave: 5.0 - 5.1 against 4.6 - 4.8 us
//     (K = 512 3.9 against 4.3, one row per wave 3.7 against 4.7);
//   * 8 bit, two launches: K in 1025 .. 2048 with two rows per wave 7.2 - 7.4 against 6.3 - 6.5 (with one 5.1 - 5.4 against
//     6.2 - 6.5), K above 2048 8.5 - 9.1 against 7.0 - 7.6;
//   * 16 bit, whose product takes longer the longer K is: K in 1025 .. 1536 with two rows per wave 9.6 - 9.8 against 8.7 -
//     9.5, K = 1800 10.1 against 10.2, K = 2048 10.1 against 10.4 (with one row 7.0 - 7.6 against 8.4 - 10.4).
bool gemm_rows_ahead_given(int bits, size_t M, size_t K, bool in_fetch) {
  if (in_fetch) return M <= 8 || K <= 512;
  if (bits == 16) return M <= 16 || K <= 1024 || K > 1664;
  return K <= 1024 || (K <= 2048 && M <= 16);
}
size_t gemm_rows_partials(size_t N) { return (N + 31) / 32; }
bool gemm_rows_glue_supported(size_t M, size_t d) { return M >= 1 && M <= 32 && d % 256 == 0 && d <= 1024; }

int launch_gemm_rows(const float* A, const float* scale, const GemmArgs& a, hipStream_t s) {
  if (!gemm_rows_supported(a.bits, a.M, a.N, a.K)) return MQ_ERR_UNSUPPORTED;
  RowsParams p = rows_params(a);
  p.a = A; p.scale = scale;
  return a.bits == 16 ? launch_rows_k<16, kRowsPlain>(p, s) : launch_rows_k<8, kRowsPlain>(p, s);
}

int launch_gemm_rows_average(const float* g_prev, const float* x, int t, float* g, const GemmArgs& a, hipStream_t s,
                             const RowsFill& fill) {
  if (!gemm_rows_glue_supported(a.M, a.K) || a.bits != 8) return MQ_ERR_UNSUPPORTED;
  RowsParams p = rows_params(a);
  p.a = g_prev; p.b = x; p.tm1 = (float)(t - 1); p.t = (float)t; p.side = g;
  return launch_rows_k<8, kRowsAverage>(p, s, fill);
}

int launch_gemm_rows_gate(const float* x, const float* f, const GemmArgs& a, hipStream_t s) {
  const size_t d = a.K / 2;
  if (!gemm_rows_glue_supported(a.M, d) || a.K != 2 * d || a.N != 2 * d || a.bits != 8) return MQ_ERR_UNSUPPORTED;
  RowsParams p = rows_params(a);
  p.a = x; p.b = f; p.K1 = (unsigned)d; p.out_amax = nullptr; p.partial_out = nullptr;
  return launch_rows_k<8, kRowsPairGate>(p, s);
}

int launch_gemm_rows_norm(const float* h, const float* r, const float* gamma, const float* beta, float eps, float* y,
                          const GemmArgs& a, hipStream_t s) {
  if (!gemm_rows_glue_supported(a.M, a.K) || a.bits != 8) return MQ_ERR_UNSUPPORTED;
  RowsParams p = rows_params(a);
  p.a = h; p.b = r; p.gamma = gamma; p.beta = beta; p.eps = eps; p.side = y;
  return launch_rows_k<8, kRowsNorm>(p, s);
}

}  // namespace mq
