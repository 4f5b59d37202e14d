// dot'_int for decode-sized activations (arxiv 1805.12096, Section 4.3: the
// product of two quantized tensors, both contiguous along K; Section 3.2: a
// decoder step multiplies a few hundred rows by every parameter matrix).
//
// With a few hundred rows the whole product is some ten thousand matrix
// instructions, a few per SIMD: time is latency, not throughput.  The tiled
// kernel walks K in a software pipeline, one stage after the other, which is
// the wrong shape for that.  Here the contraction is cut ACROSS the waves of a
// workgroup instead: a workgroup owns a 32- or 64-row by 32-column piece of the
// result, each of its waves takes a contiguous run of K, asks for all of its
// operand fragments at once (one round trip to L2), multiplies, and the partial
// sums meet in LDS.  Integer addition is exact, so the split changes no bit.
// Both operands are in fragment order; a fragment is one coalesced 1 KB read
// straight into the registers the matrix instruction takes.
#include "mq_gemm_common.h"
#include "mq_grid_max.h"

namespace mq {

namespace {

// A workgroup's max|y| into the caller's word(s), by one thread.  Same-address atomics are served one after the other, about
// 12 ns each, and the workgroups of these kernels end together: hundreds of them on one word are a tail of microseconds.  Of
// those that find it clear an eighth goes first; the others look again when those are through, and few are left with more than
// the maximum of so many.  (Who finds something there comes later than others, and waits for nobody; long sums, counted in byte
// planes, end further apart.)  Clearing the word and the quantizer included, on split K: 309 x 1500 x 1024 in 16 bit 15.7 -> 14.3 us
// (tiles 17.3), 224 x 2048 x 512 16.4 -> 15.0 (15.8), 957 x 512 x 700 19.8 -> 17.9 (19.6).
__device__ __forceinline__ void raise_amax(float* words, unsigned slots, float mx, unsigned length) {
  unsigned* dst = reinterpret_cast<unsigned*>(words) + (slots > 1 ? blockIdx.x % slots : 0);
  const unsigned bits = __float_as_uint(mx);
  unsigned there = __hip_atomic_load(dst, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (there == 0u && slots <= 1 && length <= 2048 && gridDim.x > 128 && blockIdx.x / 8 % 8 != 0) {
    const unsigned long long t0 = wall_clock64(), wait = 50 + gridDim.x / 8 * 12 / 10;      // ticks of 10 ns
    while (wall_clock64() - t0 < wait) __builtin_amdgcn_s_sleep(2);
    there = __hip_atomic_load(dst, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (bits > there) atomicMax(dst, bits);
}

// Arguments of k_gemm_small: two cache lines, what the operands' addresses need in the first.  (Every line is a miss of its own
// on each launch, about 0.15 us where the compiler puts it in front of the loads.)
struct SmallParams {
  const uint8_t *qA, *packedW;
  unsigned M, N, K;
  Tiles tiles;
  int dequant, relu;
  const float *sA, *sW, *bias;
  float* Y;                  // with dequant == 0 the raw sums, int32; with REQUANT the packed operand
  float* out_amax;           // with REQUANT the multiplier
  float* partial;            // optional: max|y| of every workgroup
  unsigned amax_slots;       // words at out_amax the workgroups spread over (0 or 1: one)
};
static_assert(sizeof(SmallParams) <= 128, "two cache lines");

// TMW: 32-row blocks per workgroup; KS: waves (= parts of K); KW: fragments per operand row block and round.
// BITS == 16: every fragment is two byte planes (high byte; low byte with its top bit flipped) and a result
// tile takes four products into three accumulators (hh, hl + lh, ll); a wave's partial sum is their
// recombination 2^16 hh + 2^8 mid + ll (mod 2^32), which adds up over the waves like the 8-bit sums, and the
// plane offsets are corrected once at the end: + 128 (rowsum[m] + colsum[n]) - 16384 K.
//
// REQUANT (16 bit, one row block): the results go to memory once, as the packed operand of the next product, quantized with a
// multiplier that was given.  The operands change places in the matrix instruction, so that a thread's four values are four
// columns of a row, which are neighbours in a fragment.
template <int BITS, int TMW, int KS, int KW, bool REQUANT = false>
__global__ __launch_bounds__(KS * 64) void k_gemm_small(const SmallParams p) {
  static_assert(!REQUANT || (BITS == 16 && TMW == 1 && KS >= 4), "one form");
  const int dequant = REQUANT ? 1 : p.dequant;
  constexpr int NPL = BITS == 16 ? 2 : 1;
  constexpr int NACC = BITS == 16 ? 3 : 1;
  extern __shared__ __attribute__((aligned(16))) int part[];      // [KS][TMW * 1024]
  const int tid = threadIdx.x, lane = tid % 64;
  // The wave index, and with it the wave's run of K, must be wave-uniform to the COMPILER (scalar registers,
  // scalar branches): a matrix instruction under a lane mask is executed even when the mask is empty.
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const PackedDims dA(BITS, p.M, p.K), dW(BITS, p.N, p.K);
  unsigned tile_m, tile_n;
  tile_at(blockIdx.x, p.tiles, tile_m, tile_n);
  const unsigned kfrags = (unsigned)dA.kfrags;
  const unsigned per = (kfrags + KS - 1) / KS;
  const unsigned kb_begin = wave * per;
  const unsigned kb_end = kb_begin + per < kfrags ? kb_begin + per : kfrags;

  // row blocks of the tile; one past the end is clamped (its rows are masked when stored)
  const uint8_t* a_src[TMW];
#pragma unroll
  for (int mt = 0; mt < TMW; ++mt) {
    unsigned rb = tile_m * TMW + mt;
    if (rb >= dA.nblocks) rb = (unsigned)dA.nblocks - 1;
    a_src[mt] = p.qA + dA.frag_offset(rb, 0) + lane * 16;
  }
  const uint8_t* w_src = p.packedW + dW.frag_offset(tile_n, 0) + lane * 16;

  // The epilogue's constants are asked for before the operands: loaded where they are used, they are a memory
  // round trip that nothing hides.  They are only looked at after the operands have been asked for as well, and no
  // load sits under a condition (a branch with a wait behind it): where there is nothing to load, a valid address is
  // read and the value not used.  Every element a thread finishes has e % 64 == lane, so they share the column n and
  // the bias.
  const int lj = lane % 32, lh = lane / 32;
  const unsigned n = tile_n * 32 + lj;
  const bool n_ok = n < p.N;
  const float* some = reinterpret_cast<const float*>(p.packedW);
  const bool has_bias = dequant && p.bias != nullptr;
  const float s_a = *(dequant ? p.sA : some), s_w = *(dequant ? p.sW : some);
  const float bias_raw = (has_bias ? p.bias : some)[has_bias ? min(n, p.N - 1) : 0u];

  // The partial sums meet in vectors of V rows, the widest that leaves every thread one: vector i of a thread holds rows
  // row_of(i) .. + V - 1 of column n.  16 bit: their sums and the column's are asked for here as well.
  constexpr int kEach = TMW * 1024 / (KS * 64), V = kEach >= 4 || REQUANT ? 4 : kEach, NV = REQUANT ? 1 : kEach / V;
  static_assert(V >= 1 && (REQUANT || NV * V * KS * 64 == TMW * 1024), "elements must divide over the threads");
  typedef uint32_t Vec __attribute__((ext_vector_type(V)));
  auto row_of = [&](int i) -> unsigned {
    const int g = (tid + i * KS * 64) / 64 * V, mt = g / 16, r = g % 16;
    return (tile_m * TMW + mt) * 32 + 8 * (r / 4) + 4 * lh + r % 4;
  };
  uint32_t rs[BITS == 16 ? NV : 1][V];
  uint32_t cs = 0;
  // REQUANT: threads 0 .. 255 finish row lj of the block, columns q0 .. q0 + 3
  const unsigned q0 = 8 * (wave % 4) + 4 * lh;
  float s_given = 0.f, bias4[4];
  if constexpr (REQUANT) {
    const uint32_t* rowsum = reinterpret_cast<const uint32_t*>(p.qA + dA.plane_bytes());
    const uint32_t* colsum = reinterpret_cast<const uint32_t*>(p.packedW + dW.plane_bytes());
    s_given = *p.out_amax;
    cs = rowsum[tile_m * 32 + lj];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      rs[0][t] = colsum[tile_n * 32 + q0 + t];
      bias4[t] = (has_bias ? p.bias : some)[has_bias ? min(tile_n * 32 + q0 + t, p.N - 1) : 0u];
    }
  } else if constexpr (BITS == 16) {
    const uint32_t* rowsum = reinterpret_cast<const uint32_t*>(p.qA + dA.plane_bytes());
    const uint32_t* colsum = reinterpret_cast<const uint32_t*>(p.packedW + dW.plane_bytes());
    cs = colsum[n];                                                // (the sums cover the padded rows of both operands)
#pragma unroll
    for (int i = 0; i < NV; ++i)
#pragma unroll
      for (int t = 0; t < V; ++t) rs[i][t] = rowsum[min(row_of(i) + t, (unsigned)dA.Np - 1)];
  }

  v16i acc[TMW][NACC];
#pragma unroll
  for (int mt = 0; mt < TMW; ++mt)
#pragma unroll
    for (int c = 0; c < NACC; ++c)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mt][c][r] = 0;

  for (unsigned kb0 = kb_begin; kb0 < kb_end; kb0 += KW) {
    u4 fa[TMW][KW][NPL], fw[KW][NPL];
#pragma unroll
    for (int j = 0; j < KW; ++j) {
      // a fragment past this wave's run is read from the run's last one (a valid address) and not used
      const unsigned kb = kb0 + j < kb_end ? kb0 + j : kb_end - 1;
#pragma unroll
      for (int pl = 0; pl < NPL; ++pl) {
        fw[j][pl] = *reinterpret_cast<const u4*>(w_src + ((size_t)kb * NPL + pl) * kFragBytes);
#pragma unroll
        for (int mt = 0; mt < TMW; ++mt)
          fa[mt][j][pl] = *reinterpret_cast<const u4*>(a_src[mt] + ((size_t)kb * NPL + pl) * kFragBytes);
      }
    }
    // All of a trip's loads are out before its first product (the compiler would rather save registers).  Products under no
    // condition of their own: a fragment that is only used under one is loaded under it, too (the compiler
    // moves the load down), behind the other fragments' products and with a round trip to memory to itself.  Fragments of the
    // parameter past the run count as zero instead.
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < KW; ++j) {
      const uint32_t inside = kb0 + j < kb_end ? ~0u : 0u;
#pragma unroll
      for (int pl = 0; pl < NPL; ++pl) fw[j][pl] &= inside;
#pragma unroll
      for (int mt = 0; mt < TMW; ++mt) {
        if constexpr (BITS == 8) {
          acc[mt][0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(as_v4i(fa[mt][j][0]), as_v4i(fw[j][0]), acc[mt][0], 0, 0, 0);
        } else {
          if constexpr (REQUANT) {
            acc[mt][0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(as_v4i(fw[j][0]), as_v4i(fa[mt][j][0]), acc[mt][0], 0, 0, 0);
            acc[mt][1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(as_v4i(fw[j][1]), as_v4i(fa[mt][j][0]), acc[mt][1], 0, 0, 0);
            acc[mt][2] = __builtin_amdgcn_mfma_i32_32x32x32_i8(as_v4i(fw[j][1]), as_v4i(fa[mt][j][1]), acc[mt][2], 0, 0, 0);
            acc[mt][1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(as_v4i(fw[j][0]), as_v4i(fa[mt][j][1]), acc[mt][1], 0, 0, 0);
            continue;
          }
          acc[mt][0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(as_v4i(fa[mt][j][0]), as_v4i(fw[j][0]), acc[mt][0], 0, 0, 0);
          acc[mt][1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(as_v4i(fa[mt][j][0]), as_v4i(fw[j][1]), acc[mt][1], 0, 0, 0);
          acc[mt][2] = __builtin_amdgcn_mfma_i32_32x32x32_i8(as_v4i(fa[mt][j][1]), as_v4i(fw[j][1]), acc[mt][2], 0, 0, 0);
          acc[mt][1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(as_v4i(fa[mt][j][1]), as_v4i(fw[j][0]), acc[mt][1], 0, 0, 0);
        }
      }
    }
  }

  const float u = dequant ? __fdiv_rn(1.0f, __fmul_rn(s_a, s_w)) : 0.f, bias = has_bias ? bias_raw : 0.f;
  const uint32_t corr = 128u * cs - 16384u * p.K;
  float local_amax = 0.f;
  // partial sums of this wave, V consecutive rows at a time: vector e = group * 64 + lane, group = (mt * 16 + r) / V
  // (REQUANT: registers are columns and lanes rows)
  Vec* mine = reinterpret_cast<Vec*>(part) + wave * (TMW * 1024 / V);
#pragma unroll
  for (int mt = 0; mt < TMW; ++mt)
#pragma unroll
    for (int r = 0; r < 16; r += V) {
      Vec v;
#pragma unroll
      for (int t = 0; t < V; ++t) {
        v[t] = (unsigned)acc[mt][0][r + t];
        if constexpr (BITS == 16) v[t] = (v[t] << 16) + ((unsigned)acc[mt][1][r + t] << 8) + (unsigned)acc[mt][2][r + t];
      }
      mine[(mt * 16 + r) / V * 64 + lane] = v;
    }
  __syncthreads();

  if constexpr (REQUANT) {
    // (the padding is the value 0, as the quantizer writes it; the row sums the next product corrects with are of the values)
    const PackedDims dO(16, p.M, p.N);
    __shared__ int row_part[4][32];
    if (wave < 4) {
      Vec v = reinterpret_cast<const Vec*>(part)[tid];
#pragma unroll
      for (int w = 1; w < KS; ++w) v += reinterpret_cast<const Vec*>(part)[w * 256 + tid];      // mod 2^32
      const unsigned m = tile_m * 32 + lj;
      uint32_t hi = 0, lo = 0;
      int row = 0;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const unsigned sum = v[t] + 128u * rs[0][t] + corr;
        float y = fmaf((float)(int)sum, u, has_bias ? bias4[t] : 0.f);
        if (p.relu) y = fmaxf(y, 0.0f);                          // NaN -> 0
        const float r = rintf(__fmul_rn(y, s_given));
        int q;
        asm("v_cvt_i32_f32 %0, %1" : "=v"(q) : "v"(r));          // saturates, NaN -> 0
        q = min(max(q, -32767), 32767);
        if (m >= p.M || tile_n * 32 + q0 + t >= p.N) q = 0;
        row += q;
        hi |= (uint32_t)((q >> 8) & 0xFF) << (8 * t);
        lo |= (uint32_t)((q & 0xFF) ^ 0x80) << (8 * t);
      }
      uint8_t* dst = reinterpret_cast<uint8_t*>(p.Y) + dO.frag_offset(tile_m, tile_n) + (lj + 32 * (q0 / 16)) * 16 + q0 % 16;
      *reinterpret_cast<uint32_t*>(dst) = hi;
      *reinterpret_cast<uint32_t*>(dst + kFragBytes) = lo;
      if (tile_n + 1 == dW.nblocks && dO.kfrags > dW.nblocks) {  // the packed width is whole pairs of fragments
        *reinterpret_cast<uint32_t*>(dst + 2 * kFragBytes) = 0u;
        *reinterpret_cast<uint32_t*>(dst + 3 * kFragBytes) = 0x80808080u;
      }
      row += __shfl_xor(row, 32, 64);
      if (lh == 0) row_part[wave][lj] = row;
    }
    __syncthreads();
    if (tid < 32 && tile_m * 32 + tid < p.M)
      atomicAdd(reinterpret_cast<int*>(reinterpret_cast<uint8_t*>(p.Y) + dO.plane_bytes()) + tile_m * 32 + tid,
                row_part[0][tid] + row_part[1][tid] + row_part[2][tid] + row_part[3][tid]);
    return;
  }

  // Every thread adds up the KS partial sums of NV vectors.
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    Vec v;
#pragma unroll
    for (int t = 0; t < V; ++t) v[t] = 0u;
#pragma unroll
    for (int w = 0; w < KS; ++w) v += reinterpret_cast<const Vec*>(part)[w * (TMW * 1024 / V) + tid + i * KS * 64];      // mod 2^32
    const unsigned m0 = row_of(i);
#pragma unroll
    for (int t = 0; t < V; ++t) {
      const unsigned m = m0 + t;
      if (n_ok && m < p.M) {
        unsigned sum = v[t];
        if constexpr (BITS == 16) sum += 128u * rs[i][t] + corr;
        if (dequant) {
          float y = fmaf((float)(int)sum, u, bias);
          if (p.relu) y = (y > 0.0f) ? y : 0.0f;
          p.Y[(size_t)m * p.N + n] = y;
          local_amax = fmaxf(local_amax, fabsf(y));
        } else {
          reinterpret_cast<int*>(p.Y)[(size_t)m * p.N + n] = (int)sum;
        }
      }
    }
  }
  if (dequant && (p.out_amax != nullptr || p.partial != nullptr)) {
    // block-wide maximum of |y|: one value per workgroup in p.partial (no atomics; the next quantizer reduces
    // them), and/or raised into *p.out_amax with at most one atomic per block; the running maximum only
    // grows, so a block that cannot raise it skips the atomic
    __shared__ float wave_amax[KS];
    local_amax = __uint_as_float(wave_max_u32(__float_as_uint(local_amax)));      // non-negative: ordered like its bits
    if (lane == 0) wave_amax[wave] = local_amax;
    __syncthreads();
    if (tid == 0) {
      float mx = wave_amax[0];
#pragma unroll
      for (int w = 1; w < KS; ++w) mx = fmaxf(mx, wave_amax[w]);
      if (p.partial != nullptr) p.partial[blockIdx.x] = mx;
      if (p.out_amax != nullptr) raise_amax(p.out_amax, p.amax_slots, mx, NPL * p.K);
    }
  }
}

template <int BITS, int TMW, int KS, int KW, bool REQUANT = false>
int launch_small(const GemmArgs& a, int dequant, hipStream_t s) {
  constexpr size_t smem = (size_t)KS * TMW * 1024 * sizeof(int);
  static_assert(smem <= 128 * 1024, "LDS budget");
  const PackedDims dA(BITS, a.M, a.K), dW(BITS, a.N, a.K);
  const size_t tiles_m = (dA.nblocks + TMW - 1) / TMW, tiles_n = dW.nblocks;
  SmallParams p{};
  p.qA = static_cast<const uint8_t*>(a.qA);
  p.packedW = static_cast<const uint8_t*>(a.packedW);
  p.M = (unsigned)a.M; p.N = (unsigned)a.N; p.K = (unsigned)a.K;
  p.dequant = dequant; p.relu = a.relu;
  p.sA = a.sA; p.sW = a.sW; p.bias = a.bias; p.Y = dequant ? a.Y : reinterpret_cast<float*>(a.C);
  p.out_amax = a.out_amax; p.partial = a.partial; p.amax_slots = a.amax_slots;
  if constexpr (REQUANT) {
    p.Y = static_cast<float*>(a.packed_out);
    p.out_amax = a.s_out;
  }
  if (tiles_m * tiles_n > 0x7FFFFFFFull) return MQ_ERR_SHAPE;
  p.tiles = tiles_of(tiles_m, tiles_n, TMW);
  auto kern = k_gemm_small<BITS, TMW, KS, KW, REQUANT>;
  static bool attr_done = false;
  if (!attr_done) {
    int rc = check_hip(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
    if (rc != MQ_OK) return rc;
    attr_done = true;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_m * tiles_n)), dim3(KS * 64), smem, s, p);
  return check_hip(hipGetLastError());
}

// The first product of the 8-bit block for few rows: relu?(A W + b), max|.| over the whole result, quant_int with 127 / max, in
// one launch (see mq_grid_max.h; every workgroup is resident).  The tiles' form (k_gemm_pp) walks K behind a pipeline and gives
// 128 x 128 of the result to a workgroup: up to a few hundred rows it leaves most of the chip idle.  Here K is split over the
// waves as in k_gemm_small; a workgroup takes TMW row blocks, the fewest that fit the grid's one round, and keeps its values in
// registers while the maxima travel.  The operands change places in the matrix instruction, so that a thread's four values are
// neighbours in a fragment of the packed result.  TMW row blocks, NB column blocks of a workgroup: two column blocks share the
// rows' reads (4 x 1 at 1001 rows would not fit the round, and reads 1.7 times as much per result).
// Whole block on a prepared workspace, us, tiles and this: 512 / 2048: 64 rows 16.0 and 12.4, 200 rows 17.0 and 13.7, 500 rows 18.1
// and 15.5, 1001 rows 20.4 and 18.4, 1024 rows 18.8 and 18.4; 1024 / 4096: 64 rows 19.2 and 14.0, 200 rows 21.0 and 17.3, 500
// rows 25.2 and 23.2; 1000 / 1000: 1200 rows 24.0 and 21.4; 128 / 4096: 400 rows 16.7 and 16.8.  However long K is: 2048 / 512:
// 32 rows 20.5 and 12.0, 1001 rows 28.1 and 19.8, 4096 rows 37.9 and 37.5; 4096 / 2048: 100 rows 31.4 and 17.3, 1001 rows 47.0
// and 43.8; 8192 / 512: 500 rows 53.2 and 27.5, 4096 rows 139 and 138.
struct AgreeParams {
  const uint8_t *qA, *packedW;
  unsigned M, N, K;
  Tiles tiles;
  int relu;
  unsigned nclear;
  const float *sA, *sW, *bias;
  uint8_t* packed_out;
  float* s_out;
  unsigned* barrier;
  unsigned* clear_words;     // optional: words of an earlier kernel's agreement, left zero
  unsigned long long ticks;
};

template <int TMW, int NB>
__global__ __launch_bounds__(512) void k_gemm_small_agree(const AgreeParams p) {
  constexpr int KS = 8 / NB, KW = 4, NV = TMW * NB <= 2 ? 1 : TMW * NB / 2;      // a vector: four columns of a row
  static_assert(NB == 1 || TMW == 4, "a round of vectors lies in one column block");
  extern __shared__ __attribute__((aligned(16))) int part[];      // [NB][KS][TMW * 256] vectors
  __shared__ float red[8];
  const int tid = threadIdx.x, lane = tid % 64, lj = lane % 32, lh = lane / 32;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const PackedDims dA(8, p.M, p.K), dW(8, p.N, p.K), dO(8, p.M, p.N);
  unsigned tile_m, tile_n;
  tile_at(blockIdx.x, p.tiles, tile_m, tile_n);
  const unsigned kfrags = (unsigned)dA.kfrags, per = (kfrags + KS - 1) / KS;
  const unsigned k_part = wave % KS, block = min(tile_n * NB + wave / KS, (unsigned)dW.nblocks - 1);      // of this wave
  const unsigned kb_begin = min(k_part * per, kfrags - 1), kb_end = min(k_part * per + per, kfrags);
  const bool some_k = k_part * per < kfrags;
  const uint8_t* a_src[TMW];
#pragma unroll
  for (int mt = 0; mt < TMW; ++mt) a_src[mt] = p.qA + dA.frag_offset(min(tile_m * TMW + mt, (unsigned)dA.nblocks - 1), 0) + lane * 16;
  const uint8_t* w_src = p.packedW + dW.frag_offset(block, 0) + lane * 16;

  // vector i of a thread: column block 2 i / TMW of the tile, row block (wave + 8 i) / 4 % TMW, row lj, columns q0 .. q0 + 3
  const unsigned q0 = 8 * (wave % 4) + 4 * lh;
  auto column = [&](int i) { return (tile_n * NB + (NB == 1 ? 0 : 2 * i / TMW)) * 32 + q0; };
  auto row_block = [&](int i) { return tile_m * TMW + (wave + 8 * i) / 4 % TMW; };
  const float* some = reinterpret_cast<const float*>(p.packedW);
  const float s_a = *p.sA, s_w = *p.sW;
  float bias[NB][4];
#pragma unroll
  for (int c = 0; c < NB; ++c)
#pragma unroll
    for (int t = 0; t < 4; ++t)
      bias[c][t] = (p.bias != nullptr ? p.bias : some)[p.bias != nullptr ? min((tile_n * NB + c) * 32 + q0 + t, p.N - 1) : 0u];

  v16i acc[TMW];
#pragma unroll
  for (int mt = 0; mt < TMW; ++mt)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[mt][r] = 0;
  if (some_k)
    for (unsigned kb0 = kb_begin; kb0 < kb_end; kb0 += KW) {
      u4 fa[TMW][KW], fw[KW];
#pragma unroll
      for (int j = 0; j < KW; ++j) {
        const unsigned kb = min(kb0 + j, kb_end - 1);
        fw[j] = *reinterpret_cast<const u4*>(w_src + (size_t)kb * kFragBytes);
#pragma unroll
        for (int mt = 0; mt < TMW; ++mt) fa[mt][j] = *reinterpret_cast<const u4*>(a_src[mt] + (size_t)kb * kFragBytes);
      }
      __builtin_amdgcn_sched_barrier(0);                           // (see k_gemm_small)
#pragma unroll
      for (int j = 0; j < KW; ++j) {
        fw[j] &= kb0 + j < kb_end ? ~0u : 0u;
#pragma unroll
        for (int mt = 0; mt < TMW; ++mt)
          acc[mt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(as_v4i(fw[j]), as_v4i(fa[mt][j]), acc[mt], 0, 0, 0);
      }
    }
  if (p.clear_words != nullptr && blockIdx.x == 0)
    for (unsigned i = tid; i < p.nclear; i += 512) p.clear_words[i] = 0u;

  typedef uint32_t Vec __attribute__((ext_vector_type(4)));
  Vec* sums = reinterpret_cast<Vec*>(part);
#pragma unroll
  for (int mt = 0; mt < TMW; ++mt)
#pragma unroll
    for (int r = 0; r < 16; r += 4)
      sums[wave * (TMW * 256) + (mt * 4 + r / 4) * 64 + lane] =
          Vec{(unsigned)acc[mt][r], (unsigned)acc[mt][r + 1], (unsigned)acc[mt][r + 2], (unsigned)acc[mt][r + 3]};
  __syncthreads();
  const float u = __fdiv_rn(1.0f, __fmul_rn(s_a, s_w));
  const bool active = TMW * NB > 1 || wave < 4;
  float y[NV][4], top = 0.f;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const unsigned m = row_block(i) * 32 + lj, n0 = column(i);
    const int c = NB == 1 ? 0 : 2 * i / TMW;
    Vec v = {0u, 0u, 0u, 0u};
    if (active)
#pragma unroll
      for (int w = 0; w < KS; ++w) v += sums[(c * KS + w) * (TMW * 256) + (tid + i * 512) % (TMW * 256)];      // mod 2^32
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      y[i][t] = fmaf((float)(int)v[t], u, p.bias != nullptr ? bias[c][t] : 0.f);
      if (p.relu) y[i][t] = fmaxf(y[i][t], 0.0f);                  // NaN -> 0
      if (!active || m >= p.M || n0 + t >= p.N) y[i][t] = 0.f;     // the padding is the value 0
      top = fmaxf(top, fabsf(y[i][t]));
    }
  }
  top = __uint_as_float(wave_max_u32(__float_as_uint(top)));
  if (lane == 0) red[wave] = top;
  __syncthreads();
  if (wave == 0) {
    if (lane == 0) {
#pragma unroll
      for (int w = 1; w < 8; ++w) top = fmaxf(top, red[w]);
      grid_max_publish(p.barrier, top);
    }
    const float amax = grid_max_collect(p.barrier, p.ticks);
    if (lane == 0) red[0] = amax;
  }
  __syncthreads();
  const float amax = red[0], s2 = amax > 0.0f ? __fdiv_rn(127.0f, amax) : 1.0f;
  if (active)
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const unsigned rb = row_block(i), cb = column(i) / 32;
      if (rb >= dO.nblocks || cb >= dW.nblocks) continue;
      int q[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const float r = rintf(__fmul_rn(y[i][t], s2));
        asm("v_cvt_i32_f32 %0, %1" : "=v"(q[t]) : "v"(r));         // saturates, NaN -> 0
        q[t] = min(max(q[t], -127), 127);
      }
      uint8_t* dst = p.packed_out + dO.frag_offset(rb, cb) + (lj + 32 * (q0 / 16)) * 16 + q0 % 16;
      *reinterpret_cast<uint32_t*>(dst) = __builtin_amdgcn_perm((uint32_t)q[1], (uint32_t)q[0], 0x0c0c0400u) |
                                          __builtin_amdgcn_perm((uint32_t)q[3], (uint32_t)q[2], 0x04000c0cu);
      if (cb + 1 == dW.nblocks && dO.kfrags > dW.nblocks) *reinterpret_cast<uint32_t*>(dst + kFragBytes) = 0u;     // whole pairs
    }
  if (blockIdx.x == 0 && tid == 0) *p.s_out = grid_max_failed(p.barrier) ? __builtin_nanf("") : s2;
}

template <int TMW, int NB>
int launch_agree(const GemmArgs& a, hipStream_t s) {
  constexpr size_t smem = (size_t)8 * TMW * 4096;
  static_assert(smem <= 128 * 1024, "LDS budget");
  const PackedDims dA(8, a.M, a.K), dW(8, a.N, a.K);
  const size_t tiles_m = (dA.nblocks + TMW - 1) / TMW, tiles_n = (dW.nblocks + NB - 1) / NB;
  auto kern = k_gemm_small_agree<TMW, NB>;
  static int max_blocks = -1;                   // workgroups the device can hold at once, asked once
  if (max_blocks < 0) {
    int rc = check_hip(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
    if (rc != MQ_OK) return rc;
    int per_cu = 0, dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(kern), 512, smem) != hipSuccess)
      return MQ_ERR_HIP;
    max_blocks = per_cu * cus;
  }
  if (tiles_m * tiles_n > (size_t)max_blocks || tiles_m * tiles_n > kBarrierSlots) return MQ_ERR_UNSUPPORTED;
  if (a.barrier == nullptr) return MQ_ERR_NULL;
  AgreeParams p{};
  p.qA = static_cast<const uint8_t*>(a.qA);
  p.packedW = static_cast<const uint8_t*>(a.packedW);
  p.M = (unsigned)a.M; p.N = (unsigned)a.N; p.K = (unsigned)a.K;
  p.tiles = tiles_of(tiles_m, tiles_n, TMW / NB);
  p.relu = a.relu; p.nclear = a.nclear;
  p.sA = a.sA; p.sW = a.sW; p.bias = a.bias;
  p.packed_out = static_cast<uint8_t*>(a.packed_out); p.s_out = a.s_out;
  p.barrier = a.barrier; p.clear_words = a.clear_words;
  p.ticks = barrier_timeout_ticks();
  hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_m * tiles_n)), dim3(512), smem, s, p);
  return check_hip(hipGetLastError());
}

// quant_int fused into the operand fetch (Section 4.2: activations are quantized on every call): A comes as
// fp32 rows, each lane loads the 16 floats of its fragment slot, multiplies by the multiplier, rounds to
// nearest even, clamps and packs them into the 16 operand bytes.  The multiplier is either given or formed
// here from partial maxima left by the kernel that produced A (127 / max, one correctly rounded division,
// as the separate quantizer does).  Every column block of a row block repeats the conversion of that row
// block; that is cheap next to a launch as long as K is short (the fp32 rows are four times the bytes).
// 16 bit: the bytes are those of the two planes, and a wave also adds up its part of every row's values (a lane holds 16 of a
// row's bytes per fragment for its products; four dot products with ones a plane) and puts 128 of that sum into its partial
// sums, so that the recombination is corrected without a row sum ever leaving the wave.
struct SmallF32Params {
  const float* A;            // [M x K] fp32, K a multiple of 32, rows 16-byte aligned; with A2: [M x K1], columns 0 .. K1 - 1
  const float* A2;           // optional second piece [M x (K - K1)]: columns K1 .. K - 1 of the input
  const float* scale;        // multiplier (npartial == 0) or partial maxima
  const float* scale2;       // more partial maxima (the second piece's), npartial2 of them
  const uint8_t* packedW;
  unsigned M, N, K, K1, tiles_n, npartial, npartial2;
  int relu;
  const float* sW;
  const float* bias;
  float* Y;
  float* scale_out;          // receives the multiplier (workgroup 0)
  float* out_amax;
  float* partial_out;        // optional: max|y| of every workgroup
  unsigned amax_slots;       // words at out_amax the workgroups spread over (0 or 1: one)
};
static_assert(sizeof(SmallF32Params) <= 128, "two cache lines, see SmallParams");

// Four elements of quant_int as bytes.  CLAMP = false: the multiplier is 127 / max over a set these elements belong to,
// rounded, so where it is finite |x s| <= 127 (1 + 2^-23) rounds to at most 127 and no clamp can act (an infinite max
// gives s = 0, products 0 or NaN, and NaN converts to 0 either way).  A max below 127 / FLT_MAX (3.7e-37) gives s = inf,
// and unclamped infinities convert to bytes -1 and 0 where quant_int says 127 and -127: the sums are others then, but
// they are finite and meet the factor 1 / (s sW) = 0, so the result is the bias either way.
template <bool CLAMP>
__device__ __forceinline__ uint32_t quant_pack4(float4 v, float s) {
  auto q = [&](float x) -> uint32_t {
    const float r = rintf(__fmul_rn(x, s));
    int i;
    asm("v_cvt_i32_f32 %0, %1" : "=v"(i) : "v"(r));      // saturates, NaN -> 0
    return (uint32_t)(CLAMP ? min(max(i, -127), 127) : i);
  };
  // bytes 0 of four words: two byte permutes and an or (0x0c selects zero)
  return __builtin_amdgcn_perm(q(v.y), q(v.x), 0x0c0c0400u) | __builtin_amdgcn_perm(q(v.w), q(v.z), 0x04000c0cu);
}
// The same in 16 bit, as the bytes of the two planes (32767 / max instead of 127 / max: the same argument without a clamp).
template <bool CLAMP>
__device__ __forceinline__ void quant_planes4(float4 v, float s, uint32_t& hi, uint32_t& lo) {
  auto q = [&](float x) -> uint32_t {
    const float r = rintf(__fmul_rn(x, s));
    int i;
    asm("v_cvt_i32_f32 %0, %1" : "=v"(i) : "v"(r));
    return (uint32_t)(CLAMP ? min(max(i, -32767), 32767) : i);
  };
  const uint32_t x = q(v.x), y = q(v.y), z = q(v.z), w = q(v.w);
  hi = __builtin_amdgcn_perm(y, x, 0x0c0c0501u) | __builtin_amdgcn_perm(w, z, 0x05010c0cu);
  lo = (__builtin_amdgcn_perm(y, x, 0x0c0c0400u) | __builtin_amdgcn_perm(w, z, 0x04000c0cu)) ^ 0x80808080u;
}

// TNW: 32-column blocks per workgroup; KS waves split K; a round is 4 fragments (128 elements of K).
// Each wave reads its own run of K from the fp32 rows in whole 512-byte pieces (two rows per load
// instruction), converts, and turns the bytes into operand fragments through a private piece of LDS:
// fragment f of a round sits at f * kPitch, K half h of a row at h * kHalf inside it (the paddings
// spread the 4-byte writes of a row over the banks), 16 bytes per row.
// Where its time goes (300 x 2048 x 512, wall clock inside the kernel before the conversion was shortened): 1.6 us until
// all loads are issued (64 KB of fp32 rows and 32 KB of parameter per workgroup through the 64 bytes per clock of a compute
// unit's address path), 1.2 until they and the partial maxima are there, 1.3 for conversion and products, 0.3 for the
// exchange, 1.2 for results and their maximum.  Without clamps where none can act, byte permutes for packing, 16-byte
// exchange through LDS and lane moves for the maxima: this product with its abs-max 9.15 -> 8.3 us, a decoder layer of 300
// sentences 74.1 -> 70.1 us.
// GIVEN: the multiplier is given (elements may exceed it and are clamped); otherwise it comes from partial maxima.
template <int BITS, int TNW, int KS, bool GIVEN>
__global__ __launch_bounds__(KS * 64) void k_gemm_small_f32(const SmallF32Params p) {
  constexpr int KW = 4, NPL = BITS == 16 ? 2 : 1, NACC = BITS == 16 ? 3 : 1;
  constexpr int kHalf = 512 + 16, kPitch = 2 * kHalf;
  extern __shared__ __attribute__((aligned(16))) int part[];      // [KS][TNW * 1024], then the staging pieces
  __shared__ float red[KS];
  const int tid = threadIdx.x, lane = tid % 64;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);      // scalar, see k_gemm_small
  uint8_t* stage = reinterpret_cast<uint8_t*>(part + KS * TNW * 1024) + wave * (NPL * KW * kPitch);
  const PackedDims dW(BITS, p.N, p.K);
  const unsigned tile_n = blockIdx.x % p.tiles_n, tile_m = blockIdx.x / p.tiles_n;
  const unsigned ksl = p.K / 32;                                  // slices that hold real elements
  const unsigned per = (ksl + KS - 1) / KS;
  const unsigned kb_begin = wave * per;
  const unsigned kb_end = kb_begin + per < ksl ? kb_begin + per : ksl;
  const int lj = lane % 32, lh = lane / 32;

  const uint8_t* w_src[TNW];
#pragma unroll
  for (int c = 0; c < TNW; ++c) {
    unsigned nb = tile_n * TNW + c;
    if (nb >= dW.nblocks) nb = (unsigned)dW.nblocks - 1;
    w_src[c] = p.packedW + dW.frag_offset(nb, 0) + lane * 16;
  }
  // load i of a round: row 2 i + lane / 32 of the tile, floats 4 (lane % 32) .. + 3 of the round's 128
  // (rows past the end repeat the last one; their results are never stored)
  unsigned a_row[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    unsigned row = tile_m * 32 + 2 * i + lh;
    if (row >= p.M) row = p.M - 1;
    a_row[i] = row;
  }
  const unsigned ld1 = p.A2 != nullptr ? p.K1 : p.K, ld2 = p.K - p.K1;
  // where this lane's four bytes of load i go: fragment lj / 8, K half (lj / 4) % 2, row 2 i + lh, byte 4 (lj % 4)
  uint8_t* st_dst = stage + (lj / 8) * kPitch + ((lj / 4) % 2) * kHalf + lh * 16 + 4 * (lj % 4);

  float4 fa[16];
  u4 fw[TNW][KW][NPL];
  auto fetch = [&](unsigned kb0) {
#pragma unroll
    for (int j = 0; j < KW; ++j) {
      const unsigned kb = kb0 + j < kb_end ? kb0 + j : kb_end - 1;
#pragma unroll
      for (int c = 0; c < TNW; ++c)
#pragma unroll
        for (int pl = 0; pl < NPL; ++pl)
          fw[c][j][pl] = *reinterpret_cast<const u4*>(w_src[c] + ((size_t)kb * NPL + pl) * kFragBytes);
    }
    // a lane whose fragment lies past the run reads the run's last fragment instead (a valid address, unused)
    const unsigned kb = kb0 + lj / 8 < kb_end ? kb0 + lj / 8 : kb_end - 1;
    const unsigned col = kb * 32 + 4 * (lj % 8);               // this lane's first column of the input
    // two-piece input: the piece, its row stride and the column inside it (K1 is a multiple of 4, so a lane's
    // four floats never straddle the pieces)
    const bool second = p.A2 != nullptr && col >= p.K1;
    const float* base = second ? p.A2 + (col - p.K1) : p.A + col;
    const unsigned ld = second ? ld2 : ld1;
#pragma unroll
    for (int i = 0; i < 16; ++i) fa[i] = *reinterpret_cast<const float4*>(base + (size_t)a_row[i] * ld);
  };
  // The partial maxima and the epilogue's constants first, without conditions around the loads (see k_gemm_small): memory
  // answers in order, so what the multiplier waits for must not stand behind the operands, nor follow its own first trip.
  // A trip serves PV maxima per thread, all 1024 that the producers leave at most.
  constexpr unsigned T = KS * 64, PV = 1024 / T;
  float pv[GIVEN ? 1 : 2 * PV];
  if constexpr (!GIVEN) {
    const unsigned n1 = p.npartial, n2 = p.npartial2;
#pragma unroll
    for (unsigned t = 0; t < PV; ++t) pv[t] = p.scale[min(t * T + tid, n1 - 1)];
    const float* second = n2 != 0 ? p.scale2 : p.scale;          // no second piece: the first one's maxima again
    const unsigned last2 = (n2 != 0 ? n2 : n1) - 1;
#pragma unroll
    for (unsigned t = 0; t < PV; ++t) pv[PV + t] = second[min(t * T + tid, last2)];
  }
  const float sW_pre = *p.sW;
  float bias_pre[TNW];
  uint32_t colsum_pre[BITS == 16 ? TNW : 1];
  const bool has_bias = p.bias != nullptr;
#pragma unroll
  for (int c = 0; c < TNW; ++c) {
    const unsigned n = (tile_n * TNW + c) * 32 + lj;
    bias_pre[c] = (has_bias ? p.bias : p.sW)[has_bias ? min(n, p.N - 1) : 0u];
    if constexpr (BITS == 16)
      colsum_pre[c] = reinterpret_cast<const uint32_t*>(p.packedW + dW.plane_bytes())[min(n, (unsigned)p.N - 1)];
  }
  __builtin_amdgcn_sched_barrier(0);
  // the first round is on its way while the multiplier is formed (a wave without a run of its own fetches the last
  // fragments again: under a condition, the wait for the maxima could not tell whether these loads stand behind them)
  fetch(kb_begin);
  __builtin_amdgcn_sched_barrier(0);

  float s;
  if constexpr (!GIVEN) {
    float m = 0.f;
#pragma unroll
    for (unsigned t = 0; t < 2 * PV; ++t) m = fmaxf(m, pv[t]);
    for (unsigned i = PV * T + tid; i < p.npartial; i += T) m = fmaxf(m, p.scale[i]);
    for (unsigned i = PV * T + tid; i < p.npartial2; i += T) m = fmaxf(m, p.scale2[i]);
    m = __uint_as_float(wave_max_u32(__float_as_uint(m)));
    if (lane == 0) red[wave] = m;
    __syncthreads();
    float amax = red[0];
#pragma unroll
    for (int w = 1; w < KS; ++w) amax = fmaxf(amax, red[w]);
    s = (amax > 0.0f) ? __fdiv_rn(BITS == 16 ? 32767.0f : 127.0f, amax) : 1.0f;
  } else {
    s = *p.scale;
  }
  if (blockIdx.x == 0 && tid == 0 && p.scale_out != nullptr) *p.scale_out = s;

  v16i acc[TNW][NACC];
#pragma unroll
  for (int c = 0; c < TNW; ++c)
#pragma unroll
    for (int b = 0; b < NACC; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[c][b][r] = 0;
  int row = 0;                 // 16 bit: row lj, this lane's half of every fragment: the sum of both planes as one number
  for (unsigned kb0 = kb_begin; kb0 < kb_end; kb0 += KW) {
    if (kb0 != kb_begin) fetch(kb0);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if constexpr (BITS == 8) {
        *reinterpret_cast<uint32_t*>(st_dst + i * 32) = quant_pack4<GIVEN>(fa[i], s);
      } else {
        uint32_t hi, lo;
        quant_planes4<GIVEN>(fa[i], s, hi, lo);
        *reinterpret_cast<uint32_t*>(st_dst + i * 32) = hi;
        *reinterpret_cast<uint32_t*>(st_dst + KW * kPitch + i * 32) = lo;
      }
    }
    // The wave reads back what it wrote itself: LDS operations of one wave complete in order, so the
    // hardware needs no wait.  The compiler does: words are written and 16-byte vectors read, types it may
    // take for non-aliasing, so both sides are fenced against compile-time motion.
    asm volatile("" ::: "memory");
    u4 a[KW][NPL];
#pragma unroll
    for (int j = 0; j < KW; ++j)
#pragma unroll
      for (int pl = 0; pl < NPL; ++pl)
        a[j][pl] = *reinterpret_cast<const u4*>(stage + (pl * KW + j) * kPitch + lh * kHalf + lj * 16);
    asm volatile("" ::: "memory");
#pragma unroll
    for (int j = 0; j < KW; ++j) {
      if (kb0 + j < kb_end) {
        if constexpr (BITS == 8) {
#pragma unroll
          for (int c = 0; c < TNW; ++c)
            acc[c][0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(as_v4i(a[j][0]), as_v4i(fw[c][j][0]), acc[c][0], 0, 0, 0);
        } else {
#pragma unroll
          for (int c = 0; c < TNW; ++c) {
            acc[c][0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(as_v4i(a[j][0]), as_v4i(fw[c][j][0]), acc[c][0], 0, 0, 0);
            acc[c][1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(as_v4i(a[j][0]), as_v4i(fw[c][j][1]), acc[c][1], 0, 0, 0);
            acc[c][2] = __builtin_amdgcn_mfma_i32_32x32x32_i8(as_v4i(a[j][1]), as_v4i(fw[c][j][1]), acc[c][2], 0, 0, 0);
            acc[c][1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(as_v4i(a[j][1]), as_v4i(fw[c][j][0]), acc[c][1], 0, 0, 0);
          }
          int high = 0;
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            high = __builtin_amdgcn_sdot4((int)a[j][0][t], 0x01010101, high, false);
            row = __builtin_amdgcn_sdot4((int)a[j][NPL - 1][t], 0x01010101, row, false);
          }
          row += 256 * high;
        }
      }
    }
  }
  // 16 bit, this wave's run of K: sum (q - 128) of the rows 8 g + 4 lh + t of the tile.  128 (rowsum + colsum) - 16384 K is 128
  // of these sums over the waves + 128 colsum.
  v4i rows_part[BITS == 16 ? 4 : 1];
  if constexpr (BITS == 16) {
    row += __shfl_xor(row, 32, 64);
    asm volatile("" ::: "memory");
    if (lh == 0) reinterpret_cast<int*>(stage)[lj] = row;
    asm volatile("" ::: "memory");
#pragma unroll
    for (int g = 0; g < 4; ++g) rows_part[g] = *reinterpret_cast<const v4i*>(stage + (8 * g + 4 * lh) * 4);
    asm volatile("" ::: "memory");
  }

  // the partial sums meet in vectors of V rows, see k_gemm_small
  constexpr int kEach = TNW * 1024 / (KS * 64), V = kEach % 4 == 0 ? 4 : kEach % 2 == 0 ? 2 : 1, NV = kEach / V;
  static_assert(V >= 1 && NV * V * KS * 64 == TNW * 1024, "elements must divide over the threads");
  typedef uint32_t Vec __attribute__((ext_vector_type(V)));
  Vec* mine = reinterpret_cast<Vec*>(part) + wave * (TNW * 1024 / V);
#pragma unroll
  for (int c = 0; c < TNW; ++c)
#pragma unroll
    for (int r = 0; r < 16; r += V) {
      Vec v;
#pragma unroll
      for (int t = 0; t < V; ++t) {
        v[t] = (unsigned)acc[c][0][r + t];
        if constexpr (BITS == 16)
          v[t] = (v[t] << 16) + ((unsigned)acc[c][1][r + t] << 8) + (unsigned)acc[c][2][r + t] +
                 128u * (unsigned)rows_part[(r + t) / 4][(r + t) % 4];
      }
      mine[(c * 16 + r) / V * 64 + lane] = v;
    }
  __syncthreads();

  const float u = __fdiv_rn(1.0f, __fmul_rn(s, sW_pre));
  float local_amax = 0.f;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    Vec v;
#pragma unroll
    for (int t = 0; t < V; ++t) v[t] = 0u;
#pragma unroll
    for (int w = 0; w < KS; ++w) v += reinterpret_cast<const Vec*>(part)[w * (TNW * 1024 / V) + tid + i * KS * 64];      // mod 2^32
    constexpr int kPerBlock = 16 / V;                                 // groups of a column block
    const int c = (wave + i * KS) / kPerBlock, r = (wave + i * KS) % kPerBlock * V;      // wave-uniform
    float bias = bias_pre[0];
#pragma unroll
    for (int cc = 1; cc < TNW; ++cc)
      if (cc == c) bias = bias_pre[cc];
    if (!has_bias) bias = 0.f;
    uint32_t corr = 0;
    if constexpr (BITS == 16) {
      corr = colsum_pre[0];
#pragma unroll
      for (int cc = 1; cc < TNW; ++cc)
        if (cc == c) corr = colsum_pre[cc];
      corr *= 128u;
    }
    const unsigned n = (tile_n * TNW + c) * 32 + lj;
    const unsigned m0 = tile_m * 32 + 8 * (r / 4) + 4 * lh + r % 4;
#pragma unroll
    for (int t = 0; t < V; ++t)
      if (n < p.N && m0 + t < p.M) {
        float y = fmaf((float)(int)(v[t] + corr), u, bias);
        if (p.relu) y = (y > 0.0f) ? y : 0.0f;
        p.Y[(size_t)(m0 + t) * p.N + n] = y;
        local_amax = fmaxf(local_amax, fabsf(y));
      }
  }
  if (p.out_amax != nullptr || p.partial_out != nullptr) {
    // as in k_gemm_small: one maximum per workgroup, without atomics, and/or the raised word
    __shared__ float wave_amax[KS];
    local_amax = __uint_as_float(wave_max_u32(__float_as_uint(local_amax)));      // non-negative: ordered like its bits
    if (lane == 0) wave_amax[wave] = local_amax;
    __syncthreads();
    if (tid == 0) {
      float mx = wave_amax[0];
#pragma unroll
      for (int w = 1; w < KS; ++w) mx = fmaxf(mx, wave_amax[w]);
      if (p.partial_out != nullptr) p.partial_out[blockIdx.x] = mx;
      if (p.out_amax != nullptr) raise_amax(p.out_amax, p.amax_slots, mx, NPL * p.K);
    }
  }
}

template <int BITS, int TNW, int KS, bool GIVEN>
int launch_small_f32_one(SmallF32Params p, hipStream_t s) {
  constexpr size_t smem = (size_t)KS * TNW * 1024 * sizeof(int) + (size_t)KS * (BITS / 8) * 4 * 2 * (512 + 16);
  static_assert(smem <= 160 * 1024, "LDS budget");
  const PackedDims dW(BITS, p.N, p.K);
  const size_t tiles_m = (p.M + 31) / 32, tiles_n = (dW.nblocks + TNW - 1) / TNW;
  p.tiles_n = (unsigned)tiles_n;
  if (tiles_m * tiles_n > 0x7FFFFFFFull) return MQ_ERR_SHAPE;
  auto kern = k_gemm_small_f32<BITS, TNW, KS, GIVEN>;
  static bool attr_done = false;
  if (!attr_done) {
    int rc = check_hip(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
    if (rc != MQ_OK) return rc;
    attr_done = true;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_m * tiles_n)), dim3(KS * 64), smem, s, p);
  return check_hip(hipGetLastError());
}

template <int BITS, int TNW, int KS>
int launch_small_f32(const SmallF32Params& p, hipStream_t s) {
  return p.npartial != 0 ? launch_small_f32_one<BITS, TNW, KS, false>(p, s) : launch_small_f32_one<BITS, TNW, KS, true>(p, s);
}

size_t row_blocks(size_t M) { return (M + 31) / 32; }
size_t column_blocks(size_t N) { return (N + 31) / 32; }
constexpr size_t kCUs = 256;

// quant_int in the operand fetch: column blocks per workgroup and waves.  What counts is the rounds: with K up to 512 a
// workgroup is four waves and up to four share a compute unit, beyond it is eight with the unit's LDS to themselves, and
// every workgroup converts all its rows, so more columns per workgroup convert less but leave units idle.  Up to K = 512 two
// column blocks from 160 workgroups on, three where they fit one round and two do not (abs-max and product, 300 x 2048 x 512:
// 8.4 -> 7.9 us, 350 rows 8.5 -> 8.0).  Beyond, the fewest columns that fit one round (300 x 2048 x 1024: three blocks 9.1,
// two in two rounds 12.4; 150 x 4096 x 1024 9.1 and 12.4; 250 x 1024 x 1024 one block 7.5, two 8.1), else workgroups of four
// waves, two to a unit (512 x 2048 x 1024 10.9 for 13.1, 256 x 4096 x 1024 11.0 for 13.2).
// 16 bit (twice the products and twice the parameter's bytes), abs-max and product: up to K = 512 one column block on four waves
// (384 x 512 x 512 7.2 us; eight waves 8.0, two blocks 8.0), beyond on eight (200 x 1024 x 1024 8.6, four waves 9.4), two blocks
// where one does not fit the round (500 x 1024 x 1024 10.8, one block 14.0).
struct SmallF32Shape {
  int blocks, waves;
};
SmallF32Shape small_f32_shape(int bits, size_t M, size_t N, size_t K) {
  auto workgroups = [&](size_t blocks) { return row_blocks(M) * ((column_blocks(N) + blocks - 1) / blocks); };
  if (bits == 16) return K <= 512 ? SmallF32Shape{1, 4} : SmallF32Shape{workgroups(1) <= kCUs ? 1 : 2, 8};
  if (K <= 512) {
    if (workgroups(2) < 160) return {1, 4};
    return {workgroups(2) > kCUs && workgroups(3) <= kCUs ? 3 : 2, 4};
  }
  for (int blocks = 1; blocks <= 3; ++blocks)
    if (workgroups(blocks) <= kCUs) return {blocks, 8};
  return {2, 4};
}

// Row blocks per workgroup, waves and fragments per trip of k_gemm_small.  Times behind the quantizer that writes the input.
//   8 bit, K up to 512: four waves, one trip of four fragments each, in any number of workgroups (two row blocks: 2000 x 512 x
//   512 8.2 us, one 7.9).  Up to one workgroup per compute unit eight waves and four fragments (256 x 1024 x 4096 9.15; sixteen
//   waves with eight 9.36).  Beyond, K up to 1024 stays there until three workgroups per unit (384 x 2048 x 1024 8.0; two row
//   blocks on four waves 8.4), longer K takes two row blocks, which read a parameter's fragments once for both: 288 x 1024 x
//   4096 10.6 (one block 11.5), 1000 x 1024 x 2048 11.7 (12.5), on eight waves where that leaves no trip half empty, else on
//   four (1280 x 700 x 1500 10.4, 10.9 on eight).
//   16 bit: two fragments a trip, which leaves registers for two and three workgroups of eight or four waves on a unit: eight
//   waves up to one workgroup per unit (384 x 512 x 512 7.2 us; sixteen waves 7.4; 256 x 1024 x 4096 15.9, four fragments
//   17.4), four beyond (320 x 1024 x 2048 13.0, four fragments and two row blocks 13.6; 1024 x 2048 x 512 10.4 and 11.6; 300 x
//   2048 x 2048 17.6, two row blocks of eight waves 19.2).
struct SmallShape {
  int row_blocks, waves, trip;
};
size_t one_block_workgroups(size_t M, size_t N) { return row_blocks(M) * column_blocks(N); }
SmallShape small_shape(int bits, size_t M, size_t N, size_t K) {
  const size_t wg = one_block_workgroups(M, N), kfrags = PackedDims(8, M, K).kfrags;
  if (bits == 16) return {1, wg <= kCUs ? 8 : 4, 2};
  if (kfrags <= 16) return {1, 4, 4};
  if (wg <= kCUs || (kfrags <= 32 && wg <= 3 * kCUs)) return {1, 8, 4};
  return {2, kfrags > 64 || (kfrags > 32 && (kfrags + 7) / 8 % 4 == 0) ? 8 : 4, 4};
}

}  // namespace

// Split K stays ahead of the tiles up to five workgroups of one row block per compute unit in 8 bit and four in 16.
// 8 bit, quantizer included: 1280 x 1024 x 2048 16.1 us, tiles 17.1; 288 x 4096 x 4096 17.4 and 21.0; 2500 x 512 x 1000 11.2 and
// 12.1; 700 x 1500 x 700 9.4 and 10.2; on the other side 1600 x 1024 x 2048 18.4 and 17.2.  16 bit: 1000 x 1024 x 2048 21.6 and
// 23.9, 2000 x 512 x 512 11.1 and 13.1, 256 x 4096 x 4096 31 and 34; on the other side 640 x 2048 x 2048 24.4 and 23.2.
// Results of few columns have thousands of rows behind those workgroups and less ahead to show for it (3500 x 300 x 2048
// 17.5 and 19.2; 7995 x 100 x 3000 46.9 and 50.4, in 16 bit 62.5 and 66.4; 4955 x 100 x 512 7.9 and 10.5).
bool gemm_small_ahead(int bits, size_t M, size_t N) {
  return one_block_workgroups(M, N) <= (bits == 16 ? 4 : 5) * kCUs;
}

// Workgroups of launch_gemm_small / launch_gemm_small_f32 for a shape = maxima written to GemmArgs::partial.
size_t gemm_small_partials(int bits, size_t M, size_t N, size_t K) {
  const size_t blocks = (size_t)small_shape(bits, M, N, K).row_blocks;
  return (row_blocks(M) + blocks - 1) / blocks * column_blocks(N);
}
size_t gemm_small_f32_partials(int bits, size_t M, size_t N, size_t K) {
  const size_t blocks = (size_t)small_f32_shape(bits, M, N, K).blocks;
  return row_blocks(M) * ((column_blocks(N) + blocks - 1) / blocks);
}

// Split-K product for few rows: packed operands of either width, raw sums or dequantize + bias (+ReLU) (+max|y|).
// Any shape is computed correctly; it is the fast choice when the result is small.
int launch_gemm_small(const GemmArgs& a, Epilogue epi, hipStream_t s) {
  if ((a.bits != 8 && a.bits != 16) || (epi != kEpiRaw && epi != kEpiDequant)) return MQ_ERR_UNSUPPORTED;
  const int dequant = epi == kEpiDequant;
  const SmallShape c = small_shape(a.bits, a.M, a.N, a.K);
  if (a.bits == 16) return c.waves == 8 ? launch_small<16, 1, 8, 2>(a, dequant, s) : launch_small<16, 1, 4, 2>(a, dequant, s);
  if (c.row_blocks == 2) return c.waves == 8 ? launch_small<8, 2, 8, 4>(a, dequant, s) : launch_small<8, 2, 4, 4>(a, dequant, s);
  return c.waves == 4 ? launch_small<8, 1, 4, 4>(a, dequant, s) : launch_small<8, 1, 8, 4>(a, dequant, s);
}

// The 16-bit product whose results are quantized with a given multiplier: packed_out, and its row sums (cleared before) by one
// addition per workgroup and row.
// Ahead of the 128 x 128 tiles up to six workgroups per compute unit.  16-bit block with fixed multipliers, 512 / 2048: 200 rows
// 14.3 us, on tiles 19.2, 700 rows 21.7 and 23.5, 1001 rows (2048 workgroups) 24.1 and 24.9, 1300 30.3 and 27.8; 1024 / 4096: 200
// rows 23.2 and 27.9, 500 rows (2048 workgroups) 33.7 and 32.9; 1000 / 1000: 900 rows 24.0 and 29.6, 1500 rows 31.7 and 33.9;
// 700 / 600: 2500 rows (1501 workgroups) 29.0 and 31.0, 3500 rows 32.8 and 32.6; 300 / 3333: 500 rows (1680) 22.0 and 21.8.
bool gemm_small_requant_ahead(size_t M, size_t N) { return one_block_workgroups(M, N) <= 6 * kCUs; }
int launch_gemm_small_requant_i16(const GemmArgs& a, hipStream_t s) {
  return one_block_workgroups(a.M, a.N) <= kCUs ? launch_small<16, 1, 8, 2, true>(a, 1, s) : launch_small<16, 1, 4, 2, true>(a, 1, s);
}

// Product + bias (+ReLU) -> max|y| -> quant_int(y) for few rows, the smallest workgroups that fit one round of the grid;
// MQ_ERR_UNSUPPORTED where none does.
int launch_gemm_small_requant_agree(const GemmArgs& a, hipStream_t s) {
  int rc = launch_agree<1, 1>(a, s);
  if (rc == MQ_ERR_UNSUPPORTED) rc = launch_agree<2, 1>(a, s);
  if (rc == MQ_ERR_UNSUPPORTED) rc = launch_agree<4, 1>(a, s);
  return rc != MQ_ERR_UNSUPPORTED ? rc : launch_agree<4, 2>(a, s);
}

// Whether quantizing inside the product pays: few rows, K short enough that re-reading the fp32 rows once
// per column tile stays below the cost of a separate quantizing launch.  K above 512 in more than two rounds is the separate
// quantizer's: 300 x 4096 x 1024 13.0 us in three launches where two take 14.7, 512 rows 13.3 and 18.0.
// 16 bit, abs-max, three launches and two: K up to 512 by two workgroups per compute unit (384 x 512 x 512 8.8 and 7.2 us, 1000 x
// 512 x 512 10.7 and 9.6; 640 workgroups, 300 x 2048 x 512, 11.3 and 11.5; 1008, 2000 x 512 x 512, 13.4 and 14.6); K up to 1024 in
// one round of up to two column blocks (500 x 1024 x 1024 12.6 and 10.8; 480 of them, 300 x 3072 x 1024, 16.0 and 16.1); K up to
// 2048 in one round of one (300 x 512 x 2048 12.8 and 11.5; two blocks, 600 x 512 x 2048, with the multiplier given 12.6 and
// 12.7).  K = 4096 with the multiplier given: 12.7 and 14.0.  max|y| in one word draws no line of its own: it adds 0.2 us with 512
// workgroups as with 96 (1000 x 512 x 512 9.3 and 9.5 us, 10.7 and 11.0 in three launches; 500 x 1024 x 256 7.8 and 8.1, 9.8 and 13.2).
bool gemm_small_f32_supported(int bits, size_t M, size_t N, size_t K) {
  if (bits == 16) {
    if (M < 1 || N < 1 || K < 32 || K % 32 != 0 || K > 2048) return false;
    const size_t blocks = K > 512 && K <= 1024 ? (column_blocks(N) + 1) / 2 : column_blocks(N);
    return row_blocks(M) * blocks <= (K <= 512 ? 2 * kCUs : kCUs);
  }
  return M >= 1 && M <= 512 && N >= 1 && K >= 32 && K % 32 == 0 &&
         (K <= 512 || (K <= 1024 && (M <= 32 || row_blocks(M) * ((column_blocks(N) + 1) / 2) <= 2 * kCUs)));
}

// quant_int(A) + dot'_int + dequantize + bias (+ReLU) (+max|y|) in one launch; see k_gemm_small_f32.
// scale: the multiplier (npartial == 0) or npartial partial maxima of |A|.
namespace {
int launch_small_f32_any(SmallF32Params p, const GemmArgs& a, hipStream_t s) {
  if (!gemm_small_f32_supported(a.bits, a.M, a.N, a.K)) return MQ_ERR_UNSUPPORTED;
  p.packedW = static_cast<const uint8_t*>(a.packedW);
  p.M = (unsigned)a.M; p.N = (unsigned)a.N; p.K = (unsigned)a.K;
  p.sW = a.sW; p.bias = a.bias; p.relu = a.relu; p.Y = a.Y; p.out_amax = a.out_amax; p.amax_slots = a.amax_slots;
  p.partial_out = a.partial;
  const SmallF32Shape shape = small_f32_shape(a.bits, a.M, a.N, a.K);
  if (a.bits == 16) {
    if (shape.waves == 4) return launch_small_f32<16, 1, 4>(p, s);
    return shape.blocks == 1 ? launch_small_f32<16, 1, 8>(p, s) : launch_small_f32<16, 2, 8>(p, s);
  }
  if (shape.waves == 4) {
    if (shape.blocks == 1) return launch_small_f32<8, 1, 4>(p, s);
    return shape.blocks == 2 ? launch_small_f32<8, 2, 4>(p, s) : launch_small_f32<8, 3, 4>(p, s);
  }
  if (shape.blocks == 1) return launch_small_f32<8, 1, 8>(p, s);
  return shape.blocks == 2 ? launch_small_f32<8, 2, 8>(p, s) : launch_small_f32<8, 3, 8>(p, s);
}
}  // namespace

int launch_gemm_small_f32(const float* A, const float* scale, unsigned npartial, float* scale_out, const GemmArgs& a,
                          hipStream_t s) {
  SmallF32Params p{};
  p.A = A; p.scale = scale; p.npartial = npartial; p.scale_out = scale_out;
  return launch_small_f32_any(p, a, s);
}

int launch_gemm_small_f32_pair(const float* A1, size_t K1, const float* part1, unsigned n1, const float* A2,
                               const float* part2, unsigned n2, float* scale_out, const GemmArgs& a, hipStream_t s) {
  if (K1 == 0 || K1 >= a.K || K1 % 4 != 0 || n1 == 0 || n2 == 0) return MQ_ERR_UNSUPPORTED;
  SmallF32Params p{};
  p.A = A1; p.A2 = A2; p.K1 = (unsigned)K1;
  p.scale = part1; p.npartial = n1; p.scale2 = part2; p.npartial2 = n2; p.scale_out = scale_out;
  return launch_small_f32_any(p, a, s);
}

}  // namespace mq
