// Greedy output layer of a decode step (arxiv 1805.12096, Section 2.3: with beam
// size 1 no softmax is evaluated, the word with the highest activation wins;
// Section 2.1: the output matrix is the tied 36 000-entry embedding).
//
// Shape of the problem: a few hundred sentences (M) against tens of thousands
// of vocabulary rows (N) at K = model size.  Per step the whole embedding has to
// stream through the chip once (N * K bytes) while the M x N logits never need
// to exist.  So:
//   * work is cut into units of 16 vocabulary rows (all of K), dealt round-robin
//     to one workgroup per compute unit; 36 000 rows give 2250 units, 8.8 per CU;
//   * the matrix instruction is v_mfma_i32_16x16x64_i8 with the embedding as
//     operand `a` and the hidden states as operand `b`: lane l then holds four
//     candidate words for ONE sentence (l % 16), so the running maxima are
//     plain per-lane registers and nothing crosses lanes until the very end;
//   * the quantized hidden states (M x K, a few 100 KB) are loaded once per
//     workgroup into REGISTERS as operand fragments, split over the eight waves
//     by 16-sentence tile; more sentences than that go in chunks (of one launch,
//     see chunk_of) that share the compute units;
//   * the packed embedding streams through LDS with direct-to-LDS loads: each
//     load instruction gathers, for one 64-element K group, the 16 rows of the
//     unit out of two 32-row fragments, so that LDS receives exactly the
//     operand image (lane l at byte 16 l); many stages are in flight;
//   * sums of 8-bit products over K <= 512 stay below 2^23, so (sum << 8 |
//     255 - stage) is a 32-bit key whose integer maximum is the arg-max with
//     the earliest stage winning ties: two VALU operations per candidate
//     (K <= 1024: below 2^24, one bit less for the stage);
//   * every workgroup writes one 64-bit (sum, index) key per sentence, its own
//     run of consecutive keys; a second small kernel reduces them and decodes.
//     No atomics, no initialisation.  (Folding that reduction into this kernel
//     was tried -- 64-bit atomic maxima per sentence with the last workgroup out
//     decoding -- and took three times as long: the 76 800 atomics serialise on
//     the few cache lines that hold the maxima.)
// 64-bit keys order by sum first and by smaller index second:
//   key = (sum ^ 0x80000000) << 32 | (0xFFFFFFFF - n);  0 means "no candidate".
#include <mutex>
#include <type_traits>

#include "mq_gemm_common.h"

namespace mq {

namespace {

constexpr int kWaves = 8;             // two per SIMD: one wave's waits hide behind the other's MFMAs
constexpr int kKG = 8;                // 64-element K groups per unit (K <= 512)
constexpr int kWideKG = 16;           // the same for K <= 1024
constexpr int kMaxTPW = 3;            // 16-sentence tiles per wave that fit the registers at K <= 512
constexpr int kWideTPW = 2;           // and at K <= 1024
constexpr int kBeamTPW = 2;           // and in beam search
constexpr int stages_of(int kg) { return kg == kKG ? 10 : 18; }            // ring slots of 8 KB: all but two in flight
// key of a candidate: sum << shift | (mask - stage)
constexpr int shift_of(int kg) { return kg == kKG ? 8 : 7; }
constexpr unsigned max_units_of(int kg) { return (1u << shift_of(kg)) - 1; }  // units per workgroup
constexpr int kMaxBlocks = 1024;      // upper bound on workgroups (columns of the partials array)

__device__ __forceinline__ void wait_vmcnt_n(int n) {
  switch (n) {
#define MQ_CASE(N) case N: __builtin_amdgcn_s_waitcnt(((N) & 0xF) | (((N) >> 4) << 14) | 0x0F70); break;
    MQ_CASE(0) MQ_CASE(1) MQ_CASE(2) MQ_CASE(3) MQ_CASE(4) MQ_CASE(5) MQ_CASE(6) MQ_CASE(7) MQ_CASE(8) MQ_CASE(9)
    MQ_CASE(10) MQ_CASE(11) MQ_CASE(12) MQ_CASE(13) MQ_CASE(14) MQ_CASE(15) MQ_CASE(16)
#undef MQ_CASE
    default: __builtin_amdgcn_s_waitcnt(0x0F70); break;
  }
}

struct ArgmaxParams {        // what the first loads' addresses need in the first 64 bytes
  const uint8_t* packedA;   // hidden states, packed 8 bit [M x K] (or, ROWM, plain rows of K bytes)
  const uint8_t* packedW;   // embedding, packed 8 bit [N x K]
  unsigned M, N, K;
  unsigned L;                    // candidates: shortlist length, or N
  // `columns` workgroups share the vocabulary.  More rows than one workgroup's registers hold: they do for every chunk of
  // chunk_rows rows (a multiple of 16) out of M; everything else describes all rows of the launch.
  unsigned columns;
  unsigned units_each, units_more;      // units of 16 candidates: every column has units_each, the first units_more one more
  unsigned chunk_rows;
  // which column and chunk a workgroup is (see chunk_of): side_by_side is 0 or all ones, inner the columns or the chunks and
  // by_inner = ceil(2^32 / inner) (as 32 bits 0 for inner = 1, which is one workgroup alone: all come out 0)
  unsigned workgroups, side_by_side, inner, by_inner;
  const int32_t* shortlist;      // optional: vocabulary rows to score, ascending; NULL = all N rows
  unsigned long long* partial;   // BEAM == 1: [columns][Mpad], Mpad = M rounded up to 16; beam search: [M][columns][BEAM]
  // beam search (BEAM > 1): partial holds [M][columns][BEAM] keys, norm [M][columns] (max, sum) pairs of
  // the softmax normaliser in base 2, u2 = log2(e) / (sA sW) is formed in the kernel
  float2* norm;
  const float* sA;
  const float* sW;
};

// Column (of the vocabulary) and chunk (of the rows) of this workgroup.  The chunks of a column read the same units and belong on
// one XCD, whose L2 then takes the units in once for all of them.  Column after column (chunk y of column x on XCD (y columns +
// x) % 8) does that where the columns are a multiple of eight (two and four chunks); there it stays (500 rows greedy 13.2 us, 14.0 in the order
// below).  Elsewhere every chunk took the units from the last-level cache: 1200 rows, k = 4 (five chunks of 51 columns) 41.3 ->
// 38.8 us, 1000 rows greedy (three of 85) 22.4 -> 20.7, 600 rows of width 1024 31.2 -> 30.0.
// (One row of workgroups: column + columns chunk, or, with `side_by_side`, chunk + chunks column after the XCD remap.  All by
// arithmetic: a branch, or what the compiler makes one of, splits the loads of the arguments.)
__device__ __forceinline__ void chunk_of(const ArgmaxParams& p, unsigned& column, unsigned& chunk) {
  const unsigned id = blockIdx.x, t = id ^ ((xcd_remap(id, p.workgroups) ^ id) & p.side_by_side);
  const unsigned q = (unsigned)(((unsigned long long)t * p.by_inner) >> 32), swap = (q ^ (t - q * p.inner)) & p.side_by_side;
  column = (t - q * p.inner) ^ swap;
  chunk = q ^ swap;
}

// What lane l feeds to the 16x16x64 MFMA for rows 16 u .. 16 u + 15 of a packed
// 8-bit operand and K group g (64 elements): K quarter l / 16 of the group lives
// in fragment 2 g + l / 32, half (l / 16) % 2, row slot (u % 2) 16 + l % 16.
// The offset splits into a per-lane constant and a wave-uniform part.
__device__ __forceinline__ unsigned operand16_lane_offset(int lane) {
  return (unsigned)(lane / 32) * kFragBytes + (unsigned)(((lane / 16) % 2) * 32 + lane % 16) * 16;
}
__device__ __forceinline__ size_t operand16_uniform_offset(const PackedDims& d, size_t unit, unsigned g) {
  return d.frag_offset(unit / 2, 2 * g) + (unit % 2) * 256;
}

// top = the BEAM largest of two descending lists, descending: the pairwise maxima of one list with the reversed other
// are the largest BEAM in bitonic order, which half-cleaners sort (a third of the comparisons of inserting one by one).
template <int BEAM>
__device__ __forceinline__ void merge_sorted(unsigned long long (&top)[BEAM], const unsigned long long (&other)[BEAM]) {
  static_assert(BEAM == 2 || BEAM == 4, "list lengths in use");
#pragma unroll
  for (int j = 0; j < BEAM; ++j) top[j] = top[j] > other[BEAM - 1 - j] ? top[j] : other[BEAM - 1 - j];
#pragma unroll
  for (int half = BEAM / 2; half >= 1; half /= 2)
#pragma unroll
    for (int j = 0; j < BEAM; ++j)
      if ((j & half) == 0) {
        const unsigned long long a = top[j], b = top[j + half];
        top[j] = a > b ? a : b;
        top[j + half] = a > b ? b : a;
      }
}

// TPW: 16-sentence tiles per wave (8 * TPW * 16 >= M).
// GATHER: candidates are the rows listed in p.shortlist (the lexical shortlist of Section 4.1: the
// output product restricted to a subset of the vocabulary).  A unit is then 16 consecutive shortlist
// positions; since every lane of a direct-to-LDS load supplies its own address, gathering the 16
// rows costs nothing extra.  Indices are candidate positions; the reduce kernel maps them back.

// BEAM > 1 (beam search, Table 2's b = 2 and b = 4 rows): every accumulator register keeps its BEAM best
// keys instead of one, and every sentence tile keeps a running (reference, sum) of 2^(logit log2 e - reference) so
// that the k best words come with normalised log-probabilities.  This is bound by vector instructions (1200 rows
// x 36 000 words are 675 000 wave-wide candidates), so a candidate costs as few as possible:
//   * sorted insertion is one maximum and BEAM - 1 median-of-three instructions (the new second of a >= b with k
//     arriving is med3(a, b, k), and so on down the list) instead of BEAM maximum / minimum pairs;
//   * the reference of the sum moves only when a logit exceeds it by more than kNormSlack (a wave-uniform branch that
//     is hardly ever taken after the first unit), so a candidate is one conversion, one multiply-add, one exponential
//     and one addition, without rescaling the sum every four candidates;
//   * every candidate of the stage before is worked off between two groups of matrix instructions of its own.
// 1200 rows, k = 4, 36 000 words, with the quantizer and the reduce kernel: 84.7 us with maximum / minimum pairs, a
// rescaled sum and every chunk of 256 rows spread over all compute units; 52.3 us with the above and the chunks sharing
// them (launch_topk_stream); 48.3 us with sorted lists merged instead of inserted one by one at the end (42 with what follows below).  240 rows:
// 29.1 -> 26.2 us.  A unit then was 0.27 us of LDS reads and waits, 0.13 of matrix instructions and 0.21 of these; the refill below
// took 6 us off the 45 units of a workgroup (1200 rows, k = 4, this kernel in the trace 42.4 -> 36.3 us).
// Greedy, 36 000 words, kernels of a captured step (quantizer included): 300 sentences of width 512 17.6 -> 16.9 us (the
// 19th of 24 tile slots' operands no longer fetched for nothing, reduce kernel), 600 sentences against 50 000 words 34.8
// -> 24.9 us (chunks that share the compute units instead of one launch pair after the other), 300 sentences of width
// 1024 41.9 -> 31.3 us (the tiled kernel's arg-max epilogue took 32.7 us of them, this one 20).
// Stages that refill the ring (more than nine units to a workgroup; captured calls, quantizer not counted): addresses and slots
// by addition, and the updates held between the matrix instructions (see `refill` and `here`): 1200 rows, k = 4 43.9 -> 41.3 us,
// k = 2 38.8 -> 35.5, 300 rows of width 1024 22.4 -> 20.7; chunks that share XCDs (chunk_of) 41.3 -> 38.8 and 35.5 -> 32.5; the
// tag as a scalar, and no division in front of the first load, 38.8 -> 37.9, 32.5 -> 31.8, 20.6 -> 19.7.
// KG: 64-element K groups held (8: K <= 512, 16: K <= 1024).  ROWM: the hidden states are plain rows (K a multiple of
// 16) instead of packed ones; only the addresses of the operand loads differ.
template <int TPW, bool GATHER, int BEAM = 1, int KG = kKG, bool ROWM = false>
__global__ __launch_bounds__(kWaves * 64) void k_argmax_stream(const ArgmaxParams p) {
  constexpr int S = stages_of(KG);
  constexpr int NH = KG / kKG;                        // stages per unit: 512 elements of K each
  constexpr int STAGE = kKG * kFragBytes;
  constexpr int SHIFT = shift_of(KG), TAGS = (1 << SHIFT) - 1;
  static_assert(kKG == kWaves, "one direct-to-LDS load per wave and stage");
  static_assert(KG % kKG == 0 && (NH == 1 || (NH == 2 && S % 2 == 0)), "stages of a unit");
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];

  const int lane = threadIdx.x % 64;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  unsigned column, chunk;
  chunk_of(p, column, chunk);
  const unsigned row0 = chunk * p.chunk_rows;         // this workgroup's rows: row0 .. row0 + rows - 1
  const unsigned rows = p.M - row0 < p.chunk_rows ? p.M - row0 : p.chunk_rows;
  const PackedDims dA(8, p.M, p.K), dW(8, p.N, p.K);
  const unsigned kgroups = (unsigned)(dW.kfrags / 2);          // real K groups (<= KG)
  const unsigned first = column, stride = p.columns;
  const unsigned nlocal = p.units_each + (first < p.units_more ? 1u : 0u);      // at most as many columns as units: at least 1
  const unsigned lane_off = operand16_lane_offset(lane);

  // stage s of the pipeline = 512 elements of K (part s % NH) of this workgroup's (s / NH)-th unit; wave w copies the
  // part's K group w (K shorter than 64 KG: a real group is copied again and its products are zeroed through `hid`)
  const uint8_t* src_lane = p.packedW + lane_off;
  // GATHER: this workgroup's candidate rows, 16 per stage, are fetched into LDS once, before any
  // direct-to-LDS load is in flight (later ordinary loads would have to drain the pipeline)
  int32_t* rows_lds = reinterpret_cast<int32_t*>(smem + S * STAGE + kWaves * kFragBytes);
  if (GATHER) {
    for (unsigned i = threadIdx.x; i < nlocal * 16; i += kWaves * 64) {
      const unsigned pos = (first + (i / 16) * stride) * 16 + i % 16;
      // positions past the end are masked later; an id outside [0, N) reads the nearest row instead of memory
      // outside the embedding (the token reported for it is the id as listed)
      const int id = pos < p.L ? p.shortlist[pos] : p.shortlist[0];
      rows_lds[i] = min(max(id, 0), (int)p.N - 1);
    }
    __syncthreads();
  }
  // A value that has to be there at this point of the program.
  auto here = [](auto& x) { asm volatile("" : "+v"(x)); };
  // One load per wave for stage s.  Past the workgroup's last unit the same instruction fetches unit 0 again into a
  // per-wave slot behind the stages that nobody reads: every stage then issues exactly one load, the number of loads
  // in flight at a given point is a constant, and the waits need neither a branch nor a table.  Needs nlocal > 0.
  auto issue = [&](unsigned s_any) {
    const bool real = s_any < nlocal * NH;
    const unsigned s = real ? s_any : 0;
    const unsigned unit = s / NH, g = (s % NH) * kKG + wave, my_group = g < kgroups ? g : kgroups - 1;
    uint8_t* dst = real ? smem + (s % S) * STAGE + wave * kFragBytes : smem + S * STAGE + wave * kFragBytes;
    const uint8_t* src;
    if (GATHER) {
      const unsigned r = (unsigned)rows_lds[unit * 16 + lane % 16];
      src = p.packedW + dW.frag_offset(r / 32, 2 * my_group + lane / 32) +
            (size_t)((r % 32) + 32 * ((lane / 16) % 2)) * 16;
    } else {
      src = src_lane + operand16_uniform_offset(dW, (size_t)first + (size_t)unit * stride, my_group);
    }
    __builtin_amdgcn_global_load_lds(
        (const __attribute__((address_space(1))) void*)src, (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
  };
  // The same for the stages that refill freed slots, one unit after the other: the unit's row, its slot and the address advance by
  // additions (a unit's offset is below 2^32: 255 x 256 units of 16 rows, 127 x 256 for K > 512).  Divisions and 64-bit products
  // for every load were 40 scalar instructions of a stage that each wave issues in line with its matrix instructions.
  unsigned fill_index = 0, fill_unit = 0, fill_slot = 0;
  const unsigned row_pitch = (unsigned)dW.kfrags * kFragBytes;
  unsigned fill_group[NH];
#pragma unroll
  for (int h = 0; h < NH; ++h) fill_group[h] = min((unsigned)(h * kKG) + wave, kgroups - 1) * (2 * kFragBytes);
  auto start_refills = [&](unsigned index) {
    fill_index = index;
    fill_unit = first + index * stride;
    fill_slot = (index * NH) % S * STAGE;
  };
  auto refill = [&]() {
    const bool real = fill_index < nlocal;
    const unsigned dst = real ? fill_slot + wave * kFragBytes : S * STAGE + wave * kFragBytes;
    if (GATHER) {
      issue(fill_index);                               // (NH == 1)
    } else {
      const unsigned unit = real ? fill_unit : first, at = (unit / 2) * row_pitch + (unit % 2) * 256;
#pragma unroll
      for (int h = 0; h < NH; ++h)
        __builtin_amdgcn_global_load_lds(
            (const __attribute__((address_space(1))) void*)(p.packedW + (at + fill_group[h]) + lane_off),
            (__attribute__((address_space(3))) void*)(smem + (dst + (real ? h * STAGE : 0))), 16, 0, 0);
    }
    ++fill_index;
    fill_unit += stride;
    fill_slot += NH * STAGE;
    if (fill_slot == S * STAGE) fill_slot = 0;
  };
  static_assert(!GATHER || NH == 1, "gathered units are one stage");
  // The first two stages go out first (their memory latency is the longest wait of the kernel), then the
  // hidden-state operands of this wave's sentence tiles (tile t = wave + 8 i covers sentences 16 t ..
  // 16 t + 15; they come from L2, every workgroup reads the same ones), then the remaining stages.  The
  // memory counter retires loads in order, so waiting for "all but the newest n" later covers stages 0
  // and 1 and the operands while the newer stages are still on their way.
  constexpr int kEarly = 2;
  constexpr int kAhead = NH == 1 ? S - 1 : S - 2;     // stages issued before the first one is multiplied
#pragma unroll
  for (int s = 0; s < kEarly; ++s) issue(s);
  // 16-sentence tiles this wave owns
  const unsigned tiles_avail = (rows + 15) / 16;
  const int ntl = (unsigned)wave < tiles_avail ? (int)((tiles_avail - 1 - wave) / kWaves) + 1 : 0;

  // running maxima, one per accumulator register: (sum << SHIFT) | (TAGS - stage).  Real sums exceed
  // -2^(31 - SHIFT), so a key whose sum field is that means "no candidate yet".
  constexpr int kNone = (int)0x80000000;
  constexpr int kNoSum = -(1 << (31 - SHIFT));
  int best[TPW][4];
  int more_best[BEAM > 1 ? TPW : 1][4][BEAM > 1 ? BEAM - 1 : 1];     // places 2 .. BEAM of each register's list
  float norm_ref[TPW], norm_sum[TPW], norm_expo[TPW][4];               // softmax normaliser, base 2 (BEAM > 1)
  float u2 = 0.f;
  if constexpr (BEAM > 1) u2 = __fmul_rn(__fdiv_rn(1.0f, __fmul_rn(*p.sA, *p.sW)), 1.44269504088896340736f);
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    norm_ref[i] = -INFINITY;
    norm_sum[i] = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      best[i][r] = kNone;
      if constexpr (BEAM > 1)
#pragma unroll
        for (int j = 0; j < BEAM - 1; ++j) more_best[i][r][j] = kNone;
    }
  }
  v4i acc0[TPW], acc1[TPW];             // sums of even and odd units
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    acc0[i] = v4i{kNoSum, kNoSum, kNoSum, kNoSum};
    acc1[i] = v4i{kNoSum, kNoSum, kNoSum, kNoSum};           // "none" for unit 0's update
  }
  auto med3 = [](int x, int y, int z) -> int { return max(min(x, y), min(max(x, y), z)); };    // v_med3_i32
  // one candidate's key into the sorted list of its register
  auto beam_insert = [&](int i, int r, int key) {
    if constexpr (BEAM > 1) {
#pragma unroll
      for (int j = BEAM - 2; j > 0; --j) more_best[i][r][j] = med3(more_best[i][r][j - 1], more_best[i][r][j], key);
      more_best[i][r][0] = med3(best[i][r], more_best[i][r][0], key);
      best[i][r] = max(best[i][r], key);
    }
  };
  // exponents (relative to the reference) of one sentence tile's four new sums; moves the reference first, in the
  // lanes where one of them exceeds it by more than kNormSlack (and at the first unit, whose reference is -inf).
  // valid: bit r clear leaves candidate r out (padding past the last candidate).
  constexpr float kNormSlack = 16.0f;
  auto beam_exponents = [&](int i, const v4i& sums, unsigned valid, float (&t)[4]) {
    float c[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      c[r] = (float)sums[r];
      t[r] = (valid >> r) & 1u ? fmaf(c[r], u2, -norm_ref[i]) : -INFINITY;
    }
    float top = fmaxf(fmaxf(t[0], t[1]), fmaxf(t[2], t[3]));
    if (__any(top > kNormSlack)) {
      if (top > kNormSlack) {
        float ref = -INFINITY;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if ((valid >> r) & 1u) ref = fmaxf(ref, __fmul_rn(c[r], u2));
        norm_sum[i] *= __builtin_amdgcn_exp2f(norm_ref[i] - ref);      // 0 * 2^-inf at the first unit
        norm_ref[i] = ref;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if ((valid >> r) & 1u) t[r] = fmaf(c[r], u2, -ref);
      }
    }
  };

  // Before stage s is multiplied, stages s and s + 1 must have landed (s + 1 is read from LDS into
  // registers while s is multiplied): of the loads issued so far the oldest s + 2 are needed, `newest` may be
  // outstanding.  With a load in every stage S - 1 + s have been issued (newest = S - 3); without, S - 1
  // (newest = S - 3 - s).
  // This wave's LDS reads of stage s have returned, too: the compiler would otherwise wait for ALL outstanding reads,
  // the first ones of stage s + 1 included, before the stage's first matrix instructions.
  // With two stages per unit the waves meet once per unit: its first stage waits for stages s to s + 2 out of the s + S - 2
  // issued (newest = S - 5) and refills the two slots that everybody is past, its second one only waits for this wave's
  // own LDS reads.  300 sentences of width 1024, 36 000 words: 31.2 -> 30.3 us for the whole output layer.
  auto land = [&](int newest) {
    wait_vmcnt_n(newest);
    __builtin_amdgcn_s_waitcnt(0xC07F);                // lgkmcnt(0)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  // Everything from the operand loads to the last stage, for a wave with NT sentence tiles.  The operand loads are
  // written as instructions so that the waiting is ours: the compiler would wait for ALL outstanding loads, the whole
  // pipeline included, at the first use.  It takes their results for there at once, so between the loads and the wait
  // there must be nothing that makes it move them: no branch that joins one value of an operand with another (which is
  // why the number of tiles is a constant here and not a condition around the loads).
  using T = std::true_type;
  using F = std::false_type;
  using P0 = std::integral_constant<int, 0>;
  using P1 = std::integral_constant<int, 1>;
  auto body = [&](auto nt_tag) {
    constexpr int NT = decltype(nt_tag)::value;
    v4i hid[NT > 0 ? NT : 1][KG];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      unsigned t = (unsigned)wave + kWaves * i;
      if (t >= tiles_avail) t = tiles_avail - 1;     // a chunk of few rows: a tile again, never written out
      t += row0 / 16;
      // one 32-bit lane offset per tile and a wave-uniform base per K group (a launch's rows are below 2^32 bytes)
      unsigned voff = lane_off, voff_last = lane_off;
      if constexpr (ROWM) {
        // this lane's sentence (past the end: the last one again), 16 bytes at K quarter lane / 16; a quarter past the
        // end of the row, which only the last group can have, reads quarter 0: it meets the embedding's zero padding
        const unsigned m = t * 16 + lane % 16, quarter = (unsigned)(lane / 16) * 16;
        voff_last = (m < p.M ? m : p.M - 1) * p.K;
        voff = voff_last + quarter;
        voff_last = (kgroups - 1) * 64 + quarter < p.K ? voff : voff_last;
      }
#pragma unroll
      for (int g = 0; g < KG; ++g) {
        const unsigned gr = (unsigned)g < kgroups ? (unsigned)g : 0u;         // groups past the end are zeroed below
        const uint8_t* base = p.packedA + (ROWM ? (size_t)gr * 64 : operand16_uniform_offset(dA, t, gr));
        const unsigned off = ROWM && gr == kgroups - 1 ? voff_last : voff;
        asm volatile("global_load_dwordx4 %0, %1, %2" : "=&v"(hid[i][g]) : "v"(off), "s"(base) : "memory");
      }
    }
#pragma unroll
    for (int s = kEarly; s < kAhead; ++s) issue(s);
    // stage 0 has to be in registers before the loop, and so have the operands: everything but the
    // stages issued after the operands may still be outstanding
    v4i e0[kKG], e1[kKG];                   // two stages per trip, so that the buffers swap roles without copies
    wait_vmcnt_n(kAhead - kEarly);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int g = 0; g < kKG; ++g) e0[g] = as_v4i(*reinterpret_cast<const u4*>(smem + lane * 16 + g * kFragBytes));
    // the operands are older than every stage, so they are there now; K groups past the end of K are zeroed
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int g = 0; g < KG; ++g) {
        asm volatile("" : "+v"(hid[i][g]));
        if ((unsigned)g >= kgroups) hid[i][g] = v4i{0, 0, 0, 0};
      }

    // One stage: 512 elements of K of a unit (in `e`) against this wave's NT sentence tiles into `cur`, while the
    // maxima are updated from `prev` (the sums of the unit before) and the next stage is read from LDS into `enext`.
    // The update's VALU work is cut into slices that sit between the MFMA groups, so it runs while the matrix pipeline
    // is busy instead of after it; the scheduling fences keep that order inside a block, and `here` keeps the compiler from
    // moving the updates of a trip's second stage behind the branch that follows it, where the waves of a SIMD, which are in
    // step, would all come to them with their matrix instructions done.
    // refill_tag: the freed slot takes a new load; first_tag: unit 0, which has no unit before it; part_tag: s % NH;
    // unit: this workgroup's; next_slot: where the next stage is.
    auto stage = [&](auto refill_tag, auto first_tag, auto part_tag, int newest, unsigned unit, unsigned next_slot, v4i (&cur)[TPW],
                     const v4i (&prev)[TPW], const v4i (&e)[kKG], v4i (&enext)[kKG]) {
      constexpr int PART = decltype(part_tag)::value;
      constexpr bool FIRST = decltype(first_tag)::value;
      if constexpr (PART == 0) {
        land(newest);
        // everybody is past stage s - 1 (and has its copy of stage s in registers), so slot s - 1 can be refilled
        if constexpr (decltype(refill_tag)::value) refill();
      } else {
        __builtin_amdgcn_s_waitcnt(0xC07F);              // lgkmcnt(0), see land
        asm volatile("" ::: "memory");
      }
      // the next stage's LDS reads go two at a time between the first MFMA groups: eight in a row would fill the LDS
      // queue (all eight waves read at the same time) and hold this wave's MFMAs back behind them, and they should be
      // back before the next barrier (after the last stage they read a finished slot again and the result is unused)
      const uint8_t* nx = smem + next_slot + lane * 16;
      // TAGS - (unit - 1), in a scalar register (masked together with each sum's shift it was an instruction more a key); unused
      // garbage for unit 0 (prev holds "none")
      int prev_tag = (TAGS + 1 - (int)unit) & TAGS;
      if constexpr (decltype(refill_tag)::value || PART != 0) asm("" : "+s"(prev_tag));
      constexpr int ITEMS = NT * 4, PER = (ITEMS + KG - 1) / KG;
      const v4i zero = {0, 0, 0, 0};
#pragma unroll
      for (int g = 0; g < kKG; ++g) {
        if (g < kKG / 2) {
          enext[2 * g] = as_v4i(*reinterpret_cast<const u4*>(nx + (2 * g) * kFragBytes));
          enext[2 * g + 1] = as_v4i(*reinterpret_cast<const u4*>(nx + (2 * g + 1) * kFragBytes));
        }
#pragma unroll
        for (int i = 0; i < NT; ++i)
          cur[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(e[g], hid[i][PART * kKG + g], PART == 0 && g == 0 ? zero : cur[i], 0, 0, 0);
        constexpr int J0 = PART * kKG;
        if constexpr (BEAM == 1) {
#pragma unroll
          for (int j = (J0 + g) * PER; j < (J0 + g + 1) * PER && j < ITEMS; ++j) {
            best[j / 4][j % 4] = max(best[j / 4][j % 4], (prev[j / 4][j % 4] << SHIFT) | prev_tag);
            if constexpr (decltype(refill_tag)::value || PART != 0) here(best[j / 4][j % 4]);
          }
        } else if constexpr (!FIRST) {
          // exponents of the unit before (norm_expo) are formed in the first group
          if (g == 0) {
#pragma unroll
            for (int i = 0; i < NT; ++i) beam_exponents(i, prev[i], 15u, norm_expo[i]);
          }
#pragma unroll
          for (int j = (J0 + g) * PER; j < (J0 + g + 1) * PER && j < ITEMS; ++j) {
            beam_insert(j / 4, j % 4, (prev[j / 4][j % 4] << SHIFT) | prev_tag);
            norm_sum[j / 4] += __builtin_amdgcn_exp2f(norm_expo[j / 4][j % 4]);
            here(best[j / 4][j % 4]);
#pragma unroll
            for (int b = 0; b < BEAM - 1; ++b) here(more_best[j / 4][j % 4][b]);
            here(norm_sum[j / 4]);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };

    if (NH == 1 && nlocal <= (unsigned)(S - 1)) {
      // The usual case (36 000 rows over 256 workgroups are 9 units each): the prologue has issued everything.
      // Unrolled, so that each stage waits with its own constant and nothing is issued inside the loop.
#pragma unroll
      for (int s = 0; s < S - 1; ++s) {
        if ((unsigned)s >= nlocal) break;
        const int newest = S - 3 - s > 0 ? S - 3 - s : 0;
        const unsigned slot = (unsigned)((s + 1) % S * STAGE);
        if (s == 0) stage(F{}, T{}, P0{}, newest, 0u, slot, acc0, acc1, e0, e1);
        else if (s % 2 == 0) stage(F{}, F{}, P0{}, newest, (unsigned)s, slot, acc0, acc1, e0, e1);
        else stage(F{}, F{}, P0{}, newest, (unsigned)s, slot, acc1, acc0, e1, e0);
      }
    } else {
      start_refills(NH == 1 ? S - 1 : (S - 2) / NH);
      unsigned slot = 0;
      auto next = [&]() {
        slot += STAGE;
        if (slot == S * STAGE) slot = 0;
        return slot;
      };
      if constexpr (NH == 1) {
        stage(T{}, T{}, P0{}, S - 3, 0u, next(), acc0, acc1, e0, e1);
        for (unsigned s = 1; s < nlocal; s += 2) {
          stage(T{}, F{}, P0{}, S - 3, s, next(), acc1, acc0, e1, e0);
          if (s + 1 < nlocal) stage(T{}, F{}, P0{}, S - 3, s + 1, next(), acc0, acc1, e0, e1);
        }
      } else {
        for (unsigned n = 0; n < nlocal; n += 2) {
          stage(T{}, F{}, P0{}, S - 5, n, next(), acc0, acc1, e0, e1);
          stage(T{}, F{}, P1{}, 0, n, next(), acc0, acc1, e1, e0);
          if (n + 1 < nlocal) {
            stage(T{}, F{}, P0{}, S - 5, n + 1, next(), acc1, acc0, e0, e1);
            stage(T{}, F{}, P1{}, 0, n + 1, next(), acc1, acc0, e1, e0);
          }
        }
      }
    }
    wait_vmcnt_n(0);      // the refills past the last unit are still landing in their slots
  };
  if (ntl == TPW) body(std::integral_constant<int, TPW>{});
  else body(std::integral_constant<int, TPW - 1>{});
  // the last stage's sums are still pending; only a workgroup's last unit can reach past N, where
  // the rows are padding and must not compete (needs at least two workgroups, which the launcher
  // guarantees whenever there is more than one unit)
  {
    const unsigned sl = nlocal - 1;
    const unsigned unit0 = (first + sl * stride) * 16 + 4 * (lane / 16);
    const int tag = TAGS - (int)sl;
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
      if constexpr (BEAM == 1) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int v = (sl % 2 == 0) ? acc0[i][r] : acc1[i][r];
          if (unit0 + r < p.L) best[i][r] = max(best[i][r], (v << SHIFT) | tag);
        }
      } else {
        if (i < ntl) {
          unsigned valid = 0;
          v4i sums;
          float t[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            sums[r] = (sl % 2 == 0) ? acc0[i][r] : acc1[i][r];
            valid |= unit0 + r < p.L ? 1u << r : 0u;
          }
          beam_exponents(i, sums, valid, t);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            beam_insert(i, r, (valid >> r) & 1u ? (sums[r] << SHIFT) | tag : kNone);
            norm_sum[i] += __builtin_amdgcn_exp2f(t[r]);
          }
        }
      }
    }
  }

  if constexpr (BEAM > 1) {
    // Per sentence tile: merge the four registers' sorted lists, still as (32-bit key, 3 - register) pairs (equal sums of
    // one unit: the smaller register is the smaller index), decode the BEAM that are left into (sum, lowest index) keys,
    // merge with the three other lane groups that hold candidates of the same sentence, and write the list and the
    // normaliser's (reference, sum) pair.
    auto decode = [&](unsigned long long k) -> unsigned long long {
      const int k32 = (int)((unsigned)(k >> 32) ^ 0x80000000u);
      const int sum = k32 >> SHIFT;
      if (sum == kNoSum) return 0ull;
      const unsigned st = (unsigned)TAGS - (unsigned)(k32 & TAGS);
      const unsigned n = (first + st * stride) * 16 + 4 * (lane / 16) + (3u - (unsigned)k);
      return ((unsigned long long)((unsigned)sum ^ 0x80000000u) << 32) | (unsigned long long)(0xFFFFFFFFu - n);
    };
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
      unsigned long long top[BEAM];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        unsigned long long list[BEAM];
#pragma unroll
        for (int j = 0; j < BEAM; ++j) {
          const unsigned k32 = (unsigned)(j == 0 ? best[i][r] : more_best[i][r][j - 1]) ^ 0x80000000u;
          list[j] = ((unsigned long long)k32 << 32) | (unsigned long long)(3 - r);
        }
        if (r == 0) {
#pragma unroll
          for (int j = 0; j < BEAM; ++j) top[j] = list[j];
        } else {
          merge_sorted(top, list);
        }
      }
#pragma unroll
      for (int j = 0; j < BEAM; ++j) top[j] = decode(top[j]);
      float mx = norm_ref[i], sm = norm_sum[i];
#pragma unroll
      for (int off = 16; off <= 32; off *= 2) {
        unsigned long long other[BEAM];
#pragma unroll
        for (int j = 0; j < BEAM; ++j) other[j] = __shfl_xor(top[j], off, 64);
        merge_sorted(top, other);
        const float omx = __shfl_xor(mx, off, 64), osm = __shfl_xor(sm, off, 64);
        const float m2 = fmaxf(mx, omx);
        if (m2 > -INFINITY) {
          sm = sm * __builtin_amdgcn_exp2f(mx - m2) + osm * __builtin_amdgcn_exp2f(omx - m2);
          mx = m2;
        }
      }
      const unsigned m = (wave + kWaves * i) * 16 + lane % 16;
      if (lane < 16 && m < rows && i < ntl) {
        const size_t at = (size_t)(row0 + m) * p.columns + column;
#pragma unroll
        for (int j = 0; j < BEAM; ++j) p.partial[at * BEAM + j] = top[j];
        p.norm[at] = make_float2(mx, sm);
      }
    }
    return;
  }
  // decode the per-register winners, pick the best of the four (smaller word index on ties), merge the
  // four lane groups that share a sentence, and write one key per sentence
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    unsigned long long key = 0ull;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int sum = best[i][r] >> SHIFT;
      if (sum != kNoSum) {
        const unsigned s = (unsigned)TAGS - (unsigned)(best[i][r] & TAGS);
        const unsigned n = (first + s * stride) * 16 + 4 * (lane / 16) + r;
        const unsigned long long k =
            ((unsigned long long)((unsigned)sum ^ 0x80000000u) << 32) | (unsigned long long)(0xFFFFFFFFu - n);
        if (k > key) key = k;
      }
    }
    unsigned long long o = __shfl_xor(key, 16, 64);
    if (o > key) key = o;
    o = __shfl_xor(key, 32, 64);
    if (o > key) key = o;
    const unsigned m = (wave + kWaves * i) * 16 + lane % 16;
    // this workgroup's keys are consecutive in memory: the 16 lanes of a sentence tile fill one 128-byte line
    if (lane < 16 && m < rows) p.partial[(size_t)column * (((size_t)p.M + 15) / 16 * 16) + row0 + m] = key;
  }
}

// One workgroup per tile of 16 sentences: 16 groups of 16 lanes each take every 16th workgroup's keys of the tile (one
// 128-byte line per group and load), the groups' maxima meet in LDS, and 16 lanes decode.  Bound by the round trip to
// keys that other dies' workgroups have just written: a lane's loads (16 for 256 workgroups) all go out before the first
// is looked at (four at a time the output layer took 0.7 us longer for 300 and for 61 sentences).  There is one wave per
// SIMD, so the instructions in front of the loads count as well: as many loads as there are columns for, and 32-bit offsets
// by addition (sixteen loads always, each with a 64-bit product for its address: 7.5 us for one sentence and a list of 200
// words, 7.0 for 61 sentences; now 5.8 and 6.4).
// cols: at most 256 (cut_stream); M: rows of one launch, so that an offset fits 32 bits.
__global__ __launch_bounds__(256) void k_argmax_reduce(const unsigned long long* __restrict__ partial, unsigned cols,
                                                       unsigned M, const float* __restrict__ sA,
                                                       const float* __restrict__ sW, int32_t* __restrict__ tok,
                                                       float* __restrict__ maxlogit,
                                                       const int32_t* __restrict__ shortlist) {
  __shared__ unsigned long long red[16][16];
  const unsigned mi = threadIdx.x % 16, gs = threadIdx.x / 16;
  const unsigned m = blockIdx.x * 16 + mi;
  const unsigned pitch = (M + 15) / 16 * 16 * 8;           // bytes of a column of keys
  unsigned long long key = 0ull;
  auto columns = [&](auto trips) {
    constexpr int T = decltype(trips)::value;
    const char* keys = reinterpret_cast<const char*>(partial);
    const unsigned row = min(m, M - 1) * 8, first = row + gs * pitch, last = row + (cols - 1) * pitch;
    unsigned long long k[T];
#pragma unroll
    for (int t = 0; t < T; ++t)                            // (past the last column: that one again, which changes nothing)
      k[t] = *reinterpret_cast<const unsigned long long*>(keys + min(first + t * (16 * pitch), last));
#pragma unroll
    for (int t = 0; t < T; ++t) key = k[t] > key ? k[t] : key;
  };
  if (cols <= 16) columns(std::integral_constant<int, 1>{});
  else if (cols <= 64) columns(std::integral_constant<int, 4>{});
  else columns(std::integral_constant<int, 16>{});
  red[gs][mi] = key;
  __syncthreads();
  if (gs == 0 && m < M) {
#pragma unroll
    for (int j = 1; j < 16; ++j)
      if (red[j][mi] > key) key = red[j][mi];
    const float u = __fdiv_rn(1.0f, __fmul_rn(*sA, *sW));
    const int best = (int)((unsigned)(key >> 32) ^ 0x80000000u);
    const unsigned pos = 0xFFFFFFFFu - (unsigned)(key & 0xFFFFFFFFull);
    tok[m] = shortlist != nullptr ? shortlist[pos] : (int32_t)pos;
    maxlogit[m] = __fmul_rn((float)best, u);
  }
}

// The value of another lane of the same row of 16 lanes, by a data-parallel-primitive move.
template <int CTRL>
__device__ __forceinline__ unsigned dpp16(unsigned x) {
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
}

// Beam search: LANES = 16 or 64 lanes per row, each takes every LANES-th workgroup's list and (reference, sum) pair, up to
// four of them in flight (so 64 lanes where there are more than 64 workgroups to a row); the lanes' lists are merged
// inside rows of 16 lanes without LDS traffic (a wave per row spent 2.4 us in k rounds of six 64-bit cross-lane
// exchanges).  Writes tok [M x k] and logprob [M x k].
template <int BEAM, int LANES>
__global__ __launch_bounds__(256) void k_topk_reduce(const unsigned long long* __restrict__ partial,
                                                     const float2* __restrict__ norm, unsigned cols, unsigned M,
                                                     unsigned k, const float* __restrict__ sA,
                                                     const float* __restrict__ sW, int32_t* __restrict__ tok,
                                                     float* __restrict__ logprob,
                                                     const int32_t* __restrict__ shortlist) {
  const unsigned sub = threadIdx.x % LANES;
  const unsigned row = blockIdx.x * (256 / LANES) + threadIdx.x / LANES;
  const unsigned m = row < M ? row : M - 1;         // lanes past the end repeat the last row and write nothing
  const float u = __fdiv_rn(1.0f, __fmul_rn(*sA, *sW));
  unsigned long long top[BEAM];
#pragma unroll
  for (int j = 0; j < BEAM; ++j) top[j] = 0ull;
  float mx = -INFINITY, sm = 0.f;
  auto join = [&](float omx, float osm) {
    const float m2 = fmaxf(mx, omx);
    if (m2 > -INFINITY) {
      sm = sm * __builtin_amdgcn_exp2f(mx - m2) + osm * __builtin_amdgcn_exp2f(omx - m2);
      mx = m2;
    }
  };
  for (unsigned g0 = sub; g0 < cols; g0 += 4 * LANES) {
    // (a slot past the end reads a valid list again, which adds nothing)
    unsigned long long list[4][BEAM];
    float2 nm[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const unsigned g = g0 + LANES * t < cols ? g0 + LANES * t : g0;
      const size_t at = (size_t)m * cols + g;
#pragma unroll
      for (int j = 0; j < BEAM; ++j) list[t][j] = partial[at * BEAM + j];
      nm[t] = norm[at];
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (g0 + LANES * t < cols) {
        merge_sorted(top, list[t]);
        join(nm[t].x, nm[t].y);
      }
  }
  auto exchange = [&](auto ctrl) {
    constexpr int C = decltype(ctrl)::value;
    unsigned long long other[BEAM];
#pragma unroll
    for (int j = 0; j < BEAM; ++j)
      other[j] = ((unsigned long long)dpp16<C>((unsigned)(top[j] >> 32)) << 32) | dpp16<C>((unsigned)top[j]);
    const float omx = __uint_as_float(dpp16<C>(__float_as_uint(mx))), osm = __uint_as_float(dpp16<C>(__float_as_uint(sm)));
    merge_sorted(top, other);
    join(omx, osm);
  };
  exchange(std::integral_constant<int, 0xB1>{});     // quad_perm [1,0,3,2]
  exchange(std::integral_constant<int, 0x4E>{});     // quad_perm [2,3,0,1]
  exchange(std::integral_constant<int, 0x141>{});    // row_half_mirror
  exchange(std::integral_constant<int, 0x140>{});    // row_mirror
  if constexpr (LANES == 64) {
#pragma unroll
    for (int off = 16; off <= 32; off *= 2) {
      unsigned long long other[BEAM];
#pragma unroll
      for (int j = 0; j < BEAM; ++j) other[j] = __shfl_xor(top[j], off, 64);
      const float omx = __shfl_xor(mx, off, 64), osm = __shfl_xor(sm, off, 64);
      merge_sorted(top, other);
      join(omx, osm);
    }
  }
  if (sub < k && row < M) {
    const float lse = (mx + __builtin_amdgcn_logf(sm)) * 0.693147180559945309417f;     // log2 -> natural log
    unsigned long long w = top[0];
#pragma unroll
    for (int j = 1; j < BEAM; ++j)
      if (sub == (unsigned)j) w = top[j];
    const int sum = (int)((unsigned)(w >> 32) ^ 0x80000000u);
    const unsigned pos = 0xFFFFFFFFu - (unsigned)(w & 0xFFFFFFFFull);
    tok[(size_t)m * k + sub] = shortlist != nullptr ? shortlist[pos] : (int32_t)pos;
    logprob[(size_t)m * k + sub] = __fmul_rn((float)sum, u) - lse;
  }
}

template <int TPW, bool GATHER, int BEAM = 1, int KG = kKG, bool ROWM = false>
int launch_stream(ArgmaxParams p, unsigned grid, hipStream_t s, unsigned ny = 1) {
  constexpr size_t smem = (size_t)stages_of(KG) * kKG * kFragBytes + (size_t)kWaves * kFragBytes +
                          (GATHER ? max_units_of(KG) * 16 * sizeof(int32_t) : 0);
  static_assert(smem <= 160 * 1024, "LDS budget");
  auto kern = k_argmax_stream<TPW, GATHER, BEAM, KG, ROWM>;
  static bool attr_done = false;
  if (!attr_done) {
    int rc = check_hip(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
    if (rc != MQ_OK) return rc;
    attr_done = true;
  }
  // (t / d is the high half of t ceil(2^32 / d) while t d < 2^32: 256 columns at most, and up to 65535 chunks)
  const bool side_by_side = grid % 8 != 0 && ny > 1 && (size_t)grid * ny * ny < ((size_t)1 << 32);
  const unsigned units = GATHER ? (p.L + 15) / 16 : (unsigned)(PackedDims(8, p.N, p.K).nblocks * 2);
  p.columns = grid;
  p.units_each = units / grid;
  p.units_more = units % grid;
  p.workgroups = grid * ny;
  p.side_by_side = side_by_side ? ~0u : 0u;
  p.inner = side_by_side ? ny : grid;
  p.by_inner = (unsigned)((((unsigned long long)1 << 32) + p.inner - 1) / p.inner);
  hipLaunchKernelGGL(kern, dim3(grid * ny), dim3(kWaves * 64), smem, s, p);
  return check_hip(hipGetLastError());
}

unsigned compute_units() {
  static unsigned cus = 0;          // of the device, asked once
  if (cus == 0) {
    int dev = 0, v = 0;
    cus = 256;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
      cus = (unsigned)v;
  }
  return cus;
}

// How a launch cuts its rows and its vocabulary.  A workgroup holds up to rows_max rows and fills a compute unit (LDS),
// so n chunks of rows share the compute units: every chunk's vocabulary is cut over an n-th of them and a workgroup
// starts (hidden states into registers) and ends (winners merged and written) once.  At most max_units units of 16
// words each (the stage's place in a key), at least two columns (both units that can reach past N are then some
// workgroup's last).
struct StreamCut {
  unsigned chunks, chunk_rows, columns;
};
StreamCut cut_stream(size_t M, size_t units, size_t rows_max, size_t max_units) {
  StreamCut c;
  c.chunks = (unsigned)((M + rows_max - 1) / rows_max);
  c.chunk_rows = (unsigned)round_up((M + c.chunks - 1) / c.chunks, 16);
  const size_t share = compute_units() / c.chunks, least = (units + max_units - 1) / max_units;
  size_t columns = share > least ? share : least;
  columns = columns < 2 ? 2 : (columns > 256 ? 256 : columns);
  c.columns = (unsigned)(units < columns ? units : columns);
  return c;
}

}  // namespace

// one launch's keys: a run of (rows of the launch, rounded up to 16) keys per workgroup column
size_t argmax_stream_ws_bytes(size_t M) {
  const size_t rows = M < (size_t)kWaves * 3 * 16 ? M : (size_t)kWaves * 3 * 16;
  return (size_t)kMaxBlocks * round_up(rows, 16) * sizeof(unsigned long long);
}

// Limits: sums must fit 24 bits (127^2 K < 2^23); at most 255 units per workgroup.  Any number of rows.
bool argmax_stream_supported(size_t M, size_t N, size_t K) {
  (void)M;
  return K <= 64 * kKG && N <= (size_t)max_units_of(kKG) * 256 * 16;
}

namespace {
// How a call's rows go into launches: chunks of rows per launch as many as run side by side with the fewest columns the
// vocabulary needs (more only queue up behind a round that is nearly empty: 4096 rows, width 1024, 36 000 words in one launch
// of 16 x 18 workgroups 216 us, in two of 8 x 32 136), spread evenly over the launches.  A launch's columns x rows never
// exceed 256 x rows_max keys.
struct StreamPlan {
  size_t units, rows_max, max_units, launch_rows;
};
StreamPlan plan_stream(size_t M, size_t units, bool wide) {
  StreamPlan p;
  p.units = units;
  p.rows_max = (size_t)kWaves * 16 * (wide ? kWideTPW : kMaxTPW);
  p.max_units = max_units_of(wide ? kWideKG : kKG);
  const size_t fewest = (units + p.max_units - 1) / p.max_units;
  const size_t chunks = (M + p.rows_max - 1) / p.rows_max, side_by_side = compute_units() / (fewest < 2 ? 2 : fewest);
  const size_t launches = side_by_side == 0 ? chunks : (chunks + side_by_side - 1) / side_by_side;
  p.launch_rows = (chunks + launches - 1) / launches * p.rows_max;      // (whole 32-row blocks)
  return p;
}
unsigned tiles_per_wave(const StreamCut& c) { return (c.chunk_rows / 16 + kWaves - 1) / kWaves; }
}  // namespace

// The same on plain row-major hidden states, K up to 1024 in whole 16-byte pieces.
bool argmax_stream_rows_supported(size_t N, size_t K) {
  return K % 16 == 0 && K <= 64 * kWideKG && N <= (size_t)max_units_of(K <= 64 * kKG ? kKG : kWideKG) * 256 * 16;
}

// Plain rows: the streaming kernel or the tiled product with the arg-max in its epilogue.  The tiled one multiplies 128 x 128
// tiles and wins where the matrix instructions are few (narrow widths, which the streaming kernel multiplies as 512 or 1024
// elements all the same) or the rows many against the words; one atomic maximum per row and 128 words holds it back.  In
// microseconds, kernels alone, fitted to 1771 timed calls (widths 16 to 1024, 300 to 50 000 words, 1 to 16 384 rows;
// 5 - 7 % off on average).  They were fitted to the streaming kernel before its refilling stages became up to 18 % faster.  With the
// present one, on the same calls (profiles/output_layer_form_timings.csv): choosing by these is 0.8 % slower than the faster form
// of each call on average, at worst 47 % (width 528, where the tiled product keeps 300 rows against 36 000 words, 26.8 for 18.2 us),
// and on 600 others (200 to 80 000 words) 0.7 %, never more than 12 % slower than the tiled product; always streaming 5.0 %, never
// streaming 17 %.
bool argmax_stream_rows_ahead(size_t M, size_t N, size_t K) {
  const bool wide = K > 64 * kKG;
  const float k = (float)((K + 63) / 64);
  const StreamPlan plan = plan_stream(M, PackedDims(8, N, K).nblocks * 2, wide);
  auto launch = [&](size_t nrows) {
    const StreamCut c = cut_stream(nrows, plan.units, plan.rows_max, plan.max_units);
    const unsigned tpw = tiles_per_wave(c);
    const float units = (float)((plan.units + c.columns - 1) / c.columns), rows = (float)c.chunk_rows;      // of a workgroup
    if (wide)
      return 5.5f + units * (0.43f + (tpw > 1 ? 0.244f : 0.f) + 0.0074f * k) + rows * (0.0114f + 0.0015f * k + 0.000093f * (float)c.chunks);
    return 5.2f + units * (0.217f + (tpw > 2 ? 0.305f : tpw > 1 ? 0.19f : 0.f) + 0.0015f * k) + rows * (0.0094f + 0.0012f * k);
  };
  const size_t full = (M - 1) / plan.launch_rows;                  // launches of launch_rows rows in front of the last one
  const float stream = (full != 0 ? (float)full * launch(plan.launch_rows) : 0.f) + launch(M - full * plan.launch_rows);
  const size_t tiles_n = (N + 127) / 128, tiles = (M + 127) / 128 * tiles_n;
  const float rounds = (float)((tiles + 255) / 256), rounds_of_two = (float)((tiles + 511) / 512);
  const float tiled = 7.6f + rounds * (0.116f + 0.158f * k) + rounds_of_two * 0.179f * k +
                      (float)tiles_n * (0.0067f + 0.0000193f * (float)M + 0.0000608f * (float)(M < 128 ? M : 128));
  return stream < tiled;
}

// hidden: packed, or (row_major) plain rows.  ws_keys: keys the partials array at ws holds.
static int launch_argmax_any(const uint8_t* hidden, bool row_major, const void* packedW, size_t M, size_t N, size_t K,
                             const float* sA, const float* sW, int32_t* tok, float* maxlogit, void* ws, size_t ws_keys,
                             const int32_t* shortlist, size_t shortlist_len, hipStream_t s) {
  const bool wide = K > 64 * kKG;
  const PackedDims dW(8, N, K), dAll(8, M, K);
  const StreamPlan plan = plan_stream(M, shortlist != nullptr ? (shortlist_len + 15) / 16 : dW.nblocks * 2, wide);
  for (size_t row0 = 0; row0 < M;) {
    const size_t nrows = M - row0 < plan.launch_rows ? M - row0 : plan.launch_rows;
    const StreamCut c = cut_stream(nrows, plan.units, plan.rows_max, plan.max_units);
    if ((size_t)c.columns * round_up(nrows, 16) > ws_keys || (plan.units + c.columns - 1) / c.columns > plan.max_units)
      return MQ_ERR_UNSUPPORTED;
    ArgmaxParams p{};
    p.packedA = row_major ? hidden + row0 * K : hidden + dAll.frag_offset(row0 / 32, 0);   // (row0: whole 32-row blocks)
    p.packedW = static_cast<const uint8_t*>(packedW);
    p.M = (unsigned)nrows; p.N = (unsigned)N; p.K = (unsigned)K;
    p.partial = static_cast<unsigned long long*>(ws);
    p.shortlist = shortlist;
    p.L = shortlist != nullptr ? (unsigned)shortlist_len : (unsigned)N;
    p.sA = sA; p.sW = sW;
    p.chunk_rows = c.chunk_rows;
    const unsigned tpw = tiles_per_wave(c);
    const unsigned g = c.columns, ny = c.chunks;
    int rc;
    if (shortlist != nullptr)
      rc = tpw == 1 ? launch_stream<1, true>(p, g, s, ny) : tpw == 2 ? launch_stream<2, true>(p, g, s, ny) : launch_stream<3, true>(p, g, s, ny);
    else if (!row_major)
      rc = tpw == 1 ? launch_stream<1, false>(p, g, s, ny) : tpw == 2 ? launch_stream<2, false>(p, g, s, ny) : launch_stream<3, false>(p, g, s, ny);
    else if (wide)
      rc = tpw == 1 ? launch_stream<1, false, 1, kWideKG, true>(p, g, s, ny) : launch_stream<2, false, 1, kWideKG, true>(p, g, s, ny);
    else
      rc = tpw == 1 ? launch_stream<1, false, 1, kKG, true>(p, g, s, ny)
                    : tpw == 2 ? launch_stream<2, false, 1, kKG, true>(p, g, s, ny) : launch_stream<3, false, 1, kKG, true>(p, g, s, ny);
    if (rc != MQ_OK) return rc;
    hipLaunchKernelGGL(k_argmax_reduce, dim3((unsigned)((nrows + 15) / 16)), dim3(256), 0, s, p.partial, g,
                       (unsigned)nrows, sA, sW, tok + row0, maxlogit + row0, shortlist);
    rc = check_hip(hipGetLastError());
    if (rc != MQ_OK) return rc;
    row0 += nrows;
  }
  return MQ_OK;
}

int launch_argmax_stream(const void* packedA, const void* packedW, size_t M, size_t N, size_t K, const float* sA,
                         const float* sW, int32_t* tok, float* maxlogit, void* ws, size_t ws_bytes, const int32_t* shortlist,
                         size_t shortlist_len, hipStream_t s) {
  if (!argmax_stream_supported(M, N, K)) return MQ_ERR_UNSUPPORTED;
  return launch_argmax_any(static_cast<const uint8_t*>(packedA), false, packedW, M, N, K, sA, sW, tok, maxlogit, ws,
                           ws_bytes / sizeof(unsigned long long), shortlist, shortlist_len, s);
}

int launch_argmax_stream_rows(const void* qA, const void* packedW, size_t M, size_t N, size_t K, const float* sA,
                              const float* sW, int32_t* tok, float* maxlogit, void* ws, size_t ws_bytes, hipStream_t s) {
  if (!argmax_stream_rows_supported(N, K)) return MQ_ERR_UNSUPPORTED;
  return launch_argmax_any(static_cast<const uint8_t*>(qA), true, packedW, M, N, K, sA, sW, tok, maxlogit, ws,
                           ws_bytes / sizeof(unsigned long long), nullptr, 0, s);
}

// ---- the same output layer for callers that cannot allocate: partial winners in a static device array ----
// kStaticRows x kStaticCols keys, 768 KiB per device, held until the process ends.  Rows that need more go in further
// launches that reuse it one after the other on the stream.
namespace {
constexpr size_t kStaticRows = (size_t)kWaves * 3 * 16;     // rows of one pass of the streaming kernel (384)
constexpr unsigned kStaticCols = 256;
constexpr int kMaxDevices = 64;
static __device__ __align__(256) unsigned long long scratch[kStaticRows * kStaticCols];
std::mutex g_scratch_mutex;
unsigned long long* g_scratch_ptr[kMaxDevices] = {};      // device address of `scratch` on each device, asked once
}  // namespace

size_t argmax_static_max_rows() { return kStaticRows * 64; }

int launch_argmax_stream_static(const void* packedA, const void* packedW, size_t M, size_t N, size_t K,
                                const float* sA, const float* sW, int32_t* tok, float* maxlogit, hipStream_t s) {
  int dev = -1;
  if (check_hip(hipGetDevice(&dev)) != MQ_OK) return MQ_ERR_HIP;
  if (dev < 0 || dev >= kMaxDevices) return MQ_ERR_UNSUPPORTED;
  unsigned long long* ptr;
  {
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
      // `scratch` itself is only a host-side handle: kernels get the address the runtime reports for this device
      void* addr = nullptr;
      const int rc = check_hip(hipGetSymbolAddress(&addr, HIP_SYMBOL(scratch)));
      if (rc != MQ_OK || addr == nullptr) return MQ_ERR_HIP;
      g_scratch_ptr[dev] = static_cast<unsigned long long*>(addr);
    }
    ptr = g_scratch_ptr[dev];
  }
  // every key the reduce kernel reads was written by this call's streaming kernel: nothing has to start at zero
  return launch_argmax_stream(packedA, packedW, M, N, K, sA, sW, tok, maxlogit, ptr, sizeof(unsigned long long) * kStaticRows * kStaticCols,
                              nullptr, 0, s);
}

size_t topk_stream_ws_bytes(size_t M, int k) {
  // every row's candidates and normalisers from up to 256 workgroups (rows go 256 to a workgroup, all chunks in one launch)
  const int beam = k <= 2 ? 2 : 4;
  return round_up((size_t)256 * M * beam * sizeof(unsigned long long), 256) + (size_t)256 * M * sizeof(float2);
}

bool topk_stream_supported(size_t M, size_t N, size_t K, int k) {
  (void)M;
  return k >= 1 && k <= 4 && (size_t)k <= N && K <= 64 * kKG && N <= (size_t)max_units_of(kKG) * 256 * 16;
}

// Beam-search output layer: the k <= 4 best words of every row with log-probabilities.  Rows are processed in
// chunks of 256 (two sentence tiles per wave), each chunk streaming the embedding once, all chunks in one launch.
int launch_topk_stream(const void* packedA, const void* packedW, size_t M, size_t N, size_t K, const float* sA,
                       const float* sW, int k, int32_t* tok, float* logprob, void* ws, const int32_t* shortlist,
                       size_t shortlist_len, hipStream_t s) {
  if (!topk_stream_supported(M, N, K, k)) return MQ_ERR_UNSUPPORTED;
  if (shortlist != nullptr && (size_t)k > shortlist_len) return MQ_ERR_SHAPE;
  const PackedDims dW(8, N, K);
  const size_t units = shortlist != nullptr ? (shortlist_len + 15) / 16 : dW.nblocks * 2;
  const int beam = k <= 2 ? 2 : 4;
  unsigned long long* keys = static_cast<unsigned long long*>(ws);
  float2* norm = reinterpret_cast<float2*>(static_cast<uint8_t*>(ws) +
                                           round_up((size_t)256 * M * beam * sizeof(unsigned long long), 256));
  // Rows go up to 256 (two sentence tiles per wave) to a workgroup; all chunks run in ONE launch that shares the compute units (cut_stream), and one
  // reduce launch follows for all rows: a launch per chunk (ten for 1200 rows) cost more than the chunks' work.
  const StreamCut c = cut_stream(M, units, (size_t)kWaves * 16 * kBeamTPW, max_units_of(kKG));
  // (65535 chunks: what chunk_of's reciprocals are good for.  The workgroups stay far below what a launch holds, 2^32 threads: the
  // entry point takes 2^40 logits at most, which are 1.1 million workgroups of 256 rows and 255 units.)
  if (c.chunks > 65535u || (units + c.columns - 1) / c.columns > max_units_of(kKG)) return MQ_ERR_UNSUPPORTED;
  ArgmaxParams p{};
  p.packedA = static_cast<const uint8_t*>(packedA);
  p.packedW = static_cast<const uint8_t*>(packedW);
  p.M = (unsigned)M; p.N = (unsigned)N; p.K = (unsigned)K;
  p.partial = keys; p.norm = norm; p.sA = sA; p.sW = sW;
  p.shortlist = shortlist;
  p.L = shortlist != nullptr ? (unsigned)shortlist_len : (unsigned)N;
  p.chunk_rows = c.chunk_rows;
  const unsigned tpw = tiles_per_wave(c);
  const unsigned grid = c.columns, ny = c.chunks;
  auto go = [&](auto gather, auto beam_tag) -> int {
    constexpr bool G = decltype(gather)::value;
    constexpr int B = decltype(beam_tag)::value;
    return tpw == 1 ? launch_stream<1, G, B>(p, grid, s, ny) : launch_stream<kBeamTPW, G, B>(p, grid, s, ny);
  };
  using B2 = std::integral_constant<int, 2>;
  using B4 = std::integral_constant<int, 4>;
  int rc;
  if (shortlist != nullptr) rc = beam == 2 ? go(std::true_type{}, B2{}) : go(std::true_type{}, B4{});
  else rc = beam == 2 ? go(std::false_type{}, B2{}) : go(std::false_type{}, B4{});
  if (rc != MQ_OK) return rc;
  auto reduce = [&](auto beam_tag, auto lanes_tag) {
    constexpr int B = decltype(beam_tag)::value, LN = decltype(lanes_tag)::value;
    hipLaunchKernelGGL((k_topk_reduce<B, LN>), dim3((unsigned)((M + 256 / LN - 1) / (256 / LN))), dim3(256), 0, s, keys, norm, grid,
                       (unsigned)M, (unsigned)k, sA, sW, tok, logprob, shortlist);
  };
  using L16 = std::integral_constant<int, 16>;
  using L64 = std::integral_constant<int, 64>;
  if (beam == 2) grid > 64 ? reduce(B2{}, L64{}) : reduce(B2{}, L16{});
  else grid > 64 ? reduce(B4{}, L64{}) : reduce(B4{}, L16{});
  return check_hip(hipGetLastError());
}

}  // namespace mq
