// One decoder layer of up to eight sentences, from the second product of the averaging network to the last normalisation, in
// ONE launch (arxiv 1805.12096, Section 3.2; Section 4.2: every activation is quantized on each call).
//
// With a handful of rows a layer is a chain of phases, each a few hundred nanoseconds of work on a few KB behind a dependency on
// everything the phase before produced.  As launches each phase costs its start (arguments, addresses, parameters and rows
// asked for one after the other from cold caches) and its end: eight of them 30 us.  Here the workgroups stay: a workgroup
// keeps its 32 columns of every product, asks for the next phase's parameters while it waits for this one's rows, and the
// rows travel through memory with the data as its own flag -- the launch in front fills the exchange buffers with a word no
// result has, device-scope relaxed stores replace it, device-scope relaxed loads poll until it is gone (1.5 us from the last
// store to everybody's registers, where a kernel boundary and the loads behind it cost 2.5 to 3).
// Figures: at launch_layer_rows.
//
// Who does what, and why no wait is for ever.  Role r owns columns 32 r .. 32 r + 31 of each product that has them (and the
// source attention of every sentence for their heads; role 0 also the last normalisation).  A workgroup claims the role of its block index when it
// starts.  If other kernels keep some workgroups of this one from starting, the others do not wait for them: one that has
// polled in vain for a while (LayerParams::patience) looks for roles nobody has claimed, claims some, and begins again at the first phase with them
// (everything it has published already it publishes again, the same words); a workgroup whose role is gone when it starts
// ends at once.  So every role belongs to a workgroup that runs, phases only wait for phases before them, and the grid drains
// under any residency.  The waits are bounded all the same (mq_set_barrier_timeout_us, half a second at most), and no result
// hangs on one: a workgroup that has waited so long twice ends, but for role 0's, which then does every role itself.
//
// Arithmetic and its order are those of the kernels this replaces (mq_gemm_rows.hip, mq_glue.hip): the same bits.
#include "mq_gemm_common.h"
#include "mq_glue.h"
#include "mq_grid_max.h"

namespace mq {

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned long long u64;

constexpr int kLW = 8;                         // waves; wave w holds row w
constexpr int kLT = kLW * 64;
constexpr unsigned kTake = 4;                  // roles taken over at a time
constexpr unsigned kTries = 2;                 // passes that wait with every role claimed
constexpr unsigned kLongest = 50000000u;       // half a second of the 100 MHz wall clock
constexpr int kHalf8 = 8 * 16 + 16, kFrag8 = 2 * kHalf8;      // a staged fragment: two K halves of eight rows, 16 bytes each

struct LayerParams {
  // (one line of arguments for the loads of the first phase, the rest in the order of the phases)
  const float* hid;
  const uint8_t* wa2;
  const float* x;
  const uint8_t* wg;
  unsigned* claim;
  unsigned M, S, aan, ffn, roles, head_shift;                    // d / heads = 1 << head_shift
  const float *sa2, *sg, *sq, *so, *s1, *s2;
  const float *ba2, *bg, *bq, *bo, *b1, *b2;
  unsigned *f, *mix;
  const uint8_t *wq, *wo, *w1, *w2;
  const float *gamma1, *beta1, *K, *V;
  unsigned *q, *ctx, *o, *hid2, *ff;                             // exchange: kUnsetWord until published
  const float *gamma2, *beta2, *gamma3, *beta3;
  float* y;
  float eps;
  unsigned patience, limit, heads;                               // ticks before roles are taken over, ticks of a wait
};

__device__ __forceinline__ uint32_t bytes_of4(const int (&q)[4]) {
  return __builtin_amdgcn_perm((uint32_t)q[1], (uint32_t)q[0], 0x0c0c0400u) | __builtin_amdgcn_perm((uint32_t)q[3], (uint32_t)q[2], 0x04000c0cu);
}

__device__ __forceinline__ void publish(unsigned* dst, float v) {
  const unsigned b = __float_as_uint(v);
  __hip_atomic_store(dst, b == kUnsetWord ? 0x7FC00000u : b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr int kDeviceScope = 16;                                // cache policy sc1

// CH pieces of 256 floats of a row into a wave's registers, element 256 c + 4 lane + t as v[c][t]; false when the row was not
// complete after `patience` ticks.  REST: no hurry.
template <bool REST = false, int CH>
__device__ __forceinline__ bool poll_row(const unsigned* row, unsigned len, f4 (&v)[CH], unsigned patience) {
  const unsigned lane = threadIdx.x % 64;
  const unsigned long long t0 = wall_clock64();
  // (16 bytes a load at device scope; every word is its own flag)
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned*>(row), 0, (int)(len * 4), 0x00027000);
  for (;;) {
    u4 a[CH];
    unsigned at = 4u * lane;
    asm volatile("" : "+v"(at));                                 // (each turn reads anew)
#pragma unroll
    for (int c = 0; c < CH; ++c)
      a[c] = __builtin_bit_cast(u4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(4 * min(256u * c + at, len - 4)), 0, kDeviceScope));
    bool there = true;
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        there = there && a[c][t] != kUnsetWord;
        v[c][t] = __uint_as_float(a[c][t]);
      }
    if (__all(there)) return true;
    if (wall_clock64() - t0 >= patience) return false;
    if constexpr (REST) __builtin_amdgcn_s_sleep(32);            // under a microsecond
  }
}

template <int CH>
__device__ __forceinline__ float row_absmax(const f4 (&v)[CH]) {
  float m = 0.f;
#pragma unroll
  for (int c = 0; c < CH; ++c)
#pragma unroll
    for (int t = 0; t < 4; ++t) m = fmaxf(m, fabsf(v[c][t]));               // drops NaN
  return __uint_as_float(wave_max_u32(__float_as_uint(m)));
}

// v = LN(v + r) gamma + beta, as k_layer_norm_wave
template <int CH>
__device__ __forceinline__ void normalise(f4 (&v)[CH], const f4 (&r)[CH], const f4 (&gv)[CH], const f4 (&bv)[CH], float eps) {
  constexpr float d = 256.0f * CH;
  float x[CH][4];
#pragma unroll
  for (int c = 0; c < CH; ++c)
#pragma unroll
    for (int t = 0; t < 4; ++t) x[c][t] = v[c][t] = v[c][t] + r[c][t];
  const float mu = row_sum_f(x) / d;
#pragma unroll
  for (int c = 0; c < CH; ++c)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      v[c][t] -= mu;
      x[c][t] = v[c][t] * v[c][t];
    }
  const float inv = __fdiv_rn(1.0f, sqrtf(row_sum_f(x) / d + eps));
#pragma unroll
  for (int c = 0; c < CH; ++c)
#pragma unroll
    for (int t = 0; t < 4; ++t) v[c][t] = v[c][t] * inv * gv[c][t] + bv[c][t];
}

// CD = d / 256; CW: the inner widths are at most 256 CW.
template <int CD, int CW>
__global__ __launch_bounds__(kLT) void k_layer_rows(const LayerParams p) {
  constexpr unsigned d = 256u * CD, nd = d / 32;
  constexpr int kStage = (CW > 2 * CD ? CW : 2 * CD) * 8 * kFrag8;
  constexpr unsigned COLS = d / 4, SG = kLT / COLS;            // source attention: float4 columns, groups that share the positions
  __shared__ __attribute__((aligned(16))) uint8_t stage[kStage];
  __shared__ __attribute__((aligned(16))) int part[kLW * 2 * 256];
  __shared__ float scores[4096];                               // [kLW][heads of 32 columns][S]
  __shared__ float red[2][kLW];
  __shared__ unsigned owned[kLayerClaims], n_owned, claimed_own, some_left;
  int tid = threadIdx.x, lane = tid % 64, lj = lane % 32, lh = lane / 32;
  unsigned wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const unsigned M = p.M, nf = p.ffn / 32;
  unsigned row = min(wave, M - 1);
  const unsigned role0 = blockIdx.x;
  // fragments of a parameter's column block: wave w holds K slices w KW .. w KW + KW - 1
  auto fetch = [&](auto& w, const uint8_t* packed, unsigned block, unsigned K) {
    constexpr int KW = sizeof(w) / sizeof(u4);
    const unsigned kfrags = K / 32;
#pragma unroll
    for (int j = 0; j < KW; ++j)
      w[j] = *reinterpret_cast<const u4*>(packed + ((size_t)block * kfrags + min(wave * KW + j, kfrags - 1)) * kFragBytes + lane * 16);
  };
  auto row_of = [&](auto& v, const float* src, unsigned len) {
    constexpr int CH = sizeof(v) / sizeof(f4);
#pragma unroll
    for (int c = 0; c < CH; ++c) v[c] = *reinterpret_cast<const f4*>(src + min(256u * c + 4u * lane, len - 4));
  };
  // quant_int of this wave's row into the staged fragments
  auto put = [&](const auto& v, unsigned len, float s) {
    constexpr int CH = sizeof(v) / sizeof(f4);
    if (wave >= M) return;
#pragma unroll
    for (int c = 0; c < CH; ++c)
      if (256u * c + 4u * lane < len) {
        int q[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const float r = rintf(__fmul_rn(v[c][t], s));
          asm("v_cvt_i32_f32 %0, %1" : "=v"(q[t]) : "v"(r));          // saturates, NaN -> 0
          q[t] = min(max(q[t], -127), 127);
        }
        *reinterpret_cast<uint32_t*>(stage + (8 * c + lane / 8) * kFrag8 + ((lane / 4) % 2) * kHalf8 + wave * 16 + 4 * (lane % 4)) = bytes_of4(q);
      }
  };
  // this wave's share of a column block's sums (rows 0 .. 7: registers 0 .. 3 of the result) to LDS
  auto multiply = [&](const auto& w, unsigned K, int nb) {
    constexpr int KW = sizeof(w) / sizeof(u4);
    constexpr int kTogether = KW < 8 ? KW : 8;                   // fragments asked for before the first is used
    v16i acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0;
#pragma unroll
    for (int j0 = 0; j0 < KW; j0 += kTogether) {
      u4 a[kTogether];
#pragma unroll
      for (int j = 0; j < kTogether; ++j)
        a[j] = *reinterpret_cast<const u4*>(stage + min(wave * KW + j0 + j, K / 32 - 1) * kFrag8 + lh * kHalf8 + (lj % 8) * 16);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < kTogether; ++j) {
        const uint32_t inside = wave * KW + j0 + j < K / 32 ? ~0u : 0u;
        acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(as_v4i(a[j]), as_v4i(w[j0 + j] & inside), acc, 0, 0, 0);
      }
    }
    reinterpret_cast<v4i*>(part)[(wave * 2 + nb) * 64 + lane] = v4i{acc[0], acc[1], acc[2], acc[3]};
  };
  // threads 0 .. 255 finish one element each: row 4 lh + wave, column lj of the block
  auto total = [&](int nb) -> int {
    unsigned sum = 0;
#pragma unroll
    for (int k = 0; k < kLW; ++k) sum += (unsigned)part[((k * 2 + nb) * 64 + lane) * 4 + (int)wave];
    return (int)sum;
  };
  unsigned em = 4 * lh + wave;                                  // (valid for tid < 256)
  // whether all rows are there, and their maximum; every thread gets the same answer
  float amax = 0.f;
  int turn = 0;                                                  // (two buffers: one barrier a time is enough)
  auto agree = [&](bool ok, float m) -> bool {
    turn ^= 1;
    if (lane == 0) red[turn][wave] = ok ? m : -1.0f;
    __syncthreads();
    float lo = red[turn][0], hi = lo;
#pragma unroll
    for (int k = 1; k < kLW; ++k) {
      lo = fminf(lo, red[turn][k]);
      hi = fmaxf(hi, red[turn][k]);
    }
    amax = hi;
    return __builtin_amdgcn_readfirstlane(lo >= 0.0f ? 1 : 0) != 0;
  };
  unsigned count = 1;                                            // roles owned (past the first pass)
  unsigned patience = p.patience;
  // One pass through the phases; false when some row did not come in time.  The first one has the workgroup's own role and
  // asks for parameters ahead; a later one serves `count` roles and is only correct (as one body in a loop the compiler keeps
  // every phase's addresses and parameters in registers across it, and spills).
  auto pass = [&](auto first_pass) -> bool {
    constexpr bool kFirst = decltype(first_pass)::value;
    auto role_at = [&](unsigned i) { return kFirst ? role0 : (unsigned)__builtin_amdgcn_readfirstlane(owned[i]); };
    auto owns_below = [&](unsigned limit) {
      if constexpr (kFirst) return role0 < limit;
      bool any = false;
      for (unsigned i = 0; i < count; ++i) any = any || owned[i] < limit;
      return __builtin_amdgcn_readfirstlane(any ? 1 : 0) != 0;
    };
    auto for_roles = [&](unsigned limit, auto body) {
      if constexpr (kFirst) {
        if (role0 < limit) body(role0);
      } else {
        for (unsigned i = 0; i < count; ++i) {
          const unsigned r = role_at(i);
          if (r < limit) body(r);
          __syncthreads();                                       // `part` and `scores` are written again
        }
      }
    };
    // quantized rows staged: finish(role, sum, bias) for threads 0 .. 255
    auto product = [&](auto& w, const uint8_t* packed, unsigned K, unsigned blocks, const float* bias, float ahead, auto finish) {
      for_roles(blocks, [&](unsigned r) {
        if constexpr (!kFirst) fetch(w, packed, r, K);
        const float b = kFirst ? ahead : bias != nullptr ? bias[r * 32 + lj] : 0.f;
        multiply(w, K, 0);
        __syncthreads();
        if (tid < 256) finish(r, total(0), b);
      });
    };
    f4 x[CD], y1[CD], y2[CD];
    // ---- f = W2 hid
    u4 w2[CW], wg[2][2 * CD];
    f4 hid[CW];
    const bool narrow = owns_below(nd), narrow0 = kFirst && narrow;
    if (narrow) row_of(hid, p.hid + (size_t)row * p.aan, p.aan);
    if (narrow0) fetch(w2, p.wa2, role0, p.aan);
    row_of(x, p.x + (size_t)row * d, d);
    if (narrow0) {
      fetch(wg[0], p.wg, role0, 2 * d);
      fetch(wg[1], p.wg, role0 + nd, 2 * d);
    }
    // (biases and multipliers of every phase; the slow pass reads them where they are used)
    auto bias_at = [&](const float* bias, unsigned block) { return bias != nullptr ? bias[block * 32 + lj] : 0.f; };
    const float sa2 = *p.sa2, sg = *p.sg, sq = *p.sq, so = *p.so, s1 = *p.s1, s2 = *p.s2;
    float ba2 = 0.f, bg1 = 0.f, bg2 = 0.f, bq = 0.f, bo = 0.f, b1 = 0.f, b2 = 0.f;
    if (narrow0) {
      ba2 = bias_at(p.ba2, role0);
      bg1 = bias_at(p.bg, role0);
      bg2 = bias_at(p.bg, role0 + nd);
      bq = bias_at(p.bq, role0);
      bo = bias_at(p.bo, role0);
      b2 = bias_at(p.b2, role0);
    }
    if (kFirst && role0 < nf) b1 = bias_at(p.b1, role0);
    unsigned was;
    if (kFirst && tid == 0) was = __hip_atomic_exchange(p.claim + role0, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_sched_barrier(0);
    // Whether the role is this workgroup's is not waited for at first: f is right whoever computes it.
    auto mine = [&] {
      if constexpr (!kFirst) return true;
      return __builtin_amdgcn_readfirstlane(claimed_own) != 0u;
    };
    auto answer = [&] {
      if constexpr (kFirst) {
        asm volatile("" : "+v"(was));                            // (or the comparison, and a wait, follow the exchange at once)
        if (tid == 0) {
          owned[0] = role0;
          n_owned = 1;
          claimed_own = was == kUnsetWord ? 1u : 0u;
        }
      }
    };
    bool ok = true;
    if (narrow) {
      agree(true, wave < M ? row_absmax(hid) : 0.f);
      const float s = amax > 0.0f ? __fdiv_rn(127.0f, amax) : 1.0f;
      put(hid, p.aan, s);
      __syncthreads();
      const float u = __fdiv_rn(1.0f, __fmul_rn(s, sa2));
      product(w2, p.wa2, p.aan, nd, p.ba2, ba2, [&](unsigned r, int sum, float b) {
        if (em < M) publish(p.f + em * d + r * 32 + lj, fmaf((float)sum, u, b));
      });
    }
    // ---- mix = sigmoid(z1) x + sigmoid(z2) f, [z1; z2] = Wg [x; f]
    u4 wq[CD], wo[CD], w1[CD];
    if (narrow0) {
      fetch(wq, p.wq, role0, d);
      fetch(wo, p.wo, role0, d);
    }
    if (kFirst && role0 < nf) fetch(w1, p.w1, role0, d);
    f4 gv[CD], bv[CD];
    row_of(gv, p.gamma1, d);
    row_of(bv, p.beta1, d);
    __builtin_amdgcn_sched_barrier(0);
    if (narrow) {
      f4 in[2 * CD], f[CD];
      ok = wave >= M || poll_row(p.f + (size_t)row * d, d, f, patience);
#pragma unroll
      for (int c = 0; c < CD; ++c) {
        in[c] = x[c];
        in[CD + c] = f[c];
      }
      answer();
      ok = agree(ok, wave < M ? row_absmax(in) : 0.f);
      if (!mine()) return true;
      if (ok) {
        const float s = amax > 0.0f ? __fdiv_rn(127.0f, amax) : 1.0f;
        put(in, 2 * d, s);
        const float u = __fdiv_rn(1.0f, __fmul_rn(s, sg));
        __syncthreads();
        for_roles(nd, [&](unsigned r) {
          const unsigned n = r * 32 + lj, m = min(em, M - 1);
          if constexpr (!kFirst) {
            fetch(wg[0], p.wg, r, 2 * d);
            fetch(wg[1], p.wg, r + nd, 2 * d);
          }
          const float bias1 = kFirst ? bg1 : bias_at(p.bg, r), bias2 = kFirst ? bg2 : bias_at(p.bg, r + nd);
          float xv = 0.f, fv = 0.f;
          if (tid < 256) {
            xv = p.x[(size_t)m * d + n];
            fv = __uint_as_float(__hip_atomic_load(p.f + (size_t)m * d + n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
          }
          multiply(wg[0], 2 * d, 0);
          multiply(wg[1], 2 * d, 1);
          __syncthreads();
          if (tid < 256 && em < M) {
            const float z1 = fmaf((float)total(0), u, bias1), z2 = fmaf((float)total(1), u, bias2);
            publish(p.mix + em * d + n, sigmoidf_(z1) * xv + sigmoidf_(z2) * fv);
          }
        });
      }
    }
    // ---- y1 = LN(mix + x), q = Wq y1 (who has no columns of q asks seldom: the fewer ask for a line, the sooner it comes)
    if (ok) {
      if (narrow) ok = wave >= M || poll_row(p.mix + (size_t)row * d, d, y1, patience);
      else ok = wave >= M || poll_row<true>(p.mix + (size_t)row * d, d, y1, patience);
      if (ok) normalise(y1, x, gv, bv, p.eps);
      if (!narrow) answer();
      ok = agree(ok, wave < M ? row_absmax(y1) : 0.f);
      if (!mine()) return true;
    }
    if (ok && narrow) {
      const float s = amax > 0.0f ? __fdiv_rn(127.0f, amax) : 1.0f;
      put(y1, d, s);
      __syncthreads();
      const float u = __fdiv_rn(1.0f, __fmul_rn(s, sq));
      product(wq, p.wq, d, nd, p.bq, bq, [&](unsigned r, int sum, float b) {
        if (em < M) publish(p.q + em * d + r * 32 + lj, fmaf((float)sum, u, b));
      });
    }
    // ---- source attention: wave w serves sentence w, for the heads of the workgroup's columns only, on its own (with a
    // sentence per workgroup instead its 1.8 us were the longest phase)
    if (ok && narrow)
      for_roles(nd, [&](unsigned r) {
        if (!ok) return;
        const unsigned S = p.S, hs = p.head_shift, dh = 1u << hs, grp = dh / 4, per = 64 / grp;      // positions a trip
        const unsigned nh = hs >= 5 ? 1u : 32u >> hs, head0 = r * 32 >> hs;                          // heads here
        const float scale = __fdiv_rn(1.0f, sqrtf((float)dh));
        const f4* K4 = reinterpret_cast<const f4*>(p.K + (size_t)row * S * d);
        const f4* V4 = reinterpret_cast<const f4*>(p.V + (size_t)row * S * d) + r * 8 + lane % 8;
        // groups that share the positions of V: SG of the eight, the others repeat them (the order of the additions is that of
        // the attention kernel this replaces)
        const unsigned sg = lane / 8;
        constexpr int kTrips = 8;
        f4 kr[kTrips], va[kTrips], q[1];
        auto keys = [&](unsigned head, unsigned s0) {
#pragma unroll
          for (int u = 0; u < kTrips; ++u)
            kr[u] = K4[(size_t)min(s0 + u * per + lane / grp, S - 1) * COLS + head * grp + (lane & (grp - 1))];
        };
        auto values = [&](unsigned s0) {
#pragma unroll
          for (int j = 0; j < kTrips; ++j) va[j] = V4[(size_t)min(s0 + j * SG + sg % SG, S - 1) * COLS];
        };
        keys(head0, 0u);
        values(0u);
        __builtin_amdgcn_sched_barrier(0);
        const unsigned q_len = hs >= 5 ? dh : 32u;
        const bool came = wave >= M || poll_row(p.q + (size_t)row * d + head0 * dh, q_len, q, patience);
        if (came && wave < M) {
          float* mine_sc = scores + wave * nh * S;
          for (unsigned hh = 0; hh < nh; ++hh) {
            f4 qr;
#pragma unroll
            for (int t = 0; t < 4; ++t) qr[t] = __shfl(q[0][t], hh * grp + (lane & (grp - 1)), kWave);
            for (unsigned s0 = 0; s0 < S; s0 += kTrips * per) {
              if (hh != 0 || s0 != 0) keys(head0 + hh, s0);
              float a[kTrips][1];
#pragma unroll
              for (int u = 0; u < kTrips; ++u)
                a[u][0] = fmaf(qr.x, kr[u].x, fmaf(qr.y, kr[u].y, fmaf(qr.z, kr[u].z, qr.w * kr[u].w)));
              group_sums_f(a, grp);
#pragma unroll
              for (int u = 0; u < kTrips; ++u) {
                const unsigned at = s0 + u * per + lane / grp;
                if ((lane & (grp - 1)) == 0 && at < S) mine_sc[hh * S + at] = a[u][0] * scale;
              }
            }
            float* sc = mine_sc + hh * S;
            float mx = -INFINITY;
            for (unsigned at = lane; at < S; at += kWave) mx = fmaxf(mx, sc[at]);
            mx = wave_max_f(mx);
            float sum = 0.f;
            for (unsigned at = lane; at < S; at += kWave) {
              const float e = expf(sc[at] - mx);
              sc[at] = e;
              sum += e;
            }
            const float inv = __fdiv_rn(1.0f, wave_sum_f(sum));
            for (unsigned at = lane; at < S; at += kWave) sc[at] *= inv;
          }
          const float* sc = mine_sc + (hs >= 5 ? 0u : (4u * (lane % 8)) >> hs) * S;
          f4 acc = {0.f, 0.f, 0.f, 0.f};
          for (unsigned s0 = 0; s0 < S; s0 += kTrips * SG) {
            if (s0 != 0) values(s0);
#pragma unroll
            for (int j = 0; j < kTrips; ++j) {
              const unsigned at = s0 + j * SG + sg % SG;
              const float w = sc[min(at, S - 1)];
#pragma unroll
              for (int t = 0; t < 4; ++t) acc[t] = at < S ? fmaf(w, va[j][t], acc[t]) : acc[t];
            }
          }
          f4 ctx = acc;
#pragma unroll
          for (unsigned g = 1; g < SG; ++g)
#pragma unroll
            for (int t = 0; t < 4; ++t) ctx[t] += __shfl(acc[t], g * 8 + lane % 8, kWave);
          if (lane < 8)
#pragma unroll
            for (int t = 0; t < 4; ++t) publish(p.ctx + row * d + r * 32 + 4 * lane + t, ctx[t]);
        }
        ok = agree(came, 0.f);
      });
    // ---- o = Wo ctx
    if (ok && narrow) {
      f4 c[CD];
      ok = wave >= M || poll_row(p.ctx + (size_t)row * d, d, c, patience);
      ok = agree(ok, wave < M ? row_absmax(c) : 0.f);
      if (ok) {
        const float s = amax > 0.0f ? __fdiv_rn(127.0f, amax) : 1.0f;
        put(c, d, s);
        __syncthreads();
        const float u = __fdiv_rn(1.0f, __fmul_rn(s, so));
        product(wo, p.wo, d, nd, p.bo, bo, [&](unsigned r, int sum, float b) {
          if (em < M) publish(p.o + em * d + r * 32 + lj, fmaf((float)sum, u, b));
        });
      }
    }
    // ---- y2 = LN(o + y1), hid2 = relu(W1 y2)
    u4 wf2[CW];
    row_of(gv, p.gamma2, d);
    row_of(bv, p.beta2, d);
    if (narrow0) fetch(wf2, p.w2, role0, p.ffn);
    __builtin_amdgcn_sched_barrier(0);
    if (ok) {
      ok = wave >= M || poll_row(p.o + (size_t)row * d, d, y2, patience);
      if (ok) normalise(y2, y1, gv, bv, p.eps);
      ok = agree(ok, wave < M ? row_absmax(y2) : 0.f);
      if (ok) {
        const float s = amax > 0.0f ? __fdiv_rn(127.0f, amax) : 1.0f;
        put(y2, d, s);
        __syncthreads();
        const float u = __fdiv_rn(1.0f, __fmul_rn(s, s1));
        product(w1, p.w1, d, nf, p.b1, b1, [&](unsigned r, int sum, float b) {
          const float v = fmaf((float)sum, u, b);
          if (em < M) publish(p.hid2 + (size_t)em * p.ffn + r * 32 + lj, v > 0.0f ? v : 0.0f);
        });
      }
    }
    // ---- ff = W2 hid2
    if (ok && narrow) {
      f4 h2[CW];
      ok = wave >= M || poll_row(p.hid2 + (size_t)row * p.ffn, p.ffn, h2, patience);
      ok = agree(ok, wave < M ? row_absmax(h2) : 0.f);
      if (ok) {
        const float s = amax > 0.0f ? __fdiv_rn(127.0f, amax) : 1.0f;
        put(h2, p.ffn, s);
        __syncthreads();
        const float u = __fdiv_rn(1.0f, __fmul_rn(s, s2));
        product(wf2, p.w2, p.ffn, nd, p.b2, b2, [&](unsigned r, int sum, float b) {
          if (em < M) publish(p.ff + em * d + r * 32 + lj, fmaf((float)sum, u, b));
        });
      }
    }
    // ---- y = LN(ff + y2)
    if (ok && owns_below(1)) {
      row_of(gv, p.gamma3, d);
      row_of(bv, p.beta3, d);
      f4 v[CD];
      ok = wave >= M || poll_row(p.ff + (size_t)row * d, d, v, patience);
      if (ok) normalise(v, y2, gv, bv, p.eps);
      ok = agree(ok, 0.f);
      if (ok && wave < M)
#pragma unroll
        for (int c = 0; c < CD; ++c) reinterpret_cast<f4*>(p.y + (size_t)row * d)[c * 64 + lane] = v[c];
    }
    return ok;
  };
  if (pass(std::true_type{})) return;
  unsigned tries = 0;                                            // passes begun with every role claimed
  do {
    // Some row did not come.  Roles nobody has claimed are taken over and everything begins again; once all are claimed it
    // is a matter of time, and of kTries passes that wait for it: one may find its time gone because the process was not
    // running, the next begins its own.  After those role 0's workgroup does the whole layer, which waits for nobody, and
    // the others end.
    __syncthreads();
    if (tries > kTries) {                                        // (its own stores did not come back to it)
      const float nan = __builtin_nanf("");
      if (wave < M)
#pragma unroll
        for (int c = 0; c < CD; ++c) reinterpret_cast<f4*>(p.y + (size_t)row * d)[c * 64 + lane] = f4{nan, nan, nan, nan};
      return;
    }
    if (tid == 0) {
      unsigned taken = 0, left = 0;
      if (tries < kTries) {
        for (unsigned r = 0; r < p.roles; ++r) {
          if (__hip_atomic_load(p.claim + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != kUnsetWord) continue;
          if (taken < kTake && __hip_atomic_exchange(p.claim + r, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == kUnsetWord)
            owned[n_owned + taken++] = r;
          else
            left = 1;
        }
        n_owned += taken;
      } else {
        bool writer = false;
        for (unsigned i = 0; i < n_owned; ++i) writer = writer || owned[i] == 0;
        n_owned = writer ? p.roles : 0;
        for (unsigned r = 0; r < n_owned; ++r) owned[r] = r;
      }
      some_left = left;
    }
    __syncthreads();
    count = __builtin_amdgcn_readfirstlane(n_owned);
    if (count == 0) return;
    if (__builtin_amdgcn_readfirstlane(some_left) == 0u) patience = tries++ < kTries ? p.limit : kLongest;
    // (a new value each time for the compiler, or it keeps every phase's addresses in registers across the loop)
    asm volatile("" : "+v"(tid));
    lane = tid % 64; lj = lane % 32; lh = lane / 32;
    wave = __builtin_amdgcn_readfirstlane(tid / 64);
    row = min(wave, M - 1);
    em = 4 * lh + wave;
  } while (!pass(std::false_type{}));
}

}  // namespace

// A layer of up to eight rows, microseconds in a captured graph, nine launches and two: 33.8 and 23.3 at 512 / 2048 and one
// sentence of 25 words (eight sentences 35.9 and 29.0), 51.6 and 32.9 at 1024 / 4096 (54.8 and 40.3), 28.1 and 21.3 at
// 256 / 1024 (29.6 and 26.4).  Of the 18 us of this launch at one sentence 2.1 go by before the first rows are there, 0.8 to 1.7 for
// each of seven exchanges, 1 in the attention, 0.6 to 1.3 for the quantization and product of a phase.  With the attention
// of a sentence in one workgroup, all heads, it was 24.5 and 29.8, 35.4 and 43.2, 21.1 and 25.7.  The widths are those with
// a vector of the row per lane and 256 registers of parameters ahead; the head widths and scores those of the attention kernel
// this replaces, with room for eight sentences' scores of 512 words; more rows than waves take the launches.
bool layer_rows_supported(size_t M, size_t S, size_t d, size_t aan, size_t ffn, int heads) {
  if (M < 1 || M > (size_t)kLW || (d != 256 && d != 512 && d != 1024)) return false;
  const size_t widest = d == 1024 ? 4096 : 2048, dh = d / (size_t)heads;
  if (aan % 64 != 0 || ffn % 64 != 0 || aan > widest || ffn > widest || aan < 64 || ffn < 64) return false;
  if (S > 512 || d % (size_t)heads != 0 || (dh & (dh - 1)) != 0 || dh < 4 || dh > 256 || (size_t)heads * S > 4096) return false;
  // What the launches cost more, in microseconds (more with wide inner products, less with many rows), against what the
  // attention costs more here.  One wave walks through a sentence's positions for its 32 columns: a head wider than those has
  // its keys read once per 32 columns, narrower ones come one after the other, where the attention launch spreads a sentence
  // over a workgroup.  Nine launches and two, us: eight sentences of 512 / 2048 with heads of 128 columns, 192 words 43.8 and 41.9,
  // 256 words 46.1 and 47.4; of 256 columns, 64 words 39.0 and 37.3, 96 words 40.4 and 42.0, 256 words 47.1 and 68.6; of 256 /
  // 1024 with one head, 32 words 29.1 and 28.8, 48 words 29.7 and 30.8; of 256 / 256 with heads of 64, 192 words 31.0 and 30.5,
  // 320 words 33.9 and 35.0; of 4, 8 words 29.1 and 33.1; one sentence of 512 / 2048 with heads of 64, 512 words 50.5 and 39.6;
  // of 1024 / 4096 with heads of 256, 192 words 65.2 and 57.8, eight sentences 69.6 and 72.2.
  const float launches = 1.0f + (float)(aan + ffn) / 700.0f + 0.5f * (float)(kLW - (int)M);
  constexpr float kPosition[3][3] = {{0.009f, 0.038f, 0.12f}, {0.009f, 0.035f, 0.105f}, {0.009f, 0.024f, 0.085f}};      // wide heads
  const float attention = dh >= 64 ? kPosition[d / 512][dh / 128] * (float)S : (32.0f / (float)dh - 1.0f) * 240.0f / (float)d - 0.16f * (float)S / (float)dh;
  return attention <= launches;
}

int launch_layer_rows(const mq_aan_layer& P, const float* x, const float* hid, const float* K, const float* V, size_t M, size_t S,
                      int heads, float eps, const LayerExchange& e, float* y, hipStream_t s) {
  LayerParams p{};
  auto bytes = [](const mq_product& w) { return static_cast<const uint8_t*>(w.packed); };
  p.wa2 = bytes(P.aan_ffn2); p.wg = bytes(P.aan_gate); p.wq = bytes(P.ctx_q); p.wo = bytes(P.ctx_o); p.w1 = bytes(P.ffn1); p.w2 = bytes(P.ffn2);
  p.sa2 = P.aan_ffn2.scale; p.sg = P.aan_gate.scale; p.sq = P.ctx_q.scale; p.so = P.ctx_o.scale; p.s1 = P.ffn1.scale; p.s2 = P.ffn2.scale;
  p.ba2 = P.aan_ffn2.bias; p.bg = P.aan_gate.bias; p.bq = P.ctx_q.bias; p.bo = P.ctx_o.bias; p.b1 = P.ffn1.bias; p.b2 = P.ffn2.bias;
  p.gamma1 = P.ln1.gamma; p.beta1 = P.ln1.beta; p.gamma2 = P.ln2.gamma; p.beta2 = P.ln2.beta; p.gamma3 = P.ln3.gamma; p.beta3 = P.ln3.beta;
  p.x = x; p.hid = hid; p.K = K; p.V = V;
  p.f = e.f; p.mix = e.mix; p.q = e.q; p.ctx = e.ctx; p.o = e.o; p.hid2 = e.hid2; p.ff = e.ff; p.claim = e.claim;
  p.y = y;
  p.M = (unsigned)M; p.S = (unsigned)S; p.heads = (unsigned)heads; p.aan = (unsigned)P.aan_ffn; p.ffn = (unsigned)P.ffn;
  while (((unsigned)P.d / p.heads >> p.head_shift) > 1) ++p.head_shift;
  p.eps = eps;
  const unsigned nd = (unsigned)P.d / 32, nf = (unsigned)P.ffn / 32;
  p.roles = nf > nd ? nf : nd;
  const unsigned long long limit = barrier_timeout_ticks();
  // 30 us, and what the attention may take (without it the workgroups that have no part in it began again in the meantime:
  // one sentence of 1024 / 4096, 192 words, heads of 256 columns 74.8 us, with it 57.8)
  const unsigned soon = 3000u + (unsigned)(S * (size_t)P.d / (size_t)heads / 8);
  p.patience = limit < soon ? (unsigned)limit : soon;
  p.limit = limit < kLongest ? (unsigned)limit : kLongest;
  const dim3 grid(p.roles), block(kLT);
  if (P.d == 256) hipLaunchKernelGGL((k_layer_rows<1, 8>), grid, block, 0, s, p);
  else if (P.d == 512) hipLaunchKernelGGL((k_layer_rows<2, 8>), grid, block, 0, s, p);
  else hipLaunchKernelGGL((k_layer_rows<4, 16>), grid, block, 0, s, p);
  return check_hip(hipGetLastError());
}

}  // namespace mq
