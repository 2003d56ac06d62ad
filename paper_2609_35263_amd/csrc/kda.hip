// gfx950 (CDNA4) kernel of libwavepp_attn: chunked prefill of a KDA (gated delta-rule) layer that
// resumes from a recurrent-state snapshot and leaves the snapshot at the chunk boundary.
//
// Per head, with per-channel decay alpha_t, write strength beta_t, key k_t, value v_t, query q_t
// (Preliminaries, "Transformer Architectures", Eq. 2-3):
//   S_t = (I - beta_t k_t k_t^T) Diag(alpha_t) S_{t-1} + beta_t k_t v_t^T,   o_t = S_t^T q_t.
//
// Chunkwise form.  Tokens are processed in blocks of C = 64.  Inside a block, with S0 the state
// before it and gamma_t = alpha_1 * ... * alpha_t (per channel, running product from the block
// start), write the state change of token t as k_t u_t^T.  Unrolling the recurrence gives
//   u_t = beta_t (v_t - S0^T (gamma_t * k_t) - sum_{s<t} u_s <k_s / gamma_s, gamma_t * k_t>),
// i.e. (I + A) U = Diag(beta) (V - K~ S0) with K~ = gamma * K and the strictly lower-triangular
// A[t][s] = beta_t <gamma_t * k_t, k_s / gamma_s>.  With T = (I + A)^-1 and R = Diag(beta)(V - K~ S0):
//   U = T R,
//   O = Q~ S0 + P U,              Q~ = gamma * Q,  P[t][s] = <gamma_t * q_t, k_s / gamma_s> (s <= t),
//   S_C = Diag(gamma_C) S0 + Kbar^T U,   Kbar_s = k_s * gamma_C / gamma_s.
// Every product of 64-token blocks with the 128 x 128 state is a bf16 MFMA contraction with fp32
// accumulation; the state itself stays in fp32 accumulators for the whole chunk.
//
// Range.  The factorization gamma_t / gamma_s = gamma_t * (1 / gamma_s) is used for a channel only
// when its block decay gamma_C is at least 2^-96, so every factor stays a normal number.  Kbar is
// built from products of the later decays (gamma_C / gamma_s without a division) and
// 1 / gamma_s = (gamma_C / gamma_s) / gamma_C, one reciprocal per channel and block.  A
// channel that decays more within one block (including alpha = 0) is "slow": it contributes to A
// and P through an exact pairwise term exp2(G_t - G_s) in log2 space instead, and its Kbar uses
// exp2(G_C - G_s).
//
// Workgroup = 8 waves on one CU, running (request, head) chains one after another, one 64-token block
// at a time.  The work of a block falls into two parts that different waves run at the same time, one
// block apart:
//   * Waves 0-3 (builders) make everything that does not depend on the state, one block ahead: the
//     decays, the scaled operands, A, P and T.
//   * Waves 4-7 (runners) carry the state.  Runner w owns state columns [32w, 32w + 32) as four
//     32 x 32 fp32 accumulator tiles.  The accumulator layout of v_mfma_f32_32x32x16_bf16 (lane =
//     column, 16 rows per lane) is reused directly as the B operand of the next contraction: the eight
//     rows a lane holds for one MFMA are its contraction slots, and the A operand is read from LDS in
//     that same (permuted) order.
// Every step of either part is a latency chain (LDS round trips, short dependent products), so two
// waves per SIMD in different parts hide each other's waits.  A wave of 4 x 64 heads x 4,096 tokens:
// 510 us with four waves that ran the parts in turn, 357-379 us now over cards, 4.3-4.6 TB/s where a plain copy
// reached 4.9; with 64 chains on 256 CUs (one 16,384-token request) it is the builders' chain, 10.7 K
// cycles a block, that bounds it (1,951 -> 1,144 us).  All eight waves in the scaling phase, the P tiles
// given to the runners, and the next block's loads anywhere but row by row in the scaling phase were
// slower.  A period has six workgroup barriers (more with slow channels); both loops below pass each of
// them once per block built:
//     barrier      builders (block n + 1)                   runners (block n)
//     .. 1         octet decay products
//     .. 2         Q~, K~, K_R, Kbar of the block           U = T R, O += P U, state update
//     .. 3         A, P                                     outputs to memory, V of block n + 1 to LDS
//     .. 4, 5, 6   T in three steps                         K~ S0 and Q~ S0 of block n + 1
// Q~, K~, P and T are single buffers: a period reads block n's before the barrier after which block
// n + 1's are written.  Kbar, gamma_C and beta are read later than that and have two.
#include <hip/hip_runtime.h>

#include "internal.h"

#include <algorithm>

namespace wavepp {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;

constexpr int kC = kKdaBlock;       // tokens per block
constexpr int kD = kKdaDim;         // d_k = d_v
// LDS row strides.  The LDS has 64 banks of 4 bytes.  A permuted A-operand read (lds_a_perm) has the
// 32 lanes of a half-wave read 8 bytes each from 32 consecutive rows: with a row stride that is an odd
// multiple of 8 bytes modulo 256 those land on 32 distinct bank pairs.  Arrays read that way keep
// rows only 8-byte aligned and are accessed 8 bytes at a time.
constexpr int RS = kD + 8;          // bf16 row stride of K_R (16-byte accesses)
constexpr int QS = kD + 4;          // bf16 row stride of Q~ and K~: 264 B
constexpr int VW = 32;              // bf16 row stride of a runner's columns of V: the 4 rows x 64 B of a
                                    // transposing read are 256 consecutive bytes
constexpr int CS = kC + 4;          // bf16 row stride of [channel][t] arrays and of P, T [t][s]: 136 B
constexpr int AS = kC + 4;          // fp32 row stride of A and of T during the inversion
constexpr int kSlowBatch = 16;      // slow channels staged per pass
constexpr float kFastFloor = 0x1p-96f;
constexpr float kLogFloor = -1000.0f;   // log2 of a zero decay: exp2 of it is exactly 0 in fp32

struct KdaLds {
  __bf16 qt[kC * QS];               // Q~ = gamma * q          [t][c]
  __bf16 kt[kC * QS];               // K~ = gamma * k          [t][c]
  union {
    __bf16 kr[kC * RS];             // K_R = k / gamma (0 for slow channels)   [t][c]
    float tf[kC * AS];              // T = (I + A)^-1 in fp32 while it is built
  };
  __bf16 kbt[2][kD * CS];           // Kbar^T                  [c][t]
  __bf16 vt[4][kC * VW];            // per runner: its columns of V [t][j]
  union {
    float a[kC * AS];               // A (beta-scaled, strictly lower)
    struct {                        // slow channels of one batch, log2-space
      float g[kSlowBatch][kC];
      float k[kSlowBatch][kC];
      float q[kSlowBatch][kC];
    } slow;
  };
  __bf16 pm[kC * CS];               // P (lower incl. diagonal)
  __bf16 tm[kC * CS];               // T in bf16; the 16-blocks above the diagonal stay zero
  float beta[2][kC];
  float gc[2][kD];                  // gamma_C per channel
  float qtot[8][kD];                // per-octet decay products
  int slow_list[kD];
  int nslow;
};

__device__ __forceinline__ bool kda_meta_ok(const KdaDevPlan& p) {
  return p.hdr->magic == kKdaMagic && p.hdr->serial == p.serial;
}

__device__ __forceinline__ float bf_lo(uint32_t x) { return __uint_as_float(x << 16); }
__device__ __forceinline__ float bf_hi(uint32_t x) { return __uint_as_float(x & 0xFFFF0000u); }

__device__ __forceinline__ bf16x8 cat(bf16x4 a, bf16x4 b) {
  return bf16x8{a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
}

// A operand whose 8 contraction slots of half-wave hf are the columns base + {0..3, 8..11} of
// row `row` (base already includes 4 * hf): the order in which an accumulator holds them.
__device__ __forceinline__ bf16x8 lds_a_perm(const __bf16* rowp, int base) {
  return cat(*reinterpret_cast<const bf16x4*>(rowp + base), *reinterpret_cast<const bf16x4*>(rowp + base + 8));
}

// Registers 8kk .. 8kk+7 of an accumulator tile, rounded to bf16: a B operand in permuted order.
__device__ __forceinline__ bf16x8 acc_to_b(const f32x16& acc, int kk) {
  bf16x8 r;
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = static_cast<__bf16>(acc[8 * kk + e]);
  return r;
}

__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Transposing LDS read: within each group of 16 lanes, lane i receives element i%4 of the 8 bytes
// addressed by lanes 4m + i/4, m = 0..3.
__device__ __forceinline__ bf16x4 lds_read_tr(const __bf16* p) {
  const i16x4 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(p));
  return __builtin_bit_cast(bf16x4, r);
}

// Workgroup barrier for LDS traffic only.  __syncthreads() also drains every outstanding global
// load of the wave (its release fence covers all memory), which would stall on the next block's
// prefetch; every exchange between waves here goes through LDS, so draining this wave's LDS
// operations before the barrier is enough.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <typename T>
__device__ __forceinline__ T const_load(const T* ptr) {
  // scalar load: the metadata is never written by this kernel
  return *((const __attribute__((address_space(4))) T*)(ptr));
}

// Position in a workgroup's run: block [blk, blk + 64) of one (request, head) chain.  Chains of unlike lengths are
// listed by workgroup after the items, by load (kListed); of like ones workgroup w of G takes chains w, 2G - 1 - w,
// 2G + w, ...  Two kernels: a single-block launch takes 0.4 us longer with the choice made in the kernel.
template <bool kListed>
struct Cursor {
  int round = 0, end = 0;        // place of the chain in the list and the end of the workgroup's part; or its round
  int blk = 0, head = 0;
  int cu = 0, len = 0, state_in = -1, state_out = -1;   // of the chain's item
  bool valid = false;

  static __device__ __forceinline__ const int32_t* list(const KdaDevPlan& p) {
    return reinterpret_cast<const int32_t*>(p.items + p.num_items);
  }
  __device__ __forceinline__ void start(const KdaDevPlan& p) {
    if (kListed) {
      round = const_load(list(p) + blockIdx.x);
      end = const_load(list(p) + blockIdx.x + 1);
    }
    open(p);
  }
  __device__ __forceinline__ void open(const KdaDevPlan& p) {
    int c;
    if (kListed) {
      valid = round < end;
      if (!valid) return;
      c = const_load(list(p) + round);
    } else {
      const int G = gridDim.x;
      c = round * G + ((round & 1) ? G - 1 - int(blockIdx.x) : int(blockIdx.x));
      valid = c < p.num_items * p.num_heads;
      if (!valid) return;
    }
    const int item = c / p.num_heads;
    head = c - item * p.num_heads;
    const auto* it = (const __attribute__((address_space(4))) KdaItem*)(p.items + item);
    cu = it->cu;
    len = it->len;
    state_in = it->state_in;
    state_out = it->state_out;
    blk = 0;
  }
  __device__ __forceinline__ bool last() const { return blk + kC >= len; }
  __device__ __forceinline__ void advance(const KdaDevPlan& p) {
    if (last()) {
      ++round;
      open(p);
    } else {
      blk += kC;
    }
  }
  __device__ __forceinline__ int rows() const { return min(kC, len - blk); }
  __device__ __forceinline__ int64_t tok0() const { return int64_t(cu) + blk; }
};

// Raw inputs of one block, as loaded by one builder thread: channels 4 cq .. 4 cq + 3 of tokens
// 8 oc .. 8 oc + 7 (alpha, k, q) and one beta.  Rows past the block's last token are not read: they keep
// what the registers held and are replaced by neutral values (alpha = 1, k = q = 0, beta = 0) when they
// are consumed.  The next block's rows are loaded as this block's are used up, one per step of the
// operand scaling: it is the phase with the most ALU work, and no burst fills the memory request queue.
struct RawBlock {
  float4 a[8];
  uint2 k[8], q[8];
  float b;
};

struct RawLoader {
  const float* a;
  const __bf16 *k, *q;
  const float* b;
  int rows, brows;               // rows left of this thread's octet, of the block from this thread's beta row on

  template <bool kListed>
  __device__ __forceinline__ void open(const float* alpha, const __bf16* kp, const __bf16* qp, const float* beta,
                                       const Cursor<kListed>& c, int H, int tid) {
    const int cq = tid & 31, oc = tid >> 5;
    const int64_t at = (c.tok0() + 8 * oc) * (int64_t(H) * kD) + int64_t(c.head) * kD + 4 * cq;
    a = alpha + at;
    k = kp + at;
    q = qp + at;
    b = beta + (c.tok0() + (tid & 63)) * H + c.head;
    rows = c.valid ? c.rows() - 8 * oc : 0;
    brows = c.valid ? c.rows() - (tid & 63) : 0;
  }
  __device__ __forceinline__ void row(RawBlock& r, int i, int64_t tok_stride) const {
    if (i < rows) {
      r.a[i] = *reinterpret_cast<const float4*>(a + i * tok_stride);
      r.k[i] = *reinterpret_cast<const uint2*>(k + i * tok_stride);
      r.q[i] = *reinterpret_cast<const uint2*>(q + i * tok_stride);
    }
  }
  __device__ __forceinline__ void write_strength(RawBlock& r) const {
    if (brows > 0) r.b = *b;
  }
};

// Element (c, t) of Kbar^T in LDS.  A builder thread writes four tokens of channels 4 cq + e, lanes 544
// bytes apart: the XOR of the 8-byte unit with c / 32 spreads the four lanes that would share a bank pair.
// A runner's read of 32 consecutive channels sees a constant XOR.
__device__ __forceinline__ int kbt_at(int c, int t) { return c * CS + (t ^ ((c >> 5) << 2)); }

// Fence for the scheduler: reads, products and stores stay on their side, ALU work may cross.
__device__ __forceinline__ void keep_order() { __builtin_amdgcn_sched_barrier(0x6); }

template <bool kListed>
__device__ __forceinline__ void build_blocks(const KdaDevPlan& p, KdaLds& ls, const __bf16* __restrict__ q,
                                             const __bf16* __restrict__ k, const float* __restrict__ alpha,
                                             const float* __restrict__ beta, int wave, int tid) {
  const int lane = tid & 63, col = lane & 31, hf = lane >> 5;
  const int H = p.num_heads;
  const int64_t tok_stride = int64_t(H) * kD;           // elements between tokens of one head
  const int cq = tid & 31, oc = tid >> 5;               // channels 4 cq + e, tokens 8 oc + i
  Cursor<kListed> cur;
  cur.start(p);
  RawBlock raw;
  RawLoader ld;
  ld.open(alpha, k, q, beta, cur, H, tid);
#pragma unroll
  for (int i = 0; i < 8; ++i) ld.row(raw, i, tok_stride);
  ld.write_strength(raw);
  for (int buf = 0; cur.valid; buf ^= 1) {
    const int L = cur.rows();
    const int64_t tok0 = cur.tok0();
    const int64_t head_off = int64_t(cur.head) * kD;
    Cursor<kListed> nxt = cur;
    nxt.advance(p);

    // ---- decays -------------------------------------------------------------------------------
    float g[8][4];                 // running decay product within the octet, inclusive
    float sfx[8][4];               // decay product of the later tokens of the octet, exclusive
    if (L < kC) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (8 * oc + i >= L) {     // rows past the end: neutral
          raw.a[i] = make_float4(1.0f, 1.0f, 1.0f, 1.0f);
          raw.k[i] = make_uint2(0, 0);
          raw.q[i] = make_uint2(0, 0);
        }
    }
    {
      float run[4] = {1.0f, 1.0f, 1.0f, 1.0f}, back[4] = {1.0f, 1.0f, 1.0f, 1.0f};
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float ai[4] = {raw.a[i].x, raw.a[i].y, raw.a[i].z, raw.a[i].w};
        const float aj[4] = {raw.a[7 - i].x, raw.a[7 - i].y, raw.a[7 - i].z, raw.a[7 - i].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          run[e] *= ai[e];
          g[i][e] = run[e];
          sfx[7 - i][e] = back[e];
          back[e] *= aj[e];
        }
      }
      *reinterpret_cast<float4*>(&ls.qtot[oc][4 * cq]) = make_float4(run[0], run[1], run[2], run[3]);
      if (tid < kC) ls.beta[buf][tid] = tid < L ? raw.b : 0.0f;
    }
    lds_barrier();   // 1

    // ---- scaled operands ----------------------------------------------------------------------
    // Products over the octets: every thread forms gamma_C = tot in the same order (the choice of slow
    // channels has to agree between the waves); pre and post are those before and after its own octet,
    // the lower or the upper of its wave's two.
    f32x4 x[8];
#pragma unroll
    for (int o = 0; o < 8; ++o) x[o] = *reinterpret_cast<const f32x4*>(&ls.qtot[o][4 * cq]);
    f32x4 tot = x[0], pre = {1.0f, 1.0f, 1.0f, 1.0f}, post = pre, own_lo = x[0], own_hi = x[1];
#pragma unroll
    for (int o = 1; o < 8; ++o) {
      if (o < 7 && o == 2 * wave) {
        pre = tot;
        own_lo = x[o];
        own_hi = x[(o + 1) & 7];
      }
      tot *= x[o];
    }
#pragma unroll
    for (int o = 7; o > 1; --o)
      if (o > 2 * wave + 1) post *= x[o];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      pre[e] = hf ? pre[e] * own_lo[e] : pre[e];
      post[e] = hf ? post[e] : post[e] * own_hi[e];
    }
    // gamma_t = pre * g, gamma_C / gamma_t = sfx * post (a product of the later decays, no division),
    // and k / gamma_t = (k gamma_C / gamma_t) / gamma_C: one reciprocal per channel
    bool slow[4];
    float rcp[4];                  // post / gamma_C
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      slow[e] = !(tot[e] >= kFastFloor);
      post[e] = slow[e] ? 0.0f : post[e];
      rcp[e] = slow[e] ? 0.0f : post[e] * __frcp_rn(tot[e]);
    }
    {
      __bf16 kb[4][8];
      ld.open(alpha, k, q, beta, nxt, H, tid);
      ld.write_strength(raw);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int t = 8 * oc + i;
        const float kf[4] = {bf_lo(raw.k[i].x), bf_hi(raw.k[i].x), bf_lo(raw.k[i].y), bf_hi(raw.k[i].y)};
        const float qf[4] = {bf_lo(raw.q[i].x), bf_hi(raw.q[i].x), bf_lo(raw.q[i].y), bf_hi(raw.q[i].y)};
        bf16x4 vq, vk, vr;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float gm = pre[e] * g[i][e];
          vq[e] = static_cast<__bf16>(qf[e] * gm);
          vk[e] = static_cast<__bf16>(kf[e] * gm);
          const float ks = kf[e] * sfx[i][e];
          vr[e] = static_cast<__bf16>(ks * rcp[e]);
          kb[e][i] = static_cast<__bf16>(ks * post[e]);
        }
        *reinterpret_cast<bf16x4*>(&ls.qt[t * QS + 4 * cq]) = vq;
        *reinterpret_cast<bf16x4*>(&ls.kt[t * QS + 4 * cq]) = vk;
        *reinterpret_cast<bf16x4*>(&ls.kr[t * RS + 4 * cq]) = vr;
        ld.row(raw, i, tok_stride);
        keep_order();
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        *reinterpret_cast<bf16x4*>(&ls.kbt[buf][kbt_at(4 * cq + e, 8 * oc)]) = bf16x4{kb[e][0], kb[e][1], kb[e][2], kb[e][3]};
        *reinterpret_cast<bf16x4*>(&ls.kbt[buf][kbt_at(4 * cq + e, 8 * oc + 4)]) = bf16x4{kb[e][4], kb[e][5], kb[e][6], kb[e][7]};
      }
      if (oc == 0) *reinterpret_cast<float4*>(&ls.gc[buf][4 * cq]) = make_float4(tot[0], tot[1], tot[2], tot[3]);
    }
    // compact list of the slow channels, in channel order (lanes 0-31 of every wave see all channels)
    int nslow = 0;
    if (__ballot(slow[0] || slow[1] || slow[2] || slow[3])) {
      const uint64_t lo32 = (lane < 32) ? ((lane == 0) ? 0ull : (~0ull >> (64 - lane))) : 0ull;
      int below = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint64_t b = __ballot(slow[e] && lane < 32);
        below += __popcll(b & lo32);
        nslow += __popcll(b);
      }
      if (wave == 0 && lane < 32) {
        int idx = below;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (slow[e]) ls.slow_list[idx++] = 4 * cq + e;
      }
    }
    if (tid == 0) ls.nslow = nslow;
    lds_barrier();   // 2

    // ---- A and P (waves 0-2: tiles (0,0), (1,0), (1,1)) ------------------------------------------
    const int tb1 = wave == 0 ? 0 : 1, sb1 = wave == 2 ? 1 : 0;
    // transposed tiles (rows s, lane = row t of A and P), so that a lane writes four consecutive s at once
    f32x16 accA = {}, accP = {};
    if (wave < 3) {
      // the operands of step kc + 3 are read while step kc's two products run
      const __bf16* kp = &ls.kt[(32 * tb1 + col) * QS + 8 * hf];
      const __bf16* qp = &ls.qt[(32 * tb1 + col) * QS + 8 * hf];
      const __bf16* rp = &ls.kr[(32 * sb1 + col) * RS + 8 * hf];
      auto ld4 = [](const __bf16* p) { return cat(*reinterpret_cast<const bf16x4*>(p), *reinterpret_cast<const bf16x4*>(p + 4)); };
      bf16x8 ak[3], aq[3], b[3];
#pragma unroll
      for (int kc = 0; kc < kD / 16 + 3; ++kc) {
        if (kc >= 3) {
          accA = mfma(b[kc % 3], ak[kc % 3], accA);
          accP = mfma(b[kc % 3], aq[kc % 3], accP);
        }
        if (kc < kD / 16) {
          ak[kc % 3] = ld4(kp + 16 * kc);
          aq[kc % 3] = ld4(qp + 16 * kc);
          b[kc % 3] = *reinterpret_cast<const bf16x8*>(rp + 16 * kc);
        }
        keep_order();
      }
    }
    // slow channels: exact pairwise terms in log2 space, 16 channels per batch, re-read from memory
    for (int base = 0; base < nslow; base += kSlowBatch) {
      lds_barrier();
      const int cl = tid >> 4, tg = tid & 15;
      const bool have = base + cl < nslow;
      const int ch = have ? ls.slow_list[base + cl] : 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int t = 4 * tg + u;
        float lg = 0.0f, kv = 0.0f, qv = 0.0f;
        if (have && t < L) {
          const int64_t idx = (tok0 + t) * tok_stride + head_off + ch;
          const float a1 = alpha[idx];
          lg = a1 > 0.0f ? fmaxf(__log2f(a1), kLogFloor) : kLogFloor;
          kv = static_cast<float>(k[idx]);
          qv = static_cast<float>(q[idx]);
        }
        ls.slow.g[cl][t] = lg;
        ls.slow.k[cl][t] = kv;
        ls.slow.q[cl][t] = qv;
      }
      lds_barrier();
      if (tid < kSlowBatch) {
        float run = 0.0f;
        for (int t = 0; t < kC; ++t) {
          run += ls.slow.g[tid][t];
          ls.slow.g[tid][t] = run;
        }
      }
      lds_barrier();
      if (have) {
        const float gC = ls.slow.g[cl][kC - 1];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int t = 4 * tg + u;
          ls.kbt[buf][kbt_at(ch, t)] = static_cast<__bf16>(ls.slow.k[cl][t] * exp2f(gC - ls.slow.g[cl][t]));
        }
      }
      if (wave < 3) {
        const int nb = min(kSlowBatch, nslow - base);
        const int t = 32 * tb1 + col;
        for (int c = 0; c < nb; ++c) {
          const float gt = ls.slow.g[c][t], kt = ls.slow.k[c][t], qt = ls.slow.q[c][t];
#pragma unroll
          for (int reg = 0; reg < 16; ++reg) {
            const int s = 32 * sb1 + 8 * (reg >> 2) + 4 * hf + (reg & 3);
            const float e = exp2f(fminf(gt - ls.slow.g[c][s], 0.0f)) * ls.slow.k[c][s];
            accA[reg] += kt * e;
            accP[reg] += qt * e;
          }
        }
      }
    }
    if (nslow > 0) lds_barrier();   // the batch scratch shares storage with A
    if (wave < 3) {
      int t = 32 * tb1 + col;
      const float bt = ls.beta[buf][t];
      asm volatile("" : "+v"(t));   // the comparisons stay here: hoisted, their masks spill
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int s0 = 32 * sb1 + 8 * b + 4 * hf;
        f32x4 av;
        bf16x4 pv;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          av[r] = s0 + r < t ? accA[4 * b + r] * bt : 0.0f;
          pv[r] = static_cast<__bf16>(s0 + r <= t ? accP[4 * b + r] : 0.0f);
        }
        *reinterpret_cast<f32x4*>(&ls.a[t * AS + s0]) = av;
        *reinterpret_cast<bf16x4*>(&ls.pm[t * CS + s0]) = pv;
      }
    }
    lds_barrier();   // 3

    // ---- T = (I + A)^-1 -----------------------------------------------------------------------
    // Each wave owns one 16 x 16 diagonal block and needs no barrier for it: the two 8 x 8 halves by
    // substitution (every lane one column and one row of a half's inverse, from coefficients read once),
    // then T = D - D (L D) with D the halves' inverses and L the block's lower-left 8 x 8, on fp32
    // MFMAs.  16 -> 32 is the same product (fp32 MFMAs, one wave per pair), 32 -> 64 runs on bf16 MFMAs
    // split over the four waves.  A 16x16 accumulator (lane group g holds rows 4g + r) is the B operand
    // of the next product when its contraction slots are taken in that order.  The phase is a latency
    // chain, so the steps are few and wide: substitution over all 16 rows and the 16 -> 32 sums on the
    // VALU took 7,400 cycles a block, this 2,700 (4 x 64 heads x 4,096 tokens: 588 us, then 510).
    {
      const int a0 = 16 * wave, n16 = lane & 15, g16 = lane >> 4;
      const float* ab = &ls.a[a0 * AS + a0];
      float* tb = &ls.tf[a0 * AS + a0];
      const int s8 = lane & 8, jc = lane & 7;
      const f32x4 la = *reinterpret_cast<const f32x4*>(&ab[n16 * AS + 4 * g16]);
      f32x4 c[8][2];
#pragma unroll
      for (int t = 1; t < 8; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          if (4 * h < t) c[t][h] = *reinterpret_cast<const f32x4*>(&ab[(s8 + t) * AS + s8 + 4 * h]);
      float xc[8], xr[8];          // column jc and row jc of the half's inverse
#pragma unroll
      for (int t = 0; t < 8; ++t) xc[t] = xr[t] = (t == jc) ? 1.0f : 0.0f;
#pragma unroll
      for (int u = 0; u < 7; ++u)
#pragma unroll
        for (int t = u + 1; t < 8; ++t) {
          xc[t] -= c[t][u >> 2][u & 3] * xc[u];
          // row: T[jc][u'] -= T[jc][t'] A[t'][u'] with t' = 7 - u, u' = 7 - t descending
          xr[7 - t] -= c[7 - u][(7 - t) >> 2][(7 - t) & 3] * xr[7 - u];
        }
      // lane group g holds rows (columns) 4g + r: non-zero only inside the lane's own half
      const int part = g16 - (s8 >> 2);
      float da[4], db[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        db[r] = part == 0 ? xc[r] : part == 1 ? xc[4 + r] : 0.0f;
        da[r] = part == 0 ? xr[r] : part == 1 ? xr[4 + r] : 0.0f;
      }
      f32x4 lx = f32x4{}, ly = f32x4{};
      const bool low = s8 && g16 < 2;
#pragma unroll
      for (int r = 0; r < 4; ++r) lx = mfma_f32(low ? la[r] : 0.0f, db[r], lx);
#pragma unroll
      for (int r = 0; r < 4; ++r) ly = mfma_f32(da[r], lx[r], ly);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float t = db[r] - ly[r];
        tb[(4 * g16 + r) * AS + n16] = t;
        ls.tm[(a0 + 4 * g16 + r) * CS + a0 + n16] = static_cast<__bf16>(t);
      }
    }
    lds_barrier();   // 4
    if (wave & 1) {
      // 16 -> 32: T_ab = -D_a (A_ab D_b) for (a, b) = (1, 0) and (3, 2)
      const int a0 = 16 * wave, b0 = a0 - 16, n16 = lane & 15, g16 = lane >> 4;
      const f32x4 la = *reinterpret_cast<const f32x4*>(&ls.a[(a0 + n16) * AS + b0 + 4 * g16]);
      const f32x4 da = *reinterpret_cast<const f32x4*>(&ls.tf[(a0 + n16) * AS + a0 + 4 * g16]);
      float db[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) db[r] = ls.tf[(b0 + 4 * g16 + r) * AS + b0 + n16];
      f32x4 x = f32x4{}, y = f32x4{};
#pragma unroll
      for (int r = 0; r < 4; ++r) x = mfma_f32(la[r], db[r], x);
#pragma unroll
      for (int r = 0; r < 4; ++r) y = mfma_f32(da[r], x[r], y);
#pragma unroll
      for (int r = 0; r < 4; ++r) ls.tm[(a0 + 4 * g16 + r) * CS + b0 + n16] = static_cast<__bf16>(-y[r]);
    }
    lds_barrier();   // 5
    {
      // 32 -> 64: T21 = -T2 (A21 T1); wave -> 16 columns c0 and 16 rows r0 of T21
      const int n16 = lane & 15, g16 = lane >> 4, c0 = 16 * (wave & 1), r0 = 16 * (wave >> 1);
      const __bf16* t1 = &ls.tm[(8 * g16 + (n16 >> 2)) * CS + c0 + 4 * (n16 & 3)];
      const bf16x8 bop = cat(lds_read_tr(t1), lds_read_tr(t1 + 4 * CS));
      f32x4 x[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const float* ar = &ls.a[(32 + 16 * i + n16) * AS + 8 * g16];
        const f32x4 lo = *reinterpret_cast<const f32x4*>(ar), hi = *reinterpret_cast<const f32x4*>(ar + 4);
        bf16x8 aop;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          aop[e] = static_cast<__bf16>(lo[e]);
          aop[4 + e] = static_cast<__bf16>(hi[e]);
        }
        x[i] = mfma16(aop, bop, f32x4{});
      }
      const __bf16* t2 = &ls.tm[(32 + r0 + n16) * CS + 32 + 4 * g16];
      const bf16x8 aop = cat(*reinterpret_cast<const bf16x4*>(t2), *reinterpret_cast<const bf16x4*>(t2 + 16));
      bf16x8 xb;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        xb[e] = static_cast<__bf16>(x[0][e]);
        xb[4 + e] = static_cast<__bf16>(x[1][e]);
      }
      const f32x4 y = mfma16(aop, xb, f32x4{});
#pragma unroll
      for (int r = 0; r < 4; ++r) ls.tm[(32 + r0 + 4 * g16 + r) * CS + c0 + n16] = static_cast<__bf16>(-y[r]);
    }
    lds_barrier();   // 6
    cur = nxt;
  }
}

template <bool kListed>
__device__ __forceinline__ void run_blocks(const KdaDevPlan& p, KdaLds& ls, const __bf16* __restrict__ v,
                                           float* __restrict__ state_pool, __bf16* __restrict__ out, int wave, int lane) {
  const int col = lane & 31, hf = lane >> 5;
  const int H = p.num_heads;
  const int64_t tok_stride = int64_t(H) * kD;
  const int j0 = 32 * wave;                             // this wave's state columns
  const int mrow = lane >> 2, mpart = 8 * (lane & 3);   // 16-byte moves of V: rows mrow + 16 i
  const int64_t v_lane = mrow * tok_stride + j0 + mpart, o_lane = col * tok_stride + j0 + 8 * hf;
  __bf16* vt = ls.vt[wave];
  Cursor<kListed> cur, nxt;
  nxt.start(p);
  // state tile ib, register 4b + r: row i = 32 ib + 8 b + 4 hf + r, column j0 + col
  f32x16 S[4], accE[2], accO[2];
  bf16x8 uB[2][2];
  for (int buf = 1;; buf ^= 1) {   // block n has buffer buf, block n + 1 the other; the first pass has no block n
    u32x4 vraw[4] = {};
    if (nxt.valid) {
      lds_barrier();   // 1
      const __bf16* src = v + nxt.tok0() * tok_stride + int64_t(nxt.head) * kD + v_lane;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (mrow + 16 * i < nxt.rows()) vraw[i] = *reinterpret_cast<const u32x4*>(src + 16 * i * tok_stride);
    }
    if (cur.valid) {
      // U = T R with R = beta (V - E) (T lower-triangular: block row tb uses block columns sb <= tb).  T's
      // operands in the order (tb, sb, kk) = (0,0,0) (0,0,1) (1,0,0) (1,0,1) (1,1,0) (1,1,1), V and beta are
      // read before any is used.  V[t0 + r][j] for r = 0..3 comes from the transposing read: lane 4m + g
      // of each 16-lane group addresses row t0 + m at column 4g of its group.
      const int grp = lane >> 4, li = lane & 15;
      const int jg = 16 * (grp & 1) + 4 * (li & 3);
      bf16x4 vv[2][4];
      f32x4 bt[2][4];
      bf16x8 ta[6];
#pragma unroll
      for (int tb = 0; tb < 2; ++tb)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const int t0 = 32 * tb + 8 * b + 4 * hf;
          vv[tb][b] = lds_read_tr(&vt[(t0 + (li >> 2)) * VW + jg]);
          bt[tb][b] = *reinterpret_cast<const f32x4*>(&ls.beta[buf][t0]);
        }
#pragma unroll
      for (int n = 0; n < 6; ++n) ta[n] = lds_a_perm(&ls.tm[(32 * (n < 2 ? 0 : 1) + col) * CS], 32 * (n < 4 ? 0 : 1) + 16 * (n & 1) + 4 * hf);
      keep_order();
      f32x16 accU[2] = {};
      bf16x8 rB[2][2];
#pragma unroll
      for (int tb = 0; tb < 2; ++tb) {
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            accE[tb][4 * b + r] = bt[tb][b][r] * (static_cast<float>(vv[tb][b][r]) - accE[tb][4 * b + r]);
        rB[tb][0] = acc_to_b(accE[tb], 0);
        rB[tb][1] = acc_to_b(accE[tb], 1);
      }
#pragma unroll
      for (int n = 0; n < 6; ++n) accU[n < 2 ? 0 : 1] = mfma(ta[n], rB[n < 4 ? 0 : 1][n & 1], accU[n < 2 ? 0 : 1]);
#pragma unroll
      for (int tb = 0; tb < 2; ++tb) {
        uB[tb][0] = acc_to_b(accU[tb], 0);
        uB[tb][1] = acc_to_b(accU[tb], 1);
      }
      // S = Diag(gamma_C) S + Kbar^T U, 16 products in the order (ib, sb, kk), and O += P U; operands are
      // read four products ahead, the decays of block row ib + 1 while block row ib is updated
      bf16x8 pa[6], a[4];
      f32x4 gm[2][4];
#pragma unroll
      for (int b = 0; b < 4; ++b) gm[0][b] = *reinterpret_cast<const f32x4*>(&ls.gc[buf][8 * b + 4 * hf]);
#pragma unroll
      for (int n = 0; n < 6; ++n) pa[n] = lds_a_perm(&ls.pm[(32 * (n < 2 ? 0 : 1) + col) * CS], 32 * (n < 4 ? 0 : 1) + 16 * (n & 1) + 4 * hf);
      auto kbt_op = [&](int m) {
        const int c = 32 * (m >> 2) + col, t = 32 * ((m >> 1) & 1) + 16 * (m & 1) + 4 * hf;
        return cat(*reinterpret_cast<const bf16x4*>(&ls.kbt[buf][kbt_at(c, t)]), *reinterpret_cast<const bf16x4*>(&ls.kbt[buf][kbt_at(c, t + 8)]));
      };
#pragma unroll
      for (int n = 0; n < 4; ++n) a[n] = kbt_op(n);
      keep_order();
#pragma unroll
      for (int n = 0; n < 6; ++n) accO[n < 2 ? 0 : 1] = mfma(uB[n < 4 ? 0 : 1][n & 1], pa[n], accO[n < 2 ? 0 : 1]);
#pragma unroll
      for (int n = 0; n < 16; ++n) {
        const int ib = n >> 2, sb = (n >> 1) & 1, kk = n & 1;
        if ((n & 3) == 0) {
          if (ib + 1 < 4) {
#pragma unroll
            for (int b = 0; b < 4; ++b)
              gm[(ib + 1) & 1][b] = *reinterpret_cast<const f32x4*>(&ls.gc[buf][32 * (ib + 1) + 8 * b + 4 * hf]);
          }
#pragma unroll
          for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) S[ib][4 * b + r] *= gm[ib & 1][b][r];
        }
        const bf16x8 cur_a = a[n & 3];
        if (n + 4 < 16) a[n & 3] = kbt_op(n + 4);
        keep_order();
        S[ib] = mfma(cur_a, uB[sb][kk], S[ib]);
      }
    }
    if (nxt.valid) {
      lds_barrier();   // 2
      const int slow = ls.nslow;
      for (int base = 0; base < slow; base += kSlowBatch)
        for (int i = 0; i < 3; ++i) lds_barrier();
      if (slow > 0) lds_barrier();
    }
    // O^T tile tb: lane = row 32 tb + col, register 4 b + r = column 8 b + 4 hf + r of the wave's 32.  The
    // half-waves trade registers so that each lane stores 8 consecutive columns.
    u32x4 ow[2][2];
    const int out_rows = cur.valid ? cur.rows() - col : 0;
    __bf16* out_at = out + cur.tok0() * tok_stride + int64_t(cur.head) * kD + o_lane;
#pragma unroll
    for (int tb = 0; tb < 2; ++tb)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const u32x4 x = __builtin_bit_cast(u32x4, acc_to_b(accO[tb], h));   // columns 16 h + 4 hf .. and 8 further
        const auto lo = __builtin_amdgcn_permlane32_swap(x[0], x[2], false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap(x[1], x[3], false, false);
        ow[tb][h] = u32x4{lo[0], hi[0], lo[1], hi[1]};
      }
    auto store_out = [&](int tb, int h) {
      if (32 * tb < out_rows) *reinterpret_cast<u32x4*>(out_at + 32 * tb * tok_stride + 16 * h) = ow[tb][h];
    };
    if (!nxt.valid) {
#pragma unroll
      for (int i = 0; i < 4; ++i) store_out(i >> 1, i & 1);
    } else {
      // (before any store of this period: the wait for these loads would wait for the stores too)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *reinterpret_cast<u32x4*>(&vt[(mrow + 16 * i) * VW + mpart]) = vraw[i];
    }
    if (cur.valid && cur.last()) {            // snapshot at the chunk boundary
      float* st = state_pool + (int64_t(cur.state_out) * H + cur.head) * kD * kD + j0 + col;
#pragma unroll
      for (int ib = 0; ib < 4; ++ib)
#pragma unroll
        for (int reg = 0; reg < 16; ++reg) st[(32 * ib + 8 * (reg >> 2) + 4 * hf + (reg & 3)) * kD] = S[ib][reg];
    }
    if (!nxt.valid) break;
    if (nxt.blk == 0) {
#pragma unroll
      for (int ib = 0; ib < 4; ++ib) S[ib] = f32x16{};
      if (nxt.state_in >= 0) {
        const float* st = state_pool + (int64_t(nxt.state_in) * H + nxt.head) * kD * kD + j0 + col;
#pragma unroll
        for (int ib = 0; ib < 4; ++ib)
#pragma unroll
          for (int reg = 0; reg < 16; ++reg) S[ib][reg] = st[(32 * ib + 8 * (reg >> 2) + 4 * hf + (reg & 3)) * kD];
      }
    }
    // E = K~ S0 and O^T = (Q~ S0)^T, operands read three steps ahead; block n's outputs leave
    // between the steps, and barriers 3 to 6 fall about where the builders reach them
    accE[0] = accE[1] = accO[0] = accO[1] = f32x16{};
    {
      bf16x8 sB[2], ak[3], aq[3];
#pragma unroll
      for (int n = 0; n < 16 + 3; ++n) {
        if (n >= 3) {
          const int m = n - 3, ib = m >> 2, kk = (m >> 1) & 1, tb = m & 1;
          if (tb == 0) sB[kk] = acc_to_b(S[ib], kk);
          accE[tb] = mfma(ak[n % 3], sB[kk], accE[tb]);
          accO[tb] = mfma(sB[kk], aq[n % 3], accO[tb]);
          if (m == 2 || m == 5 || m == 8 || m == 11) store_out((m - 2) / 6, ((m - 2) / 3) & 1);
          if (m == 5 || m == 13 || m == 14 || m == 15) lds_barrier();   // 3, 4, 5, 6
        }
        if (n < 16) {
          const int cb = 32 * (n >> 2) + 16 * ((n >> 1) & 1) + 4 * hf;
          ak[n % 3] = lds_a_perm(&ls.kt[(32 * (n & 1) + col) * QS], cb);
          aq[n % 3] = lds_a_perm(&ls.qt[(32 * (n & 1) + col) * QS], cb);
        }
        keep_order();
      }
    }
    cur = nxt;
    nxt.advance(p);
  }
}

template <bool kListed>
__global__ __launch_bounds__(512, 2) void kda_prefill_kernel(KdaDevPlan p, const __bf16* __restrict__ q,
                                                             const __bf16* __restrict__ k,
                                                             const __bf16* __restrict__ v,
                                                             const float* __restrict__ alpha,
                                                             const float* __restrict__ beta,
                                                             float* __restrict__ state_pool,
                                                             __bf16* __restrict__ out) {
  __shared__ __attribute__((aligned(16))) KdaLds ls;
  if (!kda_meta_ok(p)) return;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the 16-blocks right of an even diagonal block are read as part of its 32 x 32 block, never written
  if (tid < 256)
    for (int h = 0; h < 2; ++h)
      ls.tm[(32 * h + (tid >> 4)) * CS + 32 * h + 16 + (tid & 15)] = static_cast<__bf16>(0.0f);
  // (ordered before their first reader by the period's barriers)
  if (wave < 4)
    build_blocks<kListed>(p, ls, q, k, alpha, beta, wave, tid);
  else
    run_blocks<kListed>(p, ls, v, state_pool, out, wave - 4, tid & 63);
}

}  // namespace

hipError_t launch_kda_prefill(const KdaDevPlan& p, const void* q, const void* k, const void* v, const float* alpha,
                              const float* beta, float* state_pool, void* out, hipStream_t stream) {
  if (p.num_items == 0) return hipSuccess;
  const dim3 grid(std::min(p.num_items * p.num_heads, kNumCu)), block(512);
  hipLaunchKernelGGL(p.listed ? kda_prefill_kernel<true> : kda_prefill_kernel<false>, grid, block, 0, stream, p,
                     static_cast<const __bf16*>(q), static_cast<const __bf16*>(k), static_cast<const __bf16*>(v), alpha,
                     beta, state_pool, static_cast<__bf16*>(out));
  return hipGetLastError();
}

}  // namespace wavepp
