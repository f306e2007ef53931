// Attention of the chunk's queries over the retained cache plus the chunk itself.
// Sec. 3.2 of the paper: P = softmax(Q K^T / sqrt(D)), block boundaries from the block length L_B;
// App. A: L_B = chunk length at inference (then the chunk attends to all of itself).
//
// Flash-style kernel for gfx950: bf16 MFMA (v_mfma_f32_32x32x16_bf16), fp32 online softmax, fp32
// accumulation.  One workgroup = 8 waves = 256 queries of one head; each wave owns 32 queries (one
// column block) and walks the key axis in tiles of 64 keys.  Both products are TRANSPOSED:
//
//   S^T[key, q] = K_blk . Q^T          (A = K rows from LDS, B = Q^T held in registers for the whole loop)
//   O^T[d,   q] = V_blk^T . P^T        (A = V^T via transposing LDS reads, B = P^T straight from the S^T
//                                       accumulator registers)
//
// In the 32x32 accumulator layout a lane holds 16 rows of ONE column, so with queries as columns the
// softmax row reductions are in-register plus one half-wave swap, the rescale factor is one scalar per
// lane, and the accumulator registers of S^T already ARE the B operand of the second product (its
// contraction index - the key - may be enumerated in any order as long as V^T uses the same order).
//
// Scheduling.  On this chip the matrix and vector pipes only overlap reliably for instructions of the
// SAME wave (a wave with a matrix instruction waiting at issue blocks the vector instructions of its
// SIMD neighbour), so each wave is software-pipelined by hand: step t issues the 16 MFMAs of S^T(t+1)
// and the 16 MFMAs that add tile t-1 to O^T, and after each of them a slice of the online softmax of
// tile t (vector ALU).  Two such waves share a SIMD and fill each other's stalls.  No step looks for the
// maximum of its tile: the weights are taken relative to the maximum of the first tile and their sum, which
// is needed anyway, shows when a tile has outgrown it (the result is mathematically unchanged).  Raising that
// reference, with the rescale of O^T, is a rare out-of-line event.
//
// K/V tiles (64 keys) stream from global memory straight into a 4-deep LDS ring (global_load_lds, no
// staging registers) two to four tiles ahead of their use; rows are stored with an XOR swizzle of their
// 16-byte chunks so that both the b128 K reads and the transposing V reads are bank-conflict free
// without padding.  The two key segments (retained cache, chunk) are addressed row by row, so no
// concatenated copy exists.
#include "pafu_internal.h"

namespace pafu {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

// P^T fragments are kept as 4 dwords of packed bf16 pairs (the B operand of the second product)
__device__ __forceinline__ bf16x8 as_bf16x8(const u32x4& v) { return __builtin_bit_cast(bf16x8, v); }
__device__ __forceinline__ unsigned pack_bf16(float lo, float hi) {
  bf16x2 t;
  t[0] = (__bf16)lo;
  t[1] = (__bf16)hi;
  return __builtin_bit_cast(unsigned, t);
}

struct AttnParams {
  const int* ids;  // gather variant: retained row r of the cache segment is row ids[r] of Kc / Vc
  int n_cache;     // rows behind Kc / Vc in the gather variant
  long long ld_q, ld_c, ld_n, ld_o;
  int Lq, n_kept, Lc, block_len;
  int N_heads;  // heads per layer; the work list runs over the heads of all layers, layer by layer
  float scale_log2;  // softmax scale * log2(e)
  float k_scale, v_scale;  // 8-bit K/V: the tensors' power-of-two scales (a stored code c stands for c * scale)
};

constexpr int kAtWaves = 8;
constexpr int kAtThreads = kAtWaves * 64;
constexpr int kAtBQ = kAtWaves * 32;  // queries per workgroup
constexpr int kAtTileKeys = 64;       // keys per LDS tile = keys per pipeline step
constexpr int kAtStages = 4;          // LDS ring depth (tiles)
// Ids ring depth (gather variant).  Step t asks for the ids of tile t + 7 (kAtStages + kAtIdLead); they have landed when its
// group of two steps ends.  Tile u's K rows are copied in the group that starts 3 (u even) or 4 (u odd) steps after that, its V
// rows in the next group, and the slot's next ids, tile u + 8's, are asked for in the one behind.
constexpr int kAtIdStages = 8;
constexpr int kAtIdLead = 3;
constexpr int kAtXcds = 8;            // accelerator dies, each with its own L2
// A tile's weights are taken relative to a maximum of the tiles before it; a lane's 32 of them may sum up to this much
// before that reference is raised.  (bf16 weights and fp32 sums have the same relative precision at any scale, and what
// 2^24 times the largest V adds up to is far from overflow.)
constexpr float kAtMaxTileSum = 16777216.0f;
// ... and beyond this the weights are computed once more instead of being scaled (some may be infinite).
constexpr float kAtMaxScaledSum = 1.2676506e30f;  // 2^100
// Study builds only (never the shipped library, which is built without the macro): PAFU_ATTN_ABLATE is a bit mask that
// takes ingredients out of the inner loop so that what they cost can be measured on the same shapes and data; the
// results of such a build are meaningless.  pafu_study_build() returns the mask.
//   1: no global -> LDS tile copies inside the loop (the ring keeps the tiles of the prologue)
//   2: no softmax arithmetic (P = the upper halves of S, one byte-permute per pair; sums and maxima untouched)
#ifndef PAFU_ATTN_ABLATE
#define PAFU_ATTN_ABLATE 0
#endif
constexpr bool kAblateLoads = (PAFU_ATTN_ABLATE & 1) != 0;
constexpr bool kAblateSoftmax = (PAFU_ATTN_ABLATE & 2) != 0;
constexpr float kAtNoMax = -1.0e30f;  // reference before the first visible key (finite on purpose)
constexpr int kAtMaxRuns = 256;       // most runs a unit list is ever cut into (one per CU)
constexpr int kAtMinRunUnits = 2;     // fewest units of a run
constexpr int kAtMinCutGain = 4;      // a cut has to shorten the last round by this many units to pay for its merge pass

constexpr int attn_lds_bytes(int D, bool gather = false) {
  return 2 * kAtStages * kAtTileKeys * 2 * D + (gather ? kAtIdStages * kAtTileKeys * 4 : 0);
}

typedef __attribute__((address_space(3))) unsigned char lds_byte;

__device__ __forceinline__ float half_swap_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_swap_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// One wave-wide global -> LDS copy of 64 x 16 bytes: lane l's 16 bytes land at lds_addr + 16 l.  Written as
// inline assembly so that the compiler's own wait-count insertion does not serialise it against later LDS
// reads of OTHER ring slots; completion is tracked by hand with wait_vmcnt<N>() before a barrier.
__device__ __forceinline__ void dma_row_chunks(const void* src, unsigned lds_addr_uniform) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
               :
               : "s"(lds_addr_uniform), "v"(src)
               : "memory");
}

// The same copy addressed as a wave-uniform base plus a 32-bit per-lane byte offset, to lds_addr + lds_more.  (The sum goes
// straight into m0: sums that the compiler sees are kept in scalar registers for the whole loop, sixteen of them.)
__device__ __forceinline__ void dma_row_chunks_at(const void* base_uniform, unsigned byte_off, unsigned lds_addr_uniform,
                                                  int lds_more) {
  asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :
               : "s"(lds_addr_uniform), "v"(byte_off), "s"(base_uniform), "s"(lds_more)
               : "memory", "scc");
}

// s_waitcnt vmcnt(N) with the other counters left alone (gfx9 encoding: vmcnt = bits 3:0 and 15:14).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

__device__ __forceinline__ bf16x8 lds_read_k(const lds_byte* p) {
  return *(const __attribute__((address_space(3))) bf16x8*)p;
}
// V^T fragment: two transposing reads, 8 key rows apart
__device__ __forceinline__ bf16x8 lds_read_vt(const lds_byte* p, int row_bytes8) {
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p);
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p + row_bytes8));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Raises the reference msc of the queries whose tile has outgrown it (the sum of its weights, psum, has passed kAtMaxTileSum in
// either lane half) and scales the tile's weights, their sum and the sum so far by it; returns what O^T is to be scaled by.
__device__ __forceinline__ float attn_raise(const f32x16 (&s_cur)[2], u32x4 (&p_cur)[4], float sc, float& msc, float& l_run,
                                            float& psum) {
  float alpha = 1.f;
  // far above the reference (the first tile that a query sees, behind masked ones): take its own maximum
  if (__builtin_amdgcn_ballot_w64(psum > kAtMaxScaledSum) != 0) {
    const bool grow = half_swap_max(psum > kAtMaxTileSum ? 1.f : 0.f) != 0.f;  // both halves of a query together
    float mx = s_cur[0][0];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s_cur[kb][r]);
    mx = half_swap_max(mx);
    const float msc_new = grow ? fmaxf(msc, mx * sc) : msc;
    const float down = __builtin_amdgcn_exp2f(msc - msc_new);
    msc = msc_new;
    alpha = down;
    l_run *= down;
    psum = 0.f;
#pragma unroll
    for (int e = 0; e < 32; e += 2) {
      const float pe0 = __builtin_amdgcn_exp2f(fmaf(s_cur[e >> 4][e & 15], sc, -msc_new));
      const float pe1 = __builtin_amdgcn_exp2f(fmaf(s_cur[e >> 4][(e & 15) + 1], sc, -msc_new));
      psum += pe0;
      psum += pe1;
      p_cur[e >> 3][(e & 7) >> 1] = pack_bf16(pe0, pe1);
    }
  }
  const float up = half_swap_max(psum > kAtMaxTileSum ? (float)__builtin_amdgcn_frexp_expf(psum) : 0.f);
  const float scale = __builtin_amdgcn_exp2f(-up);
  msc += up;
  l_run *= scale;
  psum *= scale;
  alpha *= scale;
  const unsigned exponent = (unsigned)up * 0x00800080u;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    unsigned w = p_cur[i >> 2][i & 3];
    asm("v_pk_sub_u16 %0, %0, %1 clamp" : "+v"(w) : "v"(exponent));
    p_cur[i >> 2][i & 3] = w;
  }
  return alpha;
}

// Pipeline step t for one wave (32 queries), one straight-line block:
//   matrix pipe : S^T(t+1) = K(t+1) Q^T into s_nxt;  O^T += V(t-1)^T P(t-1)^T from p_prev
//   vector pipe : online softmax of s_cur = S^T(t) -> p_cur = P^T(t), running max / sum,
// with the vector work sliced between the MFMAs.  Edge cases are handled by the caller through the operands
// (masked elements of s_cur set to -inf beforehand, p_prev = 0 before the first tile, a clamped K tile when
// there is no next tile), so this is the only implementation of the step.
// s_*[kb] = key block kb (32 keys) of the tile; p_*[ks] = 16-key slice ks of the tile.
// What bounds it: the issue slots that 32 matrix instructions share with the vector work of 2048 scores, at a clock that
// the power limit sets.  (With a search for the tile's maximum in front of the exponentials a whole step took 5 % longer: 12 heads
// of 128, 4680 queries, 21060 keys, 667 us instead of 634.)
// k_at[kk] / v_at[db]: this lane's LDS addresses of the fragments in ring slot 0; the tiles are K_TILE / V_TILE bytes on,
// which goes into the offset field of the reads.
// issue(i) starts this step's global -> LDS tile copies behind slot i.  They start a few slots into the step, not at
// its start: right after the barrier all eight waves would queue their copies at once and sit behind the memory pipe
// (a wave issues nothing while its copy waits), whereas an eighth and a half of the way in they find it free.
// kf / vf: the fragments of the first MFMAs, read ahead by the step before (AHEAD_IN); this step then reads those of the next
// one (AHEAD_OUT) from the tiles K_NEXT / V_NEXT bytes on.  Otherwise it reads its own.
template <int D, int K_TILE, int V_TILE, bool AHEAD_IN, bool AHEAD_OUT, int K_NEXT, int V_NEXT, typename Issue>
__device__ __forceinline__ void attn_step(const f32x16 (&s_cur)[2], f32x16 (&s_nxt)[2], const u32x4 (&p_prev)[4],
                                          u32x4 (&p_cur)[4], f32x16 (&o)[D / 32], const bf16x8 (&qf)[D / 16],
                                          float& msc, float& l_run, const lds_byte* const (&k_at)[D / 16],
                                          const lds_byte* const (&v_at)[D / 32], bf16x8 (&kf)[2], bf16x8 (&vf)[2],
                                          float sc, Issue&& issue) {
  constexpr int ROWB = 2 * D;
  constexpr int KD = D / 16;
  constexpr int DB = D / 32;
  constexpr int NS = 2 * KD;       // MFMAs of S^T(t+1): 2 key blocks x KD contraction steps
  constexpr int NP = 4 * DB;       // MFMAs of the O^T update: 4 key slices x DB row blocks
  constexpr int NSLOT = NS + NP;   // MFMAs per step (NS == NP for D = 64 and 128)
  constexpr int EPS = 32 / NSLOT;  // scores turned into weights behind each MFMA (1 for D = 128, 2 for D = 64)
  static_assert(NS == NP, "the slot pattern alternates one MFMA of each product");
  float psum = 0.f, q_prev = 0.f, q_even = 0.f;

  // slots in groups of four: two MFMAs of S^T (w = 0), which share their query fragment, then two of O^T (w = 1), which
  // mostly share their weights.
  //   S^T MFMA m: key block m & 1, contraction step m >> 1 (the two accumulators alternate).
  //   O^T MFMA m: key slice m / DB, row block m % DB (an accumulator comes back every DB MFMAs).
  // The fragment of MFMA m + 2 is read from LDS as soon as MFMA m has been issued, into the same registers.
  // (One MFMA of each product in turn: 518 us instead of 514, 12 heads of 128, 4680 queries, 21060 keys.)
  auto k_frag = [&](int m) { return lds_read_k(k_at[m >> 1] + K_TILE + (m & 1) * 32 * ROWB); };
  auto v_frag = [&](int m) { return lds_read_vt(v_at[m % DB] + V_TILE + (16 * (m / DB)) * ROWB, 8 * ROWB); };
  if (!AHEAD_IN) {
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      kf[m] = k_frag(m);
      vf[m] = v_frag(m);
    }
  }
  f32x16 zero;
#pragma unroll
  for (int r = 0; r < 16; ++r) zero[r] = 0.f;

#pragma unroll
  for (int i = 0; i < NSLOT; ++i) {
    const int m = 2 * (i >> 2) + (i & 1), w = (i >> 1) & 1, mb = m & 1;
    // ---- matrix pipe.  The empty asm statements order each MFMA against the vector slices around it (all asm
    // volatile statements keep their relative order), which fixes the interleaving written here.
    if (w == 0) {
      const int kb = m & 1, kk = m >> 1;
      asm volatile("" : "+v"(kf[mb]));
      if (kk == 0) s_nxt[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[mb], qf[kk], zero, 0, 0, 0);
      else s_nxt[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[mb], qf[kk], s_nxt[kb], 0, 0, 0);
      asm volatile("" : "+v"(s_nxt[kb]));
      if (m + 2 < NS) kf[mb] = k_frag(m + 2);
      else if (AHEAD_OUT) kf[mb] = lds_read_k(k_at[0] + K_NEXT + mb * 32 * ROWB);
    } else {
      const int ks = m / DB, db = m % DB;
      asm volatile("" : "+v"(vf[mb]));
      o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[mb], as_bf16x8(p_prev[ks]), o[db], 0, 0, 0);
      asm volatile("" : "+v"(o[db]));
      if (m + 2 < NP) vf[mb] = v_frag(m + 2);
      else if (AHEAD_OUT) vf[mb] = lds_read_vt(v_at[mb] + V_NEXT, 8 * ROWB);
    }
    // ---- vector pipe slice
    if (kAblateSoftmax) {
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        if ((u * NSLOT) / 16 == i) {
          const int kb = u >> 3, r = 2 * (u & 7);
          p_cur[2 * kb + (r >> 3)][(r & 7) >> 1] = __builtin_amdgcn_perm(
              __float_as_uint(s_cur[kb][r + 1]), __float_as_uint(s_cur[kb][r]), 0x07060302u);
        }
      }
      psum = 1.f;
    } else {  // weights of this slot's keys, relative to the reference that the tiles before this one left
#pragma unroll
      for (int x = 0; x < EPS; ++x) {
        const int e = EPS * i + x, kb = e >> 4, r = e & 15;
        // the slice may not rise above the previous MFMA ... (tied through msc: tying the score would copy it)
        asm volatile("" : "+v"(msc));
        float pe = __builtin_amdgcn_exp2f(fmaf(s_cur[kb][r], sc, -msc));
        // the sum and the pack of the PREVIOUS key go here, behind this key's exponential: a transcendental result
        // takes several issue slots to arrive, and adding it right away stalls the wave
        if (e > 0) {
          psum += q_prev;
          asm volatile("" : "+v"(psum));
          if ((e & 1) == 0) {
            const int ep = e - 2;
            unsigned pk = pack_bf16(q_even, q_prev);
            asm volatile("" : "+v"(pk));
            p_cur[ep >> 3][(ep & 7) >> 1] = pk;
          } else {
            q_even = q_prev;
          }
        }
        q_prev = pe;
        asm volatile("" : "+v"(q_prev));  // ... nor sink below the next one
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    issue(i);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (kAblateSoftmax) {
    l_run += psum;
    return;
  }
  psum += q_prev;  // the last key
  p_cur[3][3] = pack_bf16(q_even, q_prev);
  // O^T now holds the tiles < t relative to the reference, and so are P^T(t) and its sums: nothing to rescale, unless the
  // tile outgrew it.  Then the reference of the queries concerned is raised by the power of two in the sum (of either lane
  // half), and everything is scaled by it: the packed weights in their exponent fields, exactly but for weights that
  // vanish beside the sum.  (NaN weights go on as they are: their query's result is a NaN whatever the reference.)
  // A raise costs little: 4680 over 16380 keys (12 heads of 128), scores that grow eightfold along the cache 558 us
  // (without growth 542), one NaN query in each wave 541.
  // (In place, without an else branch and out of line: copies of P^T in every step cost 4 %, the code inside the loop 1 % of the
  // 8-bit variant.)
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(psum > kAtMaxTileSum) != 0, 0)) {
    const float alpha = attn_raise(s_cur, p_cur, sc, msc, l_run, psum);
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[b][r] *= alpha;
  }
  l_run += psum;
}

template <int N>
struct Phase {
  static constexpr int value = N;
};

// Block mask / ragged tail for the tile starting at key0: register r of s[kb] holds key
// key0 + 32 kb + 8 (r/4) + 4 g + (r%4).
__device__ __forceinline__ void attn_mask(f32x16 (&s)[2], int key0, int lim, int g) {
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int kidx = key0 + 32 * kb + 8 * (r >> 2) + 4 * g + (r & 3);
      if (kidx >= lim) s[kb][r] = -INFINITY;
    }
}

// ---- work decomposition -----------------------------------------------------------------------------------------
// A work item is one (head, query tile of kAtBQ queries); its cost is counted in UNITS of two key tiles (one loop
// iteration): units(qt) = ceil(ceil(visible keys of the tile's last query / 64) / 2).  Items are ordered head-major.
// One workgroup per item leaves CUs idle in the last round of items over the CUs (a one-frame chunk of 1560 queries is 84
// items on 256 CUs; 272 items are a full round and one of 16), so with a workspace the items of an ill-filled last round
// are cut instead: their flattened unit list goes in `n_runs` equal contiguous runs to one workgroup each, behind the
// `n_whole` workgroups that take an item each.  A run covers the tail of one item, possibly some whole items, and the
// head of another.  A workgroup that does not see all units of an item writes its unnormalised O^T together with the
// reference and the row sums into the workspace (slot 2 g for the first segment of run g, 2 g + 1 for its last),
// and attn_combine_kernel merges the partial results of such items afterwards, always in run order, so the result does
// not depend on timing.
struct AttnWork {
  int n_qt;           // query tiles per head
  int units_head;     // units of one head (sum over its query tiles)
  int uniform;        // units of every query tile when they are all equal (no block mask), else 0
  int n_items;        // heads of all layers * n_qt
  int n_whole;        // workgroup g < n_whole takes item g
  int n_runs;         // equal runs over the units of the items from n_whole on
  long long u0, U;    // ... which are units [u0, u0 + U) of the flattened list
  int h0, r0;         // head of unit u0, and the units of that head in front of it; r0 + U below 2^31
  float* part_o;      // [2 n_runs][kAtBQ][D] fp32
  float* part_ml;     // [2 n_runs][2][kAtBQ] fp32: reference (log2 domain), row sum
};

__host__ __device__ inline int attn_units(int qt, int Lq, int n_kept, int Lc, int L_B) {
  const int i_last = (qt + 1) * kAtBQ - 1 < Lq ? (qt + 1) * kAtBQ - 1 : Lq - 1;
  const long long e = ((long long)(i_last / L_B) + 1) * L_B;
  const int vis = n_kept + (int)(e < Lc ? e : Lc);
  return ((vis + kAtTileKeys - 1) / kAtTileKeys + 1) / 2;
}
// (Run g of G begins with unit floor(g U / G).)

struct AttnArgs {
  AttnParams p;
  AttnWork w;
  AttnLayer layer[kAttnBatchMax];
};

// Wave-uniform values that come out of vector instructions (64-bit divisions are expanded on the vector ALU) are
// moved back to scalar registers, so that addresses built from them can serve as scalar bases.
__device__ __forceinline__ int uniform_i32(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ long long uniform_i64(long long v) {
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)(unsigned long long)v);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)((unsigned long long)v >> 32));
  return (long long)(((unsigned long long)hi << 32) | lo);
}

// The kernel's one argument where it lies, for code that shall read it anew.
typedef const __attribute__((address_space(4))) AttnArgs* KernelArgs;
__device__ __forceinline__ KernelArgs kernel_args() {
  KernelArgs a = (KernelArgs)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(a));
  return a;
}

// GATHER: the cache segment is read through an index list (index-based Select, Sec. 3.4; Eq. 7): K/V stay
// uncompacted and tile row r comes from cache row ids[r].  The 64 ids of a tile travel global -> LDS like the tiles
// themselves (one 4-byte-per-lane load per wave and step, three steps ahead of the K tile that needs them, into a
// small ring of their own), so the vector-memory queue stays one hand-counted stream and a lane picks up its row
// index with one LDS read.
//
// KV8: K and V (both key segments) are stored as 8-bit E4M3 codes with one power-of-two scale per tensor.  The tile
// copies then move half the bytes, into a ring of raw tiles; every wave converts the 1 KB of each raw tile that it
// copied itself to bf16 (scale applied, exact) and writes it, in the swizzled layout the fragment reads expect, into
// one of two bf16 slots per tensor, one step before the matrix instructions read it.  The matrix instructions, the
// softmax and the fragment reads are the bf16 kernel's; the arithmetic is no narrower than in the bf16 kernel.
template <int D, bool OUT_F32, bool GATHER, bool KV8>
__global__ __launch_bounds__(kAtThreads, 1) void chunk_attention_kernel(AttnArgs args) {
  static_assert(!KV8 || (D == 128 && !GATHER), "8-bit K/V: head dim 128, no index list");
  const AttnParams& p = args.p;
  const AttnWork& wk = args.w;
  constexpr int ROWB = 2 * D;                  // bytes per bf16 K/V row of one head (what the fragment reads see)
  constexpr int TILEB = kAtTileKeys * ROWB;    // bytes per bf16 K (or V) tile
  constexpr int CH = D / 8;                    // 16-byte chunks per bf16 row
  constexpr int RPB = 256 / ROWB;              // rows per 256 bytes (one pass over all LDS banks)
  constexpr int ELB = KV8 ? 1 : 2;             // bytes per stored K/V element
  constexpr int SROWB = ELB * D;               // bytes per stored row of one head (what the tile copies move)
  constexpr int STILEB = kAtTileKeys * SROWB;  // bytes per stored tile
  constexpr int SCH = SROWB / 16;              // 16-byte chunks per stored row
  constexpr int RPI = 1024 / SROWB;            // stored rows written by one wave-wide 16-byte-per-lane load
  constexpr int LPT = STILEB / 1024 / kAtWaves;  // such loads per wave per tensor per tile
  constexpr int CK = KV8 ? 2 : kAtStages;      // bf16 tile slots per tensor
  static_assert(LPT >= 1, "every wave copies part of every tile");
  // A barrier ends every GROUP of steps.  bf16: two steps, which start the copies of two tiles of each tensor; with 8-bit K/V
  // every step's tiles are converted in the step before.  (A barrier after each step: 517 us instead of 509, 12 heads of
  // 128, 4680 queries, 21060 keys.  Where in the first step the copies start makes no difference.)
  constexpr int GROUP = KV8 ? 1 : 2;
  constexpr int kInFlight = KV8 ? (kAtStages - 2) * 2 * LPT : 0;  // copies that may stay in flight over a barrier
  constexpr int KD = D / 16;
  constexpr int DB = D / 32;
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds_raw[];
  lds_byte* const k_ring = (lds_byte*)lds_raw;     // bf16 tiles the fragment reads address: CK slots
  lds_byte* const v_ring = k_ring + CK * TILEB;
  // 8-bit K/V: rings of raw tiles behind the bf16 slots (plain layout: lane l of wave w at w * 1024 + 16 l)
  lds_byte* const k_land = KV8 ? v_ring + CK * TILEB : k_ring;   // where the tile copies land
  lds_byte* const v_land = KV8 ? k_land + kAtStages * STILEB : v_ring;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // said to be uniform: what depends on it stays scalar
  // Query block of this wave inside the 256-query tile.  Waves w and w + 4 share a SIMD; they take neighbouring blocks,
  // so that a ragged tile (the last one of a head: 72 of 256 rows at the Wan-1.3B shape) fills SIMDs pairwise and
  // steps at the pace of the full tiles.  With block = wave its few busy waves would each have a SIMD to themselves,
  // run through the keys twice as fast as the other workgroups of the head and pull every K/V line into the L2 long
  // before they need it, i.e. once more from HBM.
  const int qblk = 2 * (wave & 3) + (wave >> 2);
  const int g = lane >> 5, c = lane & 31;
  // Logical workgroup.  Workgroups are handed to the 8 XCDs round-robin in launch order and every XCD has its own
  // L2, so XCD x (workgroups x, x + 8, ...) takes one contiguous range of the head-major item list, and one of the runs
  // behind it: at any time an XCD then streams the K/V of one or two heads instead of all of them.
  const bool is_run = (int)blockIdx.x >= wk.n_whole;
  const int total = is_run ? wk.n_runs : wk.n_whole;
  const int xcd = blockIdx.x % kAtXcds;  // (whole items and runs are only mixed when n_whole is a multiple of kAtXcds)
  const int xslot = (blockIdx.x - (is_run ? wk.n_whole : 0)) / kAtXcds;
  const int wg = xcd * (total / kAtXcds) + (xcd < total % kAtXcds ? xcd : total % kAtXcds) + xslot;
  const int L_B = p.block_len;

  // ---- global -> LDS tile loads.  Load j of this wave fills LDS rows (wave + W j) * RPI .. + RPI of a tile; lane ->
  // (row, slot); the slot receives chunk (slot ^ swizzle(row)) of that row (raw 8-bit tiles are not swizzled).  The chunk
  // does not depend on j: consecutive loads of a wave are kAtWaves * RPI rows apart, a multiple of the swizzle period.
  auto lane_chunk = [](int wave, int lane, bool is_v) {
    const int row = wave * RPI + lane / SCH, slot = lane % SCH;
    if (KV8) return slot;
    return is_v ? slot ^ (4 * ((row / RPB) & (CH / 4 - 1))) : slot ^ ((row / RPB) & (CH - 1));
  };
  const unsigned lds_wave = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(lds_byte*)lds_raw + wave * 1024);
  // ---- LDS read offsets (bytes inside a tile)
  // K fragment (A operand): lane (key row c, half g) reads chunk (2 kk + g) of row c; its slot is (2 kk) ^ kx2
  const int kx2 = g ^ ((c / RPB) & (CH - 1));
  const int k_off = c * ROWB;
  // V^T fragment via transposing reads: 16-lane group = (d-half, key group g); lane i of the group points at key
  // row rr = 4 g + i/4, four consecutive d at 4 (i%4).  32 lanes (one key group) read 4 rows x 64 bytes per
  // instruction; the swizzle spreads those over all banks.  Slot of d-block b is ((4 b) ^ vx2) + cl.
  const int i16 = lane & 15;
  const int rr = 4 * g + (i16 >> 2);
  const int vx2 = 4 * ((rr / RPB) & (CH / 4 - 1));
  const int cl = 2 * ((lane >> 4) & 1) + ((i16 & 3) >> 1);
  const int v_off = rr * ROWB + ((i16 & 1) << 3) + (cl << 4);
  const lds_byte* k_at[KD];
  const lds_byte* v_at[DB];
#pragma unroll
  for (int kk = 0; kk < KD; ++kk) k_at[kk] = k_ring + k_off + (((2 * kk) ^ kx2) << 4);
#pragma unroll
  for (int b = 0; b < DB; ++b) v_at[b] = v_ring + v_off + (((4 * b) ^ vx2) << 4);
  const float sc = p.scale_log2;
  int* const id_ring = reinterpret_cast<int*>(lds_raw + 2 * kAtStages * TILEB);  // gather variant (bf16 K/V only)

  // ---- this workgroup's units: from unit `from` of item (h, qt) on, `room` of them.  (The setup is straight-line code that
  // every launch fetches anew, so divisions and what only some launches need are kept out of the way of the others.)
  const bool masked = L_B < p.Lc;
  // (fetched with the other arguments: behind the divisions it would be another round trip to memory)
  AttnLayer first_layer = args.layer[0];
  asm volatile("" : "+s"(first_layer.Q), "+s"(first_layer.Kc), "+s"(first_layer.Vc), "+s"(first_layer.Kn), "+s"(first_layer.Vn), "+s"(first_layer.O));
  int h, qt, from = 0, room = 0x7fffffff;
  if (is_run) {
    const int U = (int)wk.U, q = U / wk.n_runs, r = U - q * wk.n_runs;  // g U / G = g q + g r / G, G at most kAtMaxRuns
    const int begin = wg * q + (int)((unsigned)(wg * r) / (unsigned)wk.n_runs);
    room = uniform_i32((wg + 1) * q + (int)((unsigned)((wg + 1) * r) / (unsigned)wk.n_runs) - begin);
    h = uniform_i32(wk.h0 + (wk.r0 + begin) / wk.units_head);
    from = uniform_i32(wk.r0 + begin - (h - wk.h0) * wk.units_head);
    if (wk.uniform) {
      qt = uniform_i32(from / wk.uniform);
      from -= qt * wk.uniform;
    } else {
      for (qt = 0;; ++qt) {
        const int cq = attn_units(qt, p.Lq, p.n_kept, p.Lc, L_B);
        if (from < cq) break;
        from -= cq;
      }
    }
  } else {
    h = uniform_i32(wg / wk.n_qt);
    qt = wg - h * wk.n_qt;
  }
  bool first_segment = true;

#pragma unroll 1
  for (;;) {
    // ---- segment: units [pa, pb) of item (h, qt) = key tiles [2 pa, 2 pb)
    const int units = wk.uniform ? wk.uniform : uniform_i32(attn_units(qt, p.Lq, p.n_kept, p.Lc, L_B));
    const int pa = uniform_i32(from);
    const int pb = uniform_i32(room < units - pa ? pa + room : units);
    const bool whole = pa == 0 && pb == units;
    const int n_iter = pb - pa;
    const int tb = 2 * pa;  // first key tile of the segment
    const int i_first = uniform_i32(qt) * kAtBQ;
    const int layer = h < p.N_heads ? 0 : uniform_i32(h / p.N_heads);
    AttnLayer L = first_layer;
    if (layer != 0) L = args.layer[layer];
    const long long head_off = (long long)uniform_i32(h - layer * p.N_heads) * D;

    // number of visible keys: per lane (its query) and the tile's first query, both cut at the segment's end
    const int key_end = 2 * pb * kAtTileKeys;
    const int q_row = i_first + qblk * 32 + c;
    int lim = p.n_kept + p.Lc, lim_min = lim;
    if (masked) {
      auto visible = [&](int i) {
        const long long e = ((long long)(i / L_B) + 1) * L_B;
        return p.n_kept + (int)(e < p.Lc ? e : p.Lc);
      };
      lim = visible(q_row < p.Lq ? q_row : p.Lq - 1);
      lim_min = visible(i_first);
    }
    lim = lim < key_end ? lim : key_end;
    lim_min = lim_min < key_end ? lim_min : key_end;

    // ids ring (gather variant): slot u % kAtIdStages holds the 64 ids of tile u, clamped to the list's end
    auto issue_ids = [&](int tile) {
      if (lane < 8) {  // wave w brings ids 8 w .. 8 w + 7 of the tile: one load per wave, 64 ids per workgroup
        int idx = tile * kAtTileKeys + 8 * wave + lane;
        idx = idx < p.n_kept ? idx : p.n_kept - 1;
        lds_byte* dst = (lds_byte*)(id_ring + (tile % kAtIdStages) * kAtTileKeys + 8 * wave);
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
                     :
                     : "s"(__builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)dst)), "v"((unsigned)idx * 4u), "s"(p.ids)
                     : "memory");
      }
    };
    auto tile_id = [&](int tile, int row) {  // cache row behind tile row `row`, never outside the cache
      const int id = ((const __attribute__((address_space(3))) int*)id_ring)[(tile % kAtIdStages) * kAtTileKeys + row];
      return id < 0 ? 0 : (id < p.n_cache ? id : p.n_cache - 1);
    };
    // gather variant: the cache segment's full tiles, this layer's and head's rows, this lane's place in the ids ring
    const int gather_tiles = GATHER ? p.n_kept / kAtTileKeys : 0;
    const unsigned gather_ld = (unsigned)(p.ld_c * ELB);
    const char* const k_rows = GATHER ? static_cast<const char*>(L.Kc) + head_off * ELB : nullptr;
    const char* const v_rows = GATHER ? static_cast<const char*>(L.Vc) + head_off * ELB : nullptr;
    const lds_byte* const id_at = (const lds_byte*)id_ring + (wave * RPI + lane / SCH) * 4;
    const unsigned k_chunk16 = (unsigned)lane_chunk(wave, lane, false) << 4, v_chunk16 = (unsigned)lane_chunk(wave, lane, true) << 4;
    // Tile t of the segment goes to ring slot t % kAtStages.
    auto lds_slot = [&](bool is_v, int slot, int j) {  // this wave's load j of a slot, from lds_wave on
      return (int)((is_v ? v_land : k_land) - (lds_byte*)lds_raw) + slot * STILEB + kAtWaves * j * 1024;
    };
    // What follows up to copy_tile is rare.  It takes its arguments from memory and its lane number through an opaque copy:
    // what the compiler may hoist out of the loop for it would fill the registers that the loop needs.
    struct Rare {
      KernelArgs a;
      int lane, wave;
    };
    auto rare = [&] {
      Rare r{kernel_args(), lane, wave};
      asm volatile("" : "+v"(r.lane));
      asm volatile("" : "+s"(r.wave));
      return r;
    };
    // row 0 of the key axis of this head, in either segment
    auto cache_base = [&](const void* t) { return static_cast<const char*>(t) + head_off * ELB; };
    auto chunk_base = [&](const void* t, int kept, long long ld_n) {
      return static_cast<const char*>(t) + head_off * ELB - (long long)kept * ld_n * ELB;
    };
    // The general copy works row by row: a tile that straddles the two key segments, or the end of the keys (rows past it
    // are masked later, so they read a valid one instead).
    auto copy_rows = [&](int tile, int slot, bool is_v) {
      const Rare r = rare();
      const auto& l = r.a->layer[layer];
      const int kept = r.a->p.n_kept, keys = kept + r.a->p.Lc;
      const char* base_c = cache_base(is_v ? l.Vc : l.Kc);
      const char* base_n = chunk_base(is_v ? l.Vn : l.Kn, kept, r.a->p.ld_n);
      const unsigned ldc_b = (unsigned)(r.a->p.ld_c * ELB), ldn_b = (unsigned)(r.a->p.ld_n * ELB);  // (below 4 GiB)
#pragma unroll
      for (int j = 0; j < LPT; ++j) {
        const int row = (r.wave + kAtWaves * j) * RPI + r.lane / SCH;
        int kidx = tile * kAtTileKeys + row;
        kidx = kidx < keys ? kidx : keys - 1;
        const bool in_cache = kidx < kept;
        if (GATHER && in_cache) kidx = tile_id(tile, row);
        const char* src = (in_cache ? base_c : base_n) +
                          (unsigned long long)(unsigned)kidx * (in_cache ? ldc_b : ldn_b) +
                          lane_chunk(r.wave, r.lane, is_v) * 16;
        dma_row_chunks(src, lds_wave + lds_slot(is_v, slot, j));
      }
    };
    // The common copy: `left` tiles from the scalar address `base` on are full and lie inside one key segment, `half` bytes
    // from load to load (or lie past the end of the keys: then the last row stands in for all of theirs).  All that a step
    // does for it is to count, add and issue.  Worked out anew for each tile from the kernel arguments it was 45 scalar
    // instructions per tensor and step, and the scalar loads among them waited for all LDS reads in flight (one counter
    // for both): together with the fragment addresses of four ring slots in the reads' offset fields a whole step takes
    // 602 us instead of 635 (12 heads of 128, 4680 queries, 21060 keys), with the 8-bit cache 477 instead of 512 (17160 keys).
    struct TileStream {
      const char* base;
      unsigned half, off;
      int left;
    };
    TileStream ks, vs;
    // prepares the copies from `tile` on; left = 0: not a full tile
    auto seek_in = [&](TileStream& s, int tile, bool is_v, const void* cache_t, const void* chunk_t, int kept, int Lc,
                       long long ld_c, long long ld_n, int wave, int lane) {
      const int keys = kept + Lc;
      const int key0 = tile * kAtTileKeys;
      const bool cache = key0 + kAtTileKeys <= kept, past = key0 >= keys;
      const bool chunk = key0 >= kept && key0 + kAtTileKeys <= keys;
      s.left = uniform_i32(past ? 0x7fffffff
                                : cache && !GATHER ? kept / kAtTileKeys - tile : chunk ? keys / kAtTileKeys - tile : 0);
      const unsigned ld_b = (unsigned)((cache ? ld_c : ld_n) * ELB);
      const unsigned step = past ? 0u : ld_b;
      s.half = (unsigned)uniform_i32((int)((unsigned)(kAtWaves * RPI) * step));
      s.base = reinterpret_cast<const char*>(
          uniform_i64((long long)reinterpret_cast<uintptr_t>(cache ? cache_base(cache_t) : chunk_base(chunk_t, kept, ld_n)) +
                      (long long)((unsigned long long)(unsigned)(past ? keys - 1 : key0) * ld_b)));
      s.off = (unsigned)(wave * RPI + lane / SCH) * step + lane_chunk(wave, lane, is_v) * 16;
    };
    auto seek = [&](TileStream& s, int tile, bool is_v) {
      const Rare r = rare();
      const auto& l = r.a->layer[layer];
      seek_in(s, tile, is_v, is_v ? l.Vc : l.Kc, is_v ? l.Vn : l.Kn, r.a->p.n_kept, r.a->p.Lc, r.a->p.ld_c, r.a->p.ld_n,
              r.wave, r.lane);
    };
    // Gather variant: the cache rows behind a tile's rows, read from the ids ring some slots before their copies are started
    // (right in front of them the wave waited for the LDS twice per tensor and step).
    unsigned row_ids[LPT];
    auto read_ids = [&](int tile) {
      const lds_byte* at = id_at + (tile % kAtIdStages) * (kAtTileKeys * 4);
#pragma unroll
      for (int j = 0; j < LPT; ++j)
        row_ids[j] = *(const __attribute__((address_space(3))) unsigned*)(at + kAtWaves * RPI * 4 * j);
    };
    auto copy_tile = [&](TileStream& s, int tile, int slot, bool is_v) {
      if (GATHER && tile < gather_tiles) {  // workgroup-uniform
        // the head's base plus a 32-bit offset (the host rejects caches of 4 GiB or more per tensor for this variant)
#pragma unroll
        for (int j = 0; j < LPT; ++j) {
          const unsigned id = row_ids[j] < (unsigned)p.n_cache ? row_ids[j] : (int)row_ids[j] < 0 ? 0u : (unsigned)p.n_cache - 1;
          dma_row_chunks_at(is_v ? v_rows : k_rows, id * gather_ld + (is_v ? v_chunk16 : k_chunk16), lds_wave,
                            lds_slot(is_v, slot, j));
        }
        return;
      }
      auto copy = [&] {
        --s.left;
#pragma unroll
        for (int j = 0; j < LPT; ++j) {
          // (the gather variant keeps the stream in vector registers: most of its tiles are none of a stream's)
          const char* base = GATHER ? reinterpret_cast<const char*>(uniform_i64((long long)reinterpret_cast<uintptr_t>(s.base)))
                                    : s.base;
          dma_row_chunks_at(base, s.off, lds_wave, lds_slot(is_v, slot, j));
          s.base = base + s.half;
        }
      };
      if (__builtin_expect(s.left > 0, 1)) {
        copy();
      } else {
        seek(s, tile, is_v);
        if (s.left > 0) copy();
        else copy_rows(tile, slot, is_v);
      }
    };
    // Step t (relative to the segment) reads K tile t+1 and V tile t-1.  bf16: steps t and t+1 (t even) form a group, during
    // which K(t+3), K(t+4), V(t+1) and V(t+2) are copied into the slots of K(t-1), K(t), V(t-3) and V(t-2), whose last readers
    // finished in the group before.  8-bit: step t copies K(t+5) and V(t+3) into the raw slots that step t-1 has converted.
    // Tiles past the end of the key axis hold clamped rows and are masked or never read.
    // In the gather variant the ids of the tiles must already be visible in the ids ring.
    auto issue_k_tile = [&](int kt, int slot, bool ids_read = false) {
      if (GATHER && !ids_read) read_ids(tb + kt);
      copy_tile(ks, tb + kt, slot, false);
    };
    auto issue_v_tile = [&](int vt, int slot, bool ids_read = false) {
      if (GATHER && !ids_read) read_ids(tb + vt);
      copy_tile(vs, tb + vt, slot, true);
    };
    // 8-bit K/V: this wave's 1 KB of a raw tile (the part it copied itself, so only its own copies must have landed)
    // -> bf16, from raw slot `from` into bf16 slot `to`.  Lane l holds 16 codes of key row w * RPI + l / SCH,
    // d = 16 (l % SCH) .. + 16: two 16-byte chunks of the bf16 row, stored with the swizzle of the fragment reads.
    auto cook = [&](int from, int to, bool is_v) {
      typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
      const u32x4 raw = *(const lds_u32x4*)((is_v ? v_land : k_land) + from * STILEB + wave * 1024 + lane * 16);
      const int row = wave * RPI + lane / SCH, chunk = lane % SCH;
      const int sw = is_v ? 4 * ((row / RPB) & (CH / 4 - 1)) : (row / RPB) & (CH - 1);
      lds_byte* dst = (is_v ? v_ring : k_ring) + to * TILEB + row * ROWB;
      const float scl = is_v ? p.v_scale : p.k_scale;
      u32x4 lo, hi;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        lo[2 * e] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[e], scl, false));
        lo[2 * e + 1] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[e], scl, true));
        hi[2 * e] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[2 + e], scl, false));
        hi[2 * e + 1] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[2 + e], scl, true));
      }
      *(lds_u32x4*)(dst + (((2 * chunk) ^ sw) << 4)) = lo;
      *(lds_u32x4*)(dst + (((2 * chunk + 1) ^ sw) << 4)) = hi;
    };
    // what step t (with t % kAtStages == ph) does for the 8-bit tiles: K(t+2) and V(t) become bf16 one step before they are
    // read
    auto cook_step = [&](int ph, int t) {
      if (t + 2 < 2 * n_iter) cook((ph + 2) % kAtStages, ph % CK, false);
      cook(ph % kAtStages, ph % CK, true);
    };

    // Q^T fragments (B operand): lane (query c, half g) holds Q[q][16 kk + 8 g .. +8]
    bf16x8 qf[KD];
    {
      const int qi = q_row < p.Lq ? q_row : p.Lq - 1;
      const unsigned short* qp = static_cast<const unsigned short*>(L.Q) + (long long)qi * p.ld_q + head_off + 8 * g;
#pragma unroll
      for (int kk = 0; kk < KD; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(qp + 16 * kk);
    }

    // ---- prologue: the first tiles of the segment, then S^T(0).  bf16: K(0..2) and V(0); step 0 starts the copies of K(3), K(4),
    // V(1) and V(2).  8-bit: K(0..3), V(0), V(1), and, when K(0) has been converted, K(4) and V(2).
    if (GATHER) {  // ids of the tiles whose loads are issued before step kAtIdLead's ids arrive
#pragma unroll
      for (int i = 0; i < kAtStages + kAtIdLead; ++i) issue_ids(tb + i);
      wait_vmcnt<0>();
      __builtin_amdgcn_s_barrier();
    }
    seek_in(ks, tb, false, L.Kc, L.Kn, p.n_kept, p.Lc, p.ld_c, p.ld_n, wave, lane);
    seek_in(vs, tb, true, L.Vc, L.Vn, p.n_kept, p.Lc, p.ld_c, p.ld_n, wave, lane);
#pragma unroll 1
    for (int i = 0; i < (KV8 ? 4 : 3); ++i) {
      issue_k_tile(i, i);
      if (i >= 2) issue_v_tile(i - 2, i - 2);
    }
    // step 0 adds the V tile in front of the first one, with weights of zero: what it reads must be finite
    {
      typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
      const u32x4 none = {0u, 0u, 0u, 0u};
      lds_byte* z = v_ring + (CK - 1) * TILEB + tid * 16;
#pragma unroll
      for (int i = 0; i < TILEB / 16 / kAtThreads; ++i) *(lds_u32x4*)(z + i * kAtThreads * 16) = none;
    }
    wait_vmcnt<0>();
    if (KV8) {  // the first product needs K(0), step 0 reads K(1)
      cook(0, 0, false);
      cook(1, 1, false);
    }
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): what was written is there before the barrier lets others read
    if (KV8) {
      // the raw ring has kAtStages slots: K(kAtStages) goes where this wave's part of K(0) was, now that it is converted
      issue_k_tile(kAtStages, 0);
      issue_v_tile(kAtStages - 2, kAtStages - 2);
    }
    __builtin_amdgcn_s_barrier();

    // A wave whose 32 queries all lie past the end (the last query tile of a head is usually ragged) still loads its
    // share of every tile and joins every barrier, but does no arithmetic: on this chip energy is time.
    if (__builtin_amdgcn_readfirstlane(i_first + qblk * 32) >= p.Lq) {
      __builtin_amdgcn_s_barrier();  // the one after the other waves' first product
#pragma unroll 1
      for (int t = 0; t < 2 * n_iter; ++t) {
        if (GATHER) issue_ids(tb + t + kAtStages + kAtIdLead);
        if (!kAblateLoads && KV8) {
          issue_k_tile(t + 5, (t + 5) % kAtStages);
          issue_v_tile(t + 3, (t + 3) % kAtStages);
        }
        if (!kAblateLoads && !KV8 && t % 2 == 0) {
          issue_k_tile(t + 3, (t + 3) % kAtStages);
          issue_k_tile(t + 4, t % kAtStages);
          issue_v_tile(t + 1, (t + 1) % kAtStages);
          issue_v_tile(t + 2, (t + 2) % kAtStages);
        }
        if (KV8) {
          cook_step(t % kAtStages, t);
          __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
        }
        if ((t + 1) % GROUP == 0) {
          wait_vmcnt<kInFlight>();
          __builtin_amdgcn_s_barrier();
        }
      }
      wait_vmcnt<0>();
    } else {
      f32x16 o[DB];
#pragma unroll
      for (int b = 0; b < DB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[b][r] = 0.f;
      f32x16 s_a[2], s_b[2];
      u32x4 p_a[4], p_b[4];
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int e = 0; e < 4; ++e) { p_a[ks][e] = 0u; p_b[ks][e] = 0u; }
      // The reference starts at a finite sentinel, not at -inf: a segment may begin with tiles that are masked
      // entirely for some queries, and (-inf) - (-inf) in the rescale factor would poison their sums.
      float msc = kAtNoMax, l_run = 0.f;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
        for (int r = 0; r < 16; ++r) s_a[kb][r] = 0.f;
#pragma unroll
        for (int kk = 0; kk < KD; ++kk) {
          const bf16x8 a = lds_read_k(k_at[kk] + kb * 32 * ROWB);
          s_a[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[kk], s_a[kb], 0, 0, 0);
        }
      }
      // Step 0 refills the ring slot of K(0): every wave must have its K(0) fragments in registers before any wave
      // issues that load.  The products above have consumed them, so one barrier here is enough; inside the loop
      // the barrier that ends step t-1 plays this role for step t.
      asm volatile("" : "+v"(s_a[0]), "+v"(s_a[1]));
      __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
      __builtin_amdgcn_s_barrier();

      // the reference starts with the maximum of the first tile (every later tile is only checked against it)
      if ((tb + 1) * kAtTileKeys > lim_min) attn_mask(s_a, tb * kAtTileKeys, lim, g);
      {
        float mx = s_a[0][0];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s_a[kb][r]);
        msc = fmaxf(msc, half_swap_max(mx) * sc);
      }

      // Step t: S^T(t+1) into the "next" registers, softmax of S^T(t), O^T += tile t-1.  Even steps go from s_a to p_a, odd
      // ones from s_b to p_b.  A segment always holds an even number of tiles: a tile past the end is fully masked and
      // contributes nothing.  Before the first tile p_b is zero, and the S^T product of the last step is never used.  The
      // steps of a turn of the ring are written out, so that every slot is a constant.
      // The two steps of a group share a barrier, and the second one's first fragments are read during the first.
      constexpr int KI = D / 32, VI = D / 8;  // slots behind which the copies start: an eighth and half of a step in
      bf16x8 kf[2], vf[2];
      auto step = [&](auto phase, int t, f32x16(&s_cur)[2], f32x16(&s_nxt)[2], const u32x4(&p_prev)[4], u32x4(&p_cur)[4]) {
        constexpr int PH = decltype(phase)::value;
        constexpr bool first = GROUP == 2 && PH % 2 == 0, second = GROUP == 2 && PH % 2 == 1;
        if (GATHER) issue_ids(tb + t + kAtStages + kAtIdLead);
        if (KV8) cook_step(PH, t);
        if (__builtin_expect((tb + t + 1) * kAtTileKeys > lim_min, 0)) attn_mask(s_cur, (tb + t) * kAtTileKeys, lim, g);
        attn_step<D, (PH + 1) % CK * TILEB, (PH + CK - 1) % CK * TILEB, second, first, (PH + 2) % CK * TILEB, PH % CK * TILEB>(
            s_cur, s_nxt, p_prev, p_cur, o, qf, msc, l_run, k_at, v_at, kf, vf, sc, [&](int i) {
              if (kAblateLoads) return;
              if (KV8) {
                if (i == KI) issue_k_tile(t + 5, (PH + 5) % kAtStages);
                if (i == VI) issue_v_tile(t + 3, (PH + 3) % kAtStages);
              } else if (first) {
                if (GATHER && i == KI - 2) read_ids(tb + t + 3);
                if (i == KI) issue_k_tile(t + 3, (PH + 3) % kAtStages, true);
                if (GATHER && i == 2 * KI - 1) read_ids(tb + t + 4);
                if (i == 2 * KI) issue_k_tile(t + 4, PH, true);
                if (GATHER && i == VI - 1) read_ids(tb + t + 1);
                if (i == VI) issue_v_tile(t + 1, (PH + 1) % kAtStages, true);
                if (GATHER && i == VI + KI - 1) read_ids(tb + t + 2);
                if (i == VI + KI) issue_v_tile(t + 2, (PH + 2) % kAtStages, true);
              }
            });
        if (KV8) __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): this step's bf16 rows are written
        if (!first) {
          wait_vmcnt<kInFlight>();
          __builtin_amdgcn_s_barrier();
        }
      };
      static_assert(kAtStages == 4, "a turn of the ring is four steps");
#pragma unroll 1
      for (int t = 0;; t += 4) {
        step(Phase<0>{}, t, s_a, s_b, p_b, p_a);
        step(Phase<1>{}, t + 1, s_b, s_a, p_a, p_b);
        if (t + 2 >= 2 * n_iter) break;
        step(Phase<2>{}, t + 2, s_a, s_b, p_b, p_a);
        step(Phase<3>{}, t + 3, s_b, s_a, p_a, p_b);
        if (t + 4 >= 2 * n_iter) break;
      }
      // the last tile's contribution
      {
        const int last = (2 * n_iter - 1) % CK * TILEB;
#pragma unroll
        for (int m = 0; m < 4 * DB; ++m) {
          const bf16x8 a = lds_read_vt(v_at[m % DB] + last + (16 * (m / DB)) * ROWB, 8 * ROWB);
          o[m % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, as_bf16x8(p_b[m / DB]), o[m % DB], 0, 0, 0);
        }
      }
      wait_vmcnt<0>();  // nothing may still be writing this workgroup's LDS when the ring is reused or it retires

      // store: lane holds query c, d = 32 b + 8 (r/4) + 4 g + (r%4)
      const float l_tot = half_swap_sum(l_run);
      if (whole) {  // normalise and write O
        const float inv = 1.0f / l_tot;
        if (q_row < p.Lq) {
#pragma unroll
          for (int b = 0; b < DB; ++b)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
              const int d0 = 32 * b + 8 * q4 + 4 * g;
              const float v0 = o[b][4 * q4 + 0] * inv, v1 = o[b][4 * q4 + 1] * inv;
              const float v2 = o[b][4 * q4 + 2] * inv, v3 = o[b][4 * q4 + 3] * inv;
              const long long off = (long long)q_row * p.ld_o + head_off + d0;
              if (OUT_F32) {
                *reinterpret_cast<float4*>(static_cast<float*>(L.O) + off) = make_float4(v0, v1, v2, v3);
              } else {
                bf16x4 ob;
                ob[0] = (__bf16)v0; ob[1] = (__bf16)v1; ob[2] = (__bf16)v2; ob[3] = (__bf16)v3;
                *reinterpret_cast<bf16x4*>(static_cast<unsigned short*>(L.O) + off) = ob;
              }
            }
        }
      } else if (q_row < p.Lq) {  // partial result of this segment, for attn_combine_kernel
        const int pslot = 2 * wg + (first_segment ? 0 : 1);
        const int ql = qblk * 32 + c;
        float* po = wk.part_o + ((long long)pslot * kAtBQ + ql) * D;
#pragma unroll
        for (int b = 0; b < DB; ++b)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4)
            *reinterpret_cast<float4*>(po + 32 * b + 8 * q4 + 4 * g) =
                make_float4(o[b][4 * q4 + 0], o[b][4 * q4 + 1], o[b][4 * q4 + 2], o[b][4 * q4 + 3]);
        if (g == 0) {
          float* pml = wk.part_ml + (long long)pslot * 2 * kAtBQ;
          pml[ql] = msc;
          pml[kAtBQ + ql] = l_tot;
        }
      }
    }
    // ---- next segment: the next item of the list, from its first unit
    first_segment = false;
    room -= n_iter;
    if (!is_run || room <= 0) break;
    __builtin_amdgcn_s_barrier();  // every wave has finished reading the ring before it is refilled
    from = 0;
    if (++qt == wk.n_qt) { qt = 0; ++h; }
  }
}

// Merges the partial results of the items that more than one workgroup worked on, in run order, whoever wrote them first:
//   O = sum_p 2^(m_p - m) O_p / sum_p 2^(m_p - m) l_p   with m = max_p m_p.
// D / 4 lanes take one query row (16 bytes of every partial result each), a wave 256 / D rows, a workgroup four waves:
// the launch is bound by the latency of its chain (maxima, then weights and rows), so rows are spread as wide as they
// go instead of being walked by a few workgroups per item.
// What precedes the loads is kept short: with 64-bit divisions and a walk over the query tiles before its own, the merge of
// 156 items of 13 unequal tiles (12 heads of 128, 3121 queries) took 26.6 us, now 16.1 (67 MB of partial results).
__device__ __forceinline__ long long attn_div(long long x, long long by, long long most) {  // x / by, 0 <= x <= most
  if (most < 1ll << 32) return (unsigned)x / (unsigned)by;
  return x / by;
}
template <int D>
constexpr int kAtCombineRows = 4 * 256 / D;  // rows per workgroup
template <int D, bool OUT_F32>
__global__ __launch_bounds__(256) void attn_combine_kernel(AttnArgs args) {
  const AttnParams& p = args.p;
  const AttnWork& wk = args.w;
  constexpr int kBands = kAtBQ / kAtCombineRows<D>;
  const int item = wk.n_whole + blockIdx.x / kBands, band = blockIdx.x % kBands;
  const int h = item / wk.n_qt, qt = item - h * wk.n_qt;
  const int row = band * kAtCombineRows<D> + threadIdx.x / (D / 4);  // query row inside the item
  const int q_row = qt * kAtBQ + row;
  if (qt * kAtBQ + band * kAtCombineRows<D> >= p.Lq) return;
  int pre = 0;
  if (wk.uniform) {
    pre = qt * wk.uniform;
  } else {  // one query tile per lane: a walk over them is as long as the rest of the kernel
    for (int q2 = threadIdx.x & 63; q2 < qt; q2 += 64) pre += attn_units(q2, p.Lq, p.n_kept, p.Lc, p.block_len);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) pre += __shfl_xor(pre, off);
    pre = uniform_i32(pre);
  }
  const int units = uniform_i32(attn_units(qt, p.Lq, p.n_kept, p.Lc, p.block_len));
  const long long U = wk.U, G = wk.n_runs;
  const long long s = (long long)h * wk.units_head + pre - wk.u0, e = s + units;
  // the run that holds unit x: the largest g with floor(g U / G) <= x
  const int g_first = (int)attn_div((s + 1) * G - 1, U, U * G), g_last = (int)attn_div(e * G - 1, U, U * G);
  if (g_first == g_last || q_row >= p.Lq) return;  // one workgroup saw the whole item and wrote O itself
  // slot of run gg's partial result for this item: 2 gg if the run starts inside the item, else 2 gg + 1
  const int slot_first = 2 * g_first + (attn_div(g_first * U, G, U * G) >= s ? 0 : 1);
  auto slot_of = [&](int gg) { return gg == g_first ? slot_first : 2 * gg; };
  const int d0 = 4 * (threadIdx.x % (D / 4));
  // All that is needed of up to kAhead runs is asked for at once (run by run it was a wait for memory each, twice); most items
  // have no more.  1560 queries (12 heads of 128, three runs per item) 10.5 -> 8.4 us, 3121 (unequal items) 16.5 -> 13.9.
  constexpr int kAhead = 4;
  struct Run {
    float m, l;
    float4 v;
  };
  auto fetch = [&](int gg, bool with_v) {
    const long long sl = slot_of(gg < g_last ? gg : g_last);
    const float* ml = wk.part_ml + sl * 2 * kAtBQ + row;
    Run r;
    r.m = ml[0];
    r.l = with_v ? ml[kAtBQ] : 0.f;
    r.v = with_v ? *reinterpret_cast<const float4*>(wk.part_o + (sl * kAtBQ + row) * D + d0) : make_float4(0.f, 0.f, 0.f, 0.f);
    return r;
  };
  Run first[kAhead];
#pragma unroll
  for (int i = 0; i < kAhead; ++i) first[i] = fetch(g_first + i, true);
  float m = kAtNoMax;
#pragma unroll
  for (int i = 0; i < kAhead; ++i) m = fmaxf(m, first[i].m);  // (the last run again where there are fewer)
#pragma unroll 4
  for (int gg = g_first + kAhead; gg <= g_last; ++gg) m = fmaxf(m, fetch(gg, false).m);
  float l = 0.f;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  auto add = [&](const Run& r) {
    const float wgt = __builtin_amdgcn_exp2f(r.m - m);
    l += r.l * wgt;
    acc.x = fmaf(r.v.x, wgt, acc.x); acc.y = fmaf(r.v.y, wgt, acc.y);
    acc.z = fmaf(r.v.z, wgt, acc.z); acc.w = fmaf(r.v.w, wgt, acc.w);
  };
#pragma unroll
  for (int i = 0; i < kAhead; ++i)
    if (g_first + i <= g_last) add(first[i]);
#pragma unroll 4
  for (int gg = g_first + kAhead; gg <= g_last; ++gg) add(fetch(gg, true));
  const float inv = 1.0f / l;
  const int layer = h < p.N_heads ? 0 : h / p.N_heads;
  void* const O = args.layer[layer].O;
  const long long off = (long long)q_row * p.ld_o + (long long)(h - layer * p.N_heads) * D + d0;
  if (OUT_F32) {
    *reinterpret_cast<float4*>(static_cast<float*>(O) + off) = make_float4(acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv);
  } else {
    bf16x4 ob;
    ob[0] = (__bf16)(acc.x * inv); ob[1] = (__bf16)(acc.y * inv); ob[2] = (__bf16)(acc.z * inv); ob[3] = (__bf16)(acc.w * inv);
    *reinterpret_cast<bf16x4*>(static_cast<unsigned short*>(O) + off) = ob;
  }
}

// ---- few queries over few keys --------------------------------------------------------------------------------------
// A workgroup takes 32 queries of one head.  Such a call is bound by latency: of arguments, of the first loads, of code that has
// to be fetched.  So each of the eight waves asks for all of one key tile at once (K and V rows into registers, from there
// through its own piece of LDS), there is no ring and no pipeline, and the code is a fraction of the long kernel's.  (2 heads of
// 64, 64 queries over 192 keys: the long kernel spends 2.6 k clocks per 64 keys, because every step's code is new to the CU.)
//
// The arithmetic is the long kernel's, operation for operation, so that a query's result has the same bits whichever of the two
// takes it (how many heads, layers or queries share a launch decides that): the reference is the first tile's maximum, S^T and
// the weights of up to eight tiles are formed side by side, and O^T and the sum of the weights take the tiles in order, in one
// wave per 32 rows of O^T.  A tile that outgrows the reference is rare: then the waves work out the weights of these tiles once
// more, one tile after the other.
//
// What bounds it: the chain of launch, arguments, rows (and ids in front of them), two barriers, and the tiles of a turn in
// order.  Each wave on its own over every eighth tile, with its own reference, and the eight results merged, gave other bits
// than the long kernel, and gathered rows, whose addresses were worked out in 64 bits for K and again for V, spilled 24
// registers at head dim 128.  That form / this one, calls back to back: 2 heads of 64, 64 queries over 192 keys 4.9 / 4.5 us
// (gathered 7.5 / 4.7), 32 heads, 256 over 1536 keys 22.5 / 12.7 (39.1 / 14.0; now by XCD), 16 heads of 128, 128 over 328
// keys 11.1 / 7.9 (15.7 / 8.3).
constexpr int kSmWaves = 8;
constexpr int kSmQ = 32;                       // queries per workgroup
// Where it is used: up to kSmGroups workgroups (one per CU: two of them on some CUs take twice as long) and kSmTiles key tiles (a
// workgroup takes in all keys of its head, where the long kernel, with a workspace, shares them among CUs; at head dim 128 no
// more fit the LDS side by side), gathered or not, with a workspace or without.  Calls back to back, this / the long kernel
// whole / cut with a workspace.  Head dim 64, 24 tiles: 4 workgroups 11.7 / 17.0 / 10.9 us, 256 12.5 / 25.7 / 21.3 (gathered
// 14.2 / 29.7 / 22.7), 320 23.5 / 26.0 / 22.4; 32 tiles: 4 workgroups 14.6 / 21.0 / 10.6, 40 15.0 / 29.4 / 14.0.  Head dim
// 128 (too short to be cut): 3 tiles, 64 workgroups 6.7 / 14.2; 7 tiles, 64 8.2 / 16.2, 256 8.7 / 16.2 (gathered 9.3 / 18.8);
// 6 tiles, 256 8.0 / 13.7, 320 14.8 / 14.5.
constexpr int kSmGroups = 256;
constexpr int kSmTiles64 = 24, kSmTiles128 = 7;
template <int D>
struct SmallLds {  // bytes from the start of the LDS
  static constexpr int slots = D == 64 ? kSmWaves : kSmTiles128;        // tiles side by side
  static constexpr int rounds = D == 64 ? (kSmTiles64 + kSmWaves - 1) / kSmWaves : 1;
  static constexpr int tile = kAtTileKeys * 2 * D;
  static constexpr int weights = slots * tile;                          // [slot][key slice][lane] 16 bytes: P^T fragments
  static constexpr int sums = weights + slots * 4 * 64 * 16;            // [slot][lane] fp32: sums of the weights
  static constexpr int alphas = sums + slots * 64 * 4;                  // [slot][query] fp32: what a raise scales O^T by
  static constexpr int msc = alphas + slots * kSmQ * 4;                 // [query] fp32: the reference
  static constexpr int outgrown = msc + kSmQ * 4;                       // [wave]: has its tile outgrown the reference?
  static constexpr int bytes = outgrown + kSmWaves * 4;
  static_assert(slots <= kSmWaves && bytes <= 160 * 1024, "");
};
static_assert(kSmTiles128 <= SmallLds<128>::slots, "head dim 128: all tiles side by side");

template <int D, bool OUT_F32, bool GATHER>
__global__ __launch_bounds__(kSmWaves * 64, 1) void attn_small_kernel(AttnArgs args) {
  constexpr int ROWB = 2 * D, CH = D / 8, RPB = 256 / ROWB, KD = D / 16, DB = D / 32;
  constexpr int VR = 64 / CH, VL = kAtTileKeys / VR;  // rows per wave-wide load, loads per tile
  typedef SmallLds<D> Lds;
  typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
  typedef __attribute__((address_space(3))) float lds_float;
  typedef __attribute__((address_space(3))) int lds_int;
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds_raw[];
  lds_byte* const lds = (lds_byte*)lds_raw;
  lds_float* const msc_of = (lds_float*)(lds + Lds::msc);
  lds_int* const outgrown = (lds_int*)(lds + Lds::outgrown);
  const AttnParams& p = args.p;
  AttnLayer L = args.layer[0];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, c = lane & 31;
  // XCD x (workgroups x, x + 8, ...) takes one contiguous range of the groups, head by head: its L2 then sees the K/V of an
  // eighth of the heads
  const int xcd = blockIdx.x % kAtXcds, per_xcd = gridDim.x / kAtXcds, more = gridDim.x % kAtXcds;
  const int group = xcd * per_xcd + (xcd < more ? xcd : more) + blockIdx.x / kAtXcds;
  const int n_qb = (p.Lq + kSmQ - 1) / kSmQ;
  const int h = uniform_i32(group / n_qb), q0 = (group - h * n_qb) * kSmQ;
  const int layer = h < p.N_heads ? 0 : uniform_i32(h / p.N_heads);
  if (layer != 0) L = args.layer[layer];
  const long long head_off = (long long)(h - layer * p.N_heads) * D;
  const int n_total = p.n_kept + p.Lc;
  const int q_row = q0 + c < p.Lq ? q0 + c : p.Lq - 1;
  int lim = n_total, vis_first = n_total, vis = n_total;  // visible keys: of this lane's query, the first one, the last one
  if (p.block_len < p.Lc) {
    auto visible = [&](int i) {
      const long long e = ((long long)(i / p.block_len) + 1) * p.block_len;
      return p.n_kept + (int)(e < p.Lc ? e : p.Lc);
    };
    lim = visible(q_row);
    vis_first = uniform_i32(visible(q0));
    vis = uniform_i32(visible(q0 + kSmQ - 1 < p.Lq ? q0 + kSmQ - 1 : p.Lq - 1));
  }
  const int tiles = (vis + kAtTileKeys - 1) / kAtTileKeys;
  lds_byte* const tile_lds = lds + wave * Lds::tile;  // (head dim 128: waves past the last slot have no tile)
  // what a wave has written to the LDS is there, and no access moves over the line; loads from global memory stay in flight
  auto sync = [] {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  auto in_order = [] { asm volatile("" ::: "memory"); };  // (one wave's LDS operations keep the order they are written in)

  // ---- a tile's rows: 16 bytes of row VR j + lane / CH per load
  u32x4 kv[VL], vv[VL];
  int ids = 0;  // GATHER: lane l holds the cache row behind row l of the wave's next tile, never outside the cache
  auto fetch_ids = [&](int t) {
    if (!GATHER) return;
    const int at = t * kAtTileKeys + lane;
    const int id = p.ids[at < p.n_kept ? at : p.n_kept - 1];
    ids = id < 0 ? 0 : (id < p.n_cache ? id : p.n_cache - 1);
  };
  auto fetch = [&](int t) {
    const int key0 = t * kAtTileKeys;
    const unsigned ldc_b = (unsigned)(p.ld_c * 2), ldn_b = (unsigned)(p.ld_n * 2);  // (64 rows span less than 4 GiB)
    const unsigned chunk16 = 16 * (lane % CH);
    const bool cache = key0 + kAtTileKeys <= p.n_kept;
    const int from = key0 < p.n_kept ? 0 : key0 - p.n_kept;  // chunk row that the chunk's offsets count from
    const char* const kc = static_cast<const char*>(L.Kc) + 2 * head_off + (GATHER ? 0 : (long long)key0 * ldc_b);
    const char* const vc = static_cast<const char*>(L.Vc) + 2 * head_off + (GATHER ? 0 : (long long)key0 * ldc_b);
    const char* const kn = static_cast<const char*>(L.Kn) + 2 * head_off + (long long)from * ldn_b;
    const char* const vn = static_cast<const char*>(L.Vn) + 2 * head_off + (long long)from * ldn_b;
    if (cache || (key0 >= p.n_kept && key0 + kAtTileKeys <= n_total)) {  // one segment: scalar bases
      const char *const kb = cache ? kc : kn, *const vb = cache ? vc : vn;
      const unsigned ld_b = cache ? ldc_b : ldn_b;
      unsigned off[VL];
#pragma unroll
      for (int j = 0; j < VL; ++j) {
        const unsigned row = GATHER && cache ? (unsigned)__shfl(ids, VR * j + lane / CH) : (unsigned)(VR * j + lane / CH);
        off[j] = row * ld_b + chunk16;  // (a gathered cache is smaller than 4 GiB)
      }
#pragma unroll
      for (int j = 0; j < VL; ++j) kv[j] = *reinterpret_cast<const u32x4*>(kb + off[j]);
#pragma unroll
      for (int j = 0; j < VL; ++j) vv[j] = *reinterpret_cast<const u32x4*>(vb + off[j]);
    } else {  // both segments, or the end of the keys (rows past it are masked: a valid one instead)
      unsigned off[VL];
      unsigned in_cache = 0;
#pragma unroll
      for (int j = 0; j < VL; ++j) {
        int key = key0 + VR * j + lane / CH;
        key = key < n_total ? key : n_total - 1;
        const bool old = key < p.n_kept;
        const unsigned cache_row = GATHER ? (unsigned)__shfl(ids, VR * j + lane / CH) : (unsigned)(key - key0);
        off[j] = (old ? cache_row * ldc_b : (unsigned)(key - p.n_kept - from) * ldn_b) + chunk16;
        in_cache |= old ? 1u << j : 0u;
      }
#pragma unroll
      for (int j = 0; j < VL; ++j) {
        kv[j] = *reinterpret_cast<const u32x4*>((in_cache >> j & 1 ? kc : kn) + off[j]);
        in_order();  // (all addresses at once would be more than the registers hold)
      }
#pragma unroll
      for (int j = 0; j < VL; ++j) {
        vv[j] = *reinterpret_cast<const u32x4*>((in_cache >> j & 1 ? vc : vn) + off[j]);
        in_order();
      }
    }
    in_order();
  };
  auto to_lds = [&](const u32x4(&x)[VL], bool is_v) {  // with the swizzles of the long kernel
#pragma unroll
    for (int j = 0; j < VL; ++j) {
      const int row = VR * j + lane / CH;
      const int ch = (lane % CH) ^ (is_v ? 4 * ((row / RPB) & (CH / 4 - 1)) : (row / RPB) & (CH - 1));
      *(lds_u32x4*)(tile_lds + row * ROWB + (ch << 4)) = x[j];
    }
    in_order();
  };

  if (wave < tiles) fetch_ids(wave);
  bf16x8 qf[KD];
  {
    const unsigned short* qp = static_cast<const unsigned short*>(L.Q) + (long long)q_row * p.ld_q + head_off + 8 * g;
#pragma unroll
    for (int kk = 0; kk < KD; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(qp + 16 * kk);
  }
  if (wave < tiles) {
    fetch(wave);
    if (Lds::rounds > 1 && wave + kSmWaves < tiles) fetch_ids(wave + kSmWaves);
  }
  // K and V^T fragments: as in the long kernel
  const int kx2 = g ^ ((c / RPB) & (CH - 1));
  const lds_byte* const k_rd = tile_lds + c * ROWB;
  const int i16 = lane & 15, rr = 4 * g + (i16 >> 2);
  const int vx2 = 4 * ((rr / RPB) & (CH / 4 - 1));
  const int d_block = wave < DB ? wave : 0;  // rows of O^T that this wave adds up
  const lds_byte* const v_rd = lds + rr * ROWB + ((i16 & 1) << 3) + ((2 * ((lane >> 4) & 1) + ((i16 & 3) >> 1)) << 4) +
                               (((4 * d_block) ^ vx2) << 4);
  lds_u32x4* const p_at = (lds_u32x4*)(lds + Lds::weights) + lane;  // + (4 slot + key slice) * 64
  lds_float* const sum_at = (lds_float*)(lds + Lds::sums) + lane;   // + 64 slot
  lds_float* const alpha_at = (lds_float*)(lds + Lds::alphas) + c;  // + kSmQ slot
  const float sc = p.scale_log2;
  f32x16 o;
#pragma unroll
  for (int r = 0; r < 16; ++r) o[r] = 0.f;
  float l_run = 0.f;

#pragma unroll 1
  for (int t0 = 0;; t0 += kSmWaves) {
    const int t = t0 + wave, n_here = tiles - t0 < kSmWaves ? tiles - t0 : kSmWaves;
    const bool busy = t < tiles;
    f32x16 s[2];
    u32x4 pw[4];
    float msc = kAtNoMax, psum = 0.f;
    auto weigh = [&] {  // the tile's weights relative to msc, in the order of the long kernel
      psum = 0.f;
#pragma unroll
      for (int e = 0; e < 32; e += 2) {
        const float p0 = __builtin_amdgcn_exp2f(fmaf(s[e >> 4][e & 15], sc, -msc));
        const float p1 = __builtin_amdgcn_exp2f(fmaf(s[e >> 4][(e & 15) + 1], sc, -msc));
        psum += p0;
        psum += p1;
        pw[e >> 3][(e & 7) >> 1] = pack_bf16(p0, p1);
      }
    };
    auto hand_over = [&] {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) p_at[(4 * wave + ks) * 64] = pw[ks];
      sum_at[64 * wave] = psum;
    };
    if (busy) {
      to_lds(kv, false);
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
        for (int r = 0; r < 16; ++r) s[kb][r] = 0.f;
#pragma unroll
        for (int kk = 0; kk < KD; ++kk)
          s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_read_k(k_rd + kb * 32 * ROWB + (((2 * kk) ^ kx2) << 4)), qf[kk],
                                                          s[kb], 0, 0, 0);
      }
      in_order();
      to_lds(vv, true);
      if ((t + 1) * kAtTileKeys > vis_first) attn_mask(s, t * kAtTileKeys, lim, g);
      if (Lds::rounds > 1 && t + kSmWaves < tiles) {
        fetch(t + kSmWaves);
        if (t + 2 * kSmWaves < tiles) fetch_ids(t + 2 * kSmWaves);
      }
    }
    if (t0 == 0) {  // the reference starts with the maximum of the first tile
      if (wave == 0) {
        float mx = s[0][0];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kb][r]);
        msc = fmaxf(kAtNoMax, half_swap_max(mx) * sc);
        if (g == 0) msc_of[c] = msc;
      }
      sync();
    }
    msc = msc_of[c];
    bool over = false;
    if (busy) {
      weigh();
      hand_over();
      over = __builtin_amdgcn_ballot_w64(psum > kAtMaxTileSum) != 0;
    }
    if (lane == 0) outgrown[wave] = over;
    sync();
    int any = 0;
#pragma unroll
    for (int w = 0; w < kSmWaves; ++w) any |= outgrown[w];
    const bool raised = uniform_i32(any) != 0;
    if (raised) {
#pragma unroll 1
      for (int w = 0; w < n_here; ++w) {
        if (w == wave) {
          msc = msc_of[c];
          weigh();
          float alpha = 1.f, unused = 0.f;
          if (__builtin_amdgcn_ballot_w64(psum > kAtMaxTileSum) != 0) alpha = attn_raise(s, pw, sc, msc, unused, psum);
          hand_over();
          if (g == 0) {
            alpha_at[kSmQ * w] = alpha;
            msc_of[c] = msc;
          }
        }
        sync();
      }
    }
    if (wave < DB) {
      u32x4 pf[4];
      bf16x8 vf[4];
      auto read = [&](int w, int ks) {
        pf[ks] = p_at[(4 * w + ks) * 64];
        vf[ks] = lds_read_vt(v_rd + w * Lds::tile + 16 * ks * ROWB, 8 * ROWB);
      };
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) read(0, ks);
#pragma unroll 1
      for (int w = 0; w < n_here; ++w) {
        const int w_next = w + 1 < n_here ? w + 1 : w;
        if (raised) {
          const float alpha = alpha_at[kSmQ * w];
          l_run *= alpha;
#pragma unroll
          for (int r = 0; r < 16; ++r) o[r] *= alpha;
        }
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          o = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[ks], as_bf16x8(pf[ks]), o, 0, 0, 0);
          read(w_next, ks);
        }
        l_run += sum_at[64 * w];
      }
    }
    if (Lds::rounds == 1 || t0 + kSmWaves >= tiles) break;
    sync();  // the tiles and their weights have been used
  }
  if (wave >= DB || q0 + c >= p.Lq) return;
  // lane holds query c, d = 32 wave + 8 (r/4) + 4 g + (r%4)
  const float inv = 1.0f / half_swap_sum(l_run);
#pragma unroll
  for (int q4 = 0; q4 < 4; ++q4) {
    const long long off = (long long)q_row * p.ld_o + head_off + 32 * wave + 8 * q4 + 4 * g;
    if (OUT_F32) {
      *reinterpret_cast<float4*>(static_cast<float*>(L.O) + off) =
          make_float4(o[4 * q4] * inv, o[4 * q4 + 1] * inv, o[4 * q4 + 2] * inv, o[4 * q4 + 3] * inv);
    } else {
      bf16x4 ob;
#pragma unroll
      for (int i = 0; i < 4; ++i) ob[i] = (__bf16)(o[4 * q4 + i] * inv);
      *reinterpret_cast<bf16x4*>(static_cast<unsigned short*>(L.O) + off) = ob;
    }
  }
}

template <int D, bool OUT_F32, bool GATHER>
int launch_small(hipStream_t st, const AttnArgs& a, int heads) {
  static LdsLimit lds_limit;
  const int rc = set_lds_limit(lds_limit, attn_small_kernel<D, OUT_F32, GATHER>, SmallLds<D>::bytes);
  if (rc != PAFU_OK) return rc;
  hipLaunchKernelGGL((attn_small_kernel<D, OUT_F32, GATHER>), dim3(heads * ((a.p.Lq + kSmQ - 1) / kSmQ)),
                     dim3(kSmWaves * 64), SmallLds<D>::bytes, st, a);
  return check_launch();
}
template <bool GATHER>
int launch_small_dims(hipStream_t st, const AttnArgs& a, int heads, int D, bool f32) {
  if (D == 128) return f32 ? launch_small<128, true, GATHER>(st, a, heads) : launch_small<128, false, GATHER>(st, a, heads);
  return f32 ? launch_small<64, true, GATHER>(st, a, heads) : launch_small<64, false, GATHER>(st, a, heads);
}

template <int D, bool OUT_F32, bool GATHER, bool KV8 = false>
int launch_variant(hipStream_t st, const AttnArgs& a) {
  static LdsLimit lds_limit;
  const int rc = set_lds_limit(lds_limit, chunk_attention_kernel<D, OUT_F32, GATHER, KV8>, attn_lds_bytes(D, GATHER));
  if (rc != PAFU_OK) return rc;
  hipLaunchKernelGGL((chunk_attention_kernel<D, OUT_F32, GATHER, KV8>), dim3(a.w.n_whole + a.w.n_runs), dim3(kAtThreads),
                     attn_lds_bytes(D, GATHER), st, a);
  if (a.w.n_runs)
    hipLaunchKernelGGL((attn_combine_kernel<D, OUT_F32>),
                       dim3((a.w.n_items - a.w.n_whole) * (kAtBQ / kAtCombineRows<D>)), dim3(256), 0, st, a);
  return check_launch();
}

template <bool GATHER>
int launch_dims(hipStream_t st, const AttnArgs& a, int D, bool f32) {
  if (D == 128) return f32 ? launch_variant<128, true, GATHER>(st, a) : launch_variant<128, false, GATHER>(st, a);
  return f32 ? launch_variant<64, true, GATHER>(st, a) : launch_variant<64, false, GATHER>(st, a);
}

}  // namespace

int attention_study_build() { return PAFU_ATTN_ABLATE; }

// Bytes of workspace with which every launch can cut its work into equal runs: two partial-result slots for each of
// at most kAtMaxRuns workgroups.
size_t attention_workspace_bytes(int D) {
  return (size_t)2 * kAtMaxRuns * ((size_t)kAtBQ * D + 2 * kAtBQ) * sizeof(float);
}

int launch_attention(hipStream_t st, const AttnLayer* layers, int n_layers, int Lq, int n_kept, int Lc, int N, int D,
                     long long ld_q, long long ld_c, long long ld_n, long long ld_o, int block_len, float scale,
                     int out_dtype, void* workspace, size_t workspace_bytes, const int* ids, int n_cache, int kv_dtype,
                     float k_scale, float v_scale) {
  AttnArgs a;
  AttnParams& p = a.p;
  for (int l = 0; l < n_layers; ++l) a.layer[l] = layers[l];
  p.ids = ids;
  p.n_cache = n_cache;
  p.ld_q = ld_q; p.ld_c = ld_c; p.ld_n = ld_n; p.ld_o = ld_o;
  p.Lq = Lq; p.n_kept = n_kept; p.Lc = Lc; p.N_heads = N;
  p.block_len = block_len < Lc ? block_len : Lc;  // blocks at least as long as the chunk mean "no mask"
  p.scale_log2 = scale * 1.44269504088896340736f;
  p.k_scale = k_scale;
  p.v_scale = v_scale;

  const bool f32 = out_dtype == PAFU_F32, gather = ids != nullptr && n_kept > 0;
  const long long tiles = ((long long)n_kept + Lc + kAtTileKeys - 1) / kAtTileKeys;
  const long long groups = (long long)N * n_layers * ((Lq + kSmQ - 1) / kSmQ);
  if (kv_dtype == PAFU_BF16 && tiles <= (D == 64 ? kSmTiles64 : kSmTiles128) && groups <= kSmGroups)
    return gather ? launch_small_dims<true>(st, a, N * n_layers, D, f32) : launch_small_dims<false>(st, a, N * n_layers, D, f32);

  AttnWork& w = a.w;
  w.n_qt = (Lq + kAtBQ - 1) / kAtBQ;
  long long units_head = 0;
  const int u0_item = attn_units(0, Lq, n_kept, Lc, p.block_len);
  bool uniform = true;
  for (int qt = 0; qt < w.n_qt; ++qt) {
    const int cq = attn_units(qt, Lq, n_kept, Lc, p.block_len);
    units_head += cq;
    uniform = uniform && cq == u0_item;
  }
  w.units_head = (int)units_head;
  w.uniform = uniform ? u0_item : 0;
  const long long heads = (long long)N * n_layers, items = heads * w.n_qt;
  int cus = compute_units();
  if (cus > kAtMaxRuns) cus = kAtMaxRuns;
  w.n_items = (int)items;
  w.n_whole = (int)items;
  w.n_runs = 0;
  w.u0 = w.U = 0;
  w.h0 = w.r0 = 0;
  w.part_o = nullptr;
  w.part_ml = nullptr;
  // Cut the last round when it fills at most four fifths of the CUs (above that the launch is limited by power, not by CU
  // time, and the merge pass only adds to it: 228 items on 256 CUs were 4 percent slower) and the cut shortens it by more
  // than the merge pass takes.  Measured against whole items, start / now: 12 items of 57 units (51 queries over 7154
  // keys, D = 64) 122 / 25 us; 12 of 44 units 126 / 28 us; 5 of 10 units (D = 64) 29 / 17 us; 84 of 71: 194 / 168 us (3 runs per item
  // instead of 256 equal ones: 183); 272 of 44 (D = 64): 412 / 234 us; 520 of 36: 745 / 539 us.
  const long long last = items % cus;  // items of the last round
  const bool mixed = items > last && cus % kAtXcds != 0;  // (the kernel's XCD mapping needs whole rounds of XCDs)
  if (last > 0 && last * 5 <= (long long)cus * 4 && !mixed && workspace != nullptr) {
    const int first_cut = (int)(items - last);
    long long u0 = (long long)(first_cut / w.n_qt) * units_head;
    for (int qt = 0; qt < first_cut % w.n_qt; ++qt) u0 += attn_units(qt, Lq, n_kept, Lc, p.block_len);
    const long long U = units_head * heads - u0;
    int longest = 0;  // what the last round takes without a cut
    for (int qt = 0; qt < w.n_qt; ++qt) {
      const int cq = attn_units(qt, Lq, n_kept, Lc, p.block_len);
      longest = cq > longest ? cq : longest;
    }
    long long runs = U / kAtMinRunUnits < cus ? U / kAtMinRunUnits : cus;
    if (uniform && u0_item >= 2 * kAtMinRunUnits && last * 2 <= cus) {
      // the same number of runs in every item, unless that leaves too much of the chip idle: a run that crosses from one
      // item to the next starts twice (queries, ring, first product), which takes about as long as 3/2 units
      long long per_item = cus / last < u0_item / kAtMinRunUnits ? cus / last : u0_item / kAtMinRunUnits;
      const long long run = (u0_item + per_item - 1) / per_item;
      per_item = (u0_item + run - 1) / run;
      if (2 * run <= 2 * ((U + runs - 1) / runs) + 3) runs = per_item * last;
    }
    const size_t need = (size_t)2 * runs * ((size_t)kAtBQ * D + 2 * kAtBQ) * sizeof(float);
    const long long r0 = u0 - (long long)(first_cut / w.n_qt) * units_head;
    // (r0 + U: the kernel finds a run's first item in 32 bits)
    if (runs > last && longest - (U + runs - 1) / runs >= kAtMinCutGain && r0 + U < 1ll << 31 && workspace_bytes >= need &&
        (reinterpret_cast<uintptr_t>(workspace) & 15u) == 0) {
      w.n_whole = first_cut;
      w.n_runs = (int)runs;
      w.u0 = u0;
      w.U = U;
      w.h0 = first_cut / w.n_qt;
      w.r0 = (int)r0;
      w.part_o = static_cast<float*>(workspace);
      w.part_ml = w.part_o + (size_t)2 * runs * kAtBQ * D;
    }
  }
  if (kv_dtype == PAFU_FP8_E4M3)  // validated by the caller: head dim 128, no index list
    return f32 ? launch_variant<128, true, false, true>(st, a) : launch_variant<128, false, false, true>(st, a);
  return gather ? launch_dims<true>(st, a, D, f32) : launch_dims<false>(st, a, D, f32);
}

}  // namespace pafu
