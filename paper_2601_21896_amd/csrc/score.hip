// Salience Estimation Head (S-MLP) forward: s[t] = mean_o( W2 . act(W1 . x[t] + b1) + b2 ).
// App. A "S-MLP" and Sec. 3.3-3.4 of the paper (two linear layers, SiLU in between, mean over outputs).
//
// The mean over the outputs of a linear layer is a linear layer with the averaged weight row: some launches average a
// few rows of W2/b2 themselves, for many rows a tiny pre-kernel folds them into one row w2bar[M] and a scalar; layer 1,
// the activation, the dot with the averaged row and the bias are one pass over X.
//
// bf16 paths: layer 1 is a skinny dense contraction [M x F] . [F x T], so it runs on the matrix cores
// (v_mfma_f32_32x32x16_bf16, fp32 accumulate).  H = W1.X is produced as H^T tiles (rows = hidden units,
// columns = tokens), so one lane holds 16 hidden units of ONE token per tile and the reduction over hidden
// units is almost entirely in-register.
//  - score_stream_kernel (M a multiple of 256): the measured path.
//    W1 and the features both stream global -> LDS through a ring of 64-feature slabs; a workgroup owns several 32-token
//    tiles so that one W1 fragment feeds several matrix instructions.  Described in detail above the kernel.
//    In a rollout step one extra workgroup of this launch runs the top-k selection on the stored score list
//    (select_body.h), which does not depend on the chunk's scores (Alg. 2: Top-k before the chunk is appended).
//  - score_mfma_kernel (M a multiple of 32): a wave owns 32 tokens and loads their feature rows straight
//    into B-operand registers; W1 is staged through LDS in 64-feature slabs shared by the waves of a workgroup.
//
// fp32 inputs, or shapes the tiles do not divide: plain fp32 FMAs, through LDS tiles where rows are whole 16-byte chunks.
//
// A score is compared with scores of other launches (a rollout selects on a list that many chunks have added to), so its
// bits are a function of the token and the head alone: whatever the number of tokens, the layers in the launch and the
// scratch, the same kernel's order of sums is kept.
#include "pafu_internal.h"
#include "select_body.h"

namespace pafu {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

__device__ __forceinline__ float bf16_bits_to_f32(unsigned short b) { return __uint_as_float((uint32_t)b << 16); }

__device__ __forceinline__ float act_accurate(float h, int act) {
  if (act == PAFU_ACT_SILU) return h / (1.0f + expf(-h));
  return 0.5f * h * (1.0f + erff(h * 0.70710678118654752440f));
}

// w2bar[m] = mean_o W2[o][m];  w2bar[M] = mean_o b2[o]
__global__ void fold_w2_kernel(const float* __restrict__ W2, const float* __restrict__ b2, int M, int n_out,
                               float* __restrict__ w2bar) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  const float inv = 1.0f / (float)n_out;
  if (m < M) {
    float s = 0.f;
    for (int o = 0; o < n_out; ++o) s += W2[(long long)o * M + m];
    w2bar[m] = s * inv;
  } else if (m == M) {
    float s = 0.f;
    if (b2 != nullptr)
      for (int o = 0; o < n_out; ++o) s += b2[o];
    w2bar[M] = s * inv;
  }
}

// What a launch of the tiled kernels scores: up to kScoreBatchMax layers of one geometry.
struct ScoreArgs {
  int T, Fs, F;
  long long ld_x;
  int M, act;
  int n_out;    // rows of W2 / b2 that the kernel averages itself (1: W2 / b2 are one row, folded or as given)
  float inv_out;
  int n_layers;
  int groups;   // token groups of a layer
  int splits;   // workgroups that share the hidden units of one token group; above 1 they write their activations
  float* acts;  // [layer][M][ld_acts] activations of the hidden units, added up by score_sum_kernel
  long long ld_acts;
  float* w2bar;  // [layer][M] averaged second layer, written by the first token group's workgroups (n_out > 1)
  SelectJob ride;
  ScoreLayer layer[kScoreBatchMax];
};

// The layer that a workgroup works on.  Arguments are read from memory where they are used, and a launch starts with as many
// round trips as the code in front of its first load has steps (six were 1 us of 13.5: 4680 tokens, 1536 features, 256
// units).  So everything that one layer needs is asked for at once, and only further layers go through the table.
__device__ __forceinline__ ScoreLayer layer_args(const ScoreArgs& A, int li) {
  ScoreLayer L = A.layer[0];
  asm volatile("" ::"s"(A.T), "s"(A.Fs), "s"(A.F), "s"(A.ld_x), "s"(A.M), "s"(A.act), "s"(A.n_out), "s"(A.inv_out), "s"(L.x[0]),
               "s"(L.x[1]), "s"(L.x[2]), "s"(L.W1), "s"(L.b1), "s"(L.W2), "s"(L.b2), "s"(L.out), "s"(A.n_layers), "s"(A.groups),
               "s"(A.splits));
  if (li > 0) L = A.layer[li];
  return L;
}

// averaged second layer of 4 hidden units from m on, in the order of fold_w2_kernel
__device__ __forceinline__ float4 averaged_w2(const float* __restrict__ W2, int M, int n_out, float inv, int m) {
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
  for (int o = 0; o < n_out; ++o) {
    const float4 w = *reinterpret_cast<const float4*>(W2 + (long long)o * M + m);
    s.x += w.x; s.y += w.y; s.z += w.z; s.w += w.w;
  }
  return make_float4(s.x * inv, s.y * inv, s.z * inv, s.w * inv);
}
__device__ __forceinline__ float folded_b2(const float* __restrict__ b2, int n_out, float inv) {
  if (b2 == nullptr) return 0.f;
  float s = 0.f;
#pragma unroll 4
  for (int o = 0; o < n_out; ++o) s += b2[o];
  return s * inv;
}

// Second layer of a token whose hidden units were shared by several workgroups.  One wave per (unit quarter, half) and 32
// tokens: a lane adds up the units that it would have held at the end of the passes of the unsplit kernel, in the same
// order, and the lane halves and the eight waves are added in the same order too.
__global__ __launch_bounds__(512) void score_sum_kernel(ScoreArgs a) {
  __shared__ float red[8 * 32];
  const ScoreLayer L = layer_args(a, blockIdx.y);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 5, c = lane & 31;
  const int t = blockIdx.x * 32 + c;
  const int m_wave = 64 * (wave & 3) + 32 * (wave >> 2) + 4 * g;
  const float* acts = a.acts + (long long)blockIdx.y * a.M * a.ld_acts + t;  // (ld_acts covers the last 32 tokens)
  const float* w2 = a.n_out == 1 ? L.W2 : a.w2bar + (long long)blockIdx.y * a.M;
  float partial = 0.f;
  for (int mp = m_wave; mp < a.M; mp += 256) {
    float v[16];
    float4 w[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      w[q] = *reinterpret_cast<const float4*>(w2 + mp + 8 * q);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[4 * q + e] = acts[(mp + 8 * q + e) * a.ld_acts];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      partial = fmaf(w[q].x, v[4 * q], partial);
      partial = fmaf(w[q].y, v[4 * q + 1], partial);
      partial = fmaf(w[q].z, v[4 * q + 2], partial);
      partial = fmaf(w[q].w, v[4 * q + 3], partial);
    }
  }
  partial += __shfl_xor(partial, 32);
  if (g == 0) red[wave * 32 + c] = partial;
  __syncthreads();
  if (threadIdx.x < 32 && t < a.T) {
    float v = folded_b2(L.b2, a.n_out, a.inv_out);
#pragma unroll
    for (int w = 0; w < 8; ++w) v += red[w * 32 + c];
    L.out[t] = v;
  }
}

// ---------------------------------------------------------------------------------- generic path
template <bool BF16>
__device__ __forceinline__ float load_elem(const void* p, long long i) {
  if (BF16) return bf16_bits_to_f32(static_cast<const unsigned short*>(p)[i]);
  return static_cast<const float*>(p)[i];
}

// 256 threads = 16 tokens x 16 hidden-unit lanes.
template <bool BF16>
__global__ __launch_bounds__(256) void score_generic_kernel(const void* x0, const void* x1, const void* x2, int n_seg,
                                                            int T, int Fs, long long ld_x, const void* W1,
                                                            const float* b1, const float* w2bar, const float* b2bar,
                                                            int M, int act, float* out) {
  const int t = blockIdx.x * 16 + (threadIdx.x >> 4);
  const int ml = threadIdx.x & 15;
  const int tt = t < T ? t : T - 1;
  const long long F = (long long)n_seg * Fs;
  float partial = 0.f;
  for (int m = ml; m < M; m += 16) {
    float h = b1 ? b1[m] : 0.f;
    for (int s = 0; s < n_seg; ++s) {
      const void* xs = s == 0 ? x0 : (s == 1 ? x1 : x2);
      const long long xo = (long long)tt * ld_x;
      const long long wo = (long long)m * F + (long long)s * Fs;
      float h0 = 0.f, h1 = 0.f, h2 = 0.f, h3 = 0.f;
      int f = 0;
      for (; f + 3 < Fs; f += 4) {
        h0 = fmaf(load_elem<BF16>(W1, wo + f), load_elem<BF16>(xs, xo + f), h0);
        h1 = fmaf(load_elem<BF16>(W1, wo + f + 1), load_elem<BF16>(xs, xo + f + 1), h1);
        h2 = fmaf(load_elem<BF16>(W1, wo + f + 2), load_elem<BF16>(xs, xo + f + 2), h2);
        h3 = fmaf(load_elem<BF16>(W1, wo + f + 3), load_elem<BF16>(xs, xo + f + 3), h3);
      }
      for (; f < Fs; ++f) h0 = fmaf(load_elem<BF16>(W1, wo + f), load_elem<BF16>(xs, xo + f), h0);
      h += (h0 + h1) + (h2 + h3);
    }
    partial = fmaf(w2bar[m], act_accurate(h, act), partial);
  }
  partial += __shfl_xor(partial, 8);
  partial += __shfl_xor(partial, 4);
  partial += __shfl_xor(partial, 2);
  partial += __shfl_xor(partial, 1);
  if (ml == 0 && t < T) out[t] = partial + (b2bar ? *b2bar : 0.f);
}

// The same for fp32 inputs whose rows are whole 16-byte chunks, with the same operations in the same order (a selection may
// follow from these scores, so two scores that are close must not change places): the features of 16 tokens and the
// weights of 32 hidden units go through LDS in pieces of 128 features, the next piece in flight meanwhile, instead of being
// read element by element.  A step of a small model is a chain of latencies: 320 tokens, 128 features and 32 units take
// 6.3 us (12.3 element by element), 1800 tokens, 256 features and 64 units 14.3 (37).
constexpr int kSfPiece = 128;            // features per piece
constexpr int kSfRow = kSfPiece + 4;     // floats per LDS row: 16 consecutive rows start in distinct banks
constexpr int kSfUnits = 32;
__global__ __launch_bounds__(256) void score_f32_kernel(ScoreArgs A) {
  __shared__ __attribute__((aligned(16))) float ws[kSfUnits * kSfRow], xs[16 * kSfRow];
  const ScoreLayer& L = A.layer[blockIdx.y];
  const int tid = threadIdx.x, tl = tid >> 4, ml = tid & 15;
  const int t0 = blockIdx.x * 16, t = t0 + tl;
  const int n_seg = A.F / A.Fs, pieces = (A.Fs + kSfPiece - 1) / kSfPiece;
  const int col = (tid & 31) * 4, row = tid >> 5;  // this thread's 16 bytes of 8 rows at a time
  float4 wr[kSfUnits / 8], xr[2];
  auto fetch = [&](int m0, int i) {  // piece i of the units m0 ..; columns past the segment's end are not read
    const int seg = i / pieces, f = (i - seg * pieces) * kSfPiece + col;
    if (f >= A.Fs) return;
    const float* xp = static_cast<const float*>(seg == 0 ? L.x[0] : (seg == 1 ? L.x[1] : L.x[2]));
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int tt = t0 + row + 8 * j;
      xr[j] = *reinterpret_cast<const float4*>(xp + (long long)(tt < A.T ? tt : A.T - 1) * A.ld_x + f);
    }
#pragma unroll
    for (int j = 0; j < kSfUnits / 8; ++j) {
      const int m = m0 + row + 8 * j;
      wr[j] = *reinterpret_cast<const float4*>(static_cast<const float*>(L.W1) + (long long)(m < A.M ? m : A.M - 1) * A.F +
                                               (long long)seg * A.Fs + f);
    }
  };
#pragma unroll
  for (int j = 0; j < kSfUnits / 8; ++j) wr[j] = make_float4(0.f, 0.f, 0.f, 0.f);
  xr[0] = xr[1] = wr[0];
  float partial = 0.f;
  fetch(0, 0);
  const float b2 = folded_b2(L.b2, A.n_out, A.inv_out);
  for (int m0 = 0; m0 < A.M; m0 += kSfUnits) {
    float h[2], w2[2], acc[2][4];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int m = m0 + ml + 16 * u;
      h[u] = L.b1 != nullptr && m < A.M ? L.b1[m] : 0.f;
      acc[u][0] = acc[u][1] = acc[u][2] = acc[u][3] = 0.f;
      // (asked for here: behind the products it would be one more wait for memory)
      w2[u] = 0.f;
      if (m < A.M) {
        if (A.n_out == 1) {
          w2[u] = L.W2[m];
        } else {
#pragma unroll 4
          for (int o = 0; o < A.n_out; ++o) w2[u] += L.W2[(long long)o * A.M + m];
          w2[u] *= A.inv_out;
        }
      }
    }
    for (int i = 0; i < n_seg * pieces; ++i) {
      __syncthreads();  // the previous piece has been used
#pragma unroll
      for (int j = 0; j < kSfUnits / 8; ++j) *reinterpret_cast<float4*>(ws + (row + 8 * j) * kSfRow + col) = wr[j];
#pragma unroll
      for (int j = 0; j < 2; ++j) *reinterpret_cast<float4*>(xs + (row + 8 * j) * kSfRow + col) = xr[j];
      __syncthreads();
      if (i + 1 < n_seg * pieces) fetch(m0, i + 1);
      else if (m0 + kSfUnits < A.M) fetch(m0 + kSfUnits, 0);
      const int in_seg = i % pieces, width = A.Fs - in_seg * kSfPiece < kSfPiece ? A.Fs - in_seg * kSfPiece : kSfPiece;
#pragma unroll 8
      for (int f = 0; f < width; f += 4) {
        const float4 x = *reinterpret_cast<const float4*>(xs + tl * kSfRow + f);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const float4 w = *reinterpret_cast<const float4*>(ws + (ml + 16 * u) * kSfRow + f);
          acc[u][0] = fmaf(w.x, x.x, acc[u][0]);
          acc[u][1] = fmaf(w.y, x.y, acc[u][1]);
          acc[u][2] = fmaf(w.z, x.z, acc[u][2]);
          acc[u][3] = fmaf(w.w, x.w, acc[u][3]);
        }
      }
      if (in_seg == pieces - 1) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          h[u] += (acc[u][0] + acc[u][1]) + (acc[u][2] + acc[u][3]);
          acc[u][0] = acc[u][1] = acc[u][2] = acc[u][3] = 0.f;
        }
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int m = m0 + ml + 16 * u;
      if (m < A.M) partial = fmaf(w2[u], act_accurate(h[u], A.act), partial);
    }
  }
  partial += __shfl_xor(partial, 8);
  partial += __shfl_xor(partial, 4);
  partial += __shfl_xor(partial, 2);
  partial += __shfl_xor(partial, 1);
  if (ml == 0 && t < A.T) L.out[t] = partial + b2;
}

// ---------------------------------------------------------------------------------- MFMA path
constexpr int kScThreads = 256;
constexpr int kScTokPerWave = 32;
constexpr int kScTokPerWg = 128;
constexpr int kScSlab = 64;                 // features per LDS slab
constexpr int kScRowBytes = kScSlab * 2 + 16;  // 144 B: padded so that 16 consecutive rows hit distinct banks
// two slabs of W1, then the second layer's weights and the biases of a pass's units
constexpr int sc_lds_bytes(int mb) { return 2 * mb * 32 * kScRowBytes + 2 * mb * 32 * 4; }

__device__ __forceinline__ float fast_silu(float h) {
  // h * sigmoid(h), sigmoid via exp2 and a reciprocal
  const float e = __builtin_amdgcn_exp2f(-1.44269504088896340736f * h);
  return h * __builtin_amdgcn_rcpf(1.0f + e);
}

// MB = 32-row hidden blocks per pass over X (MB*32 hidden units are accumulated at once); one layer per blockIdx.y.
template <int MB>
__global__ __launch_bounds__(kScThreads, 2) void score_mfma_kernel(ScoreArgs A) {
  const ScoreLayer L = layer_args(A, blockIdx.y);
  const unsigned short* const x0 = static_cast<const unsigned short*>(L.x[0]);
  const unsigned short* const x1 = static_cast<const unsigned short*>(L.x[1]);
  const unsigned short* const x2 = static_cast<const unsigned short*>(L.x[2]);
  const unsigned short* const W1 = static_cast<const unsigned short*>(L.W1);
  const float* const b1 = L.b1;
  const int T = A.T, Fs = A.Fs, F = A.F, M = A.M, act = A.act;
  const long long ld_x = A.ld_x;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 5, c = lane & 31;
  const int tok = blockIdx.x * kScTokPerWg + wave * kScTokPerWave + c;
  const int tokc = tok < T ? tok : T - 1;
  const int n_slabs = F / kScSlab;
  const int slabs_per_seg = Fs / kScSlab;
  // this thread's part of a W1 slab: rows (i*32 + tid/8), 16-byte chunk tid%8
  const int w_row = tid >> 3, w_chunk = tid & 7;

  float b2 = 0.f, partial = 0.f;
  constexpr int kScMBlocks = MB;
  constexpr int kScBufBytes = MB * 32 * kScRowBytes;
  float* const w2s = reinterpret_cast<float*>(lds + 2 * kScBufBytes);
#pragma unroll 1
  for (int mp = 0; mp < M; mp += kScMBlocks * 32) {
    f32x16 acc[kScMBlocks];
#pragma unroll
    for (int b = 0; b < kScMBlocks; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[b][r] = 0.f;

    u32x4 wreg[kScMBlocks];
    bf16x8 xreg[4];
    const unsigned short* wbase = W1 + (long long)(mp + w_row) * F + w_chunk * 8;
#define PAFU_LOAD_SLAB(S)                                                                          \
  do {                                                                                             \
    const unsigned short* wsrc = wbase + (long long)(S) * kScSlab;                                 \
    _Pragma("unroll") for (int i = 0; i < kScMBlocks; ++i)                                         \
        wreg[i] = *reinterpret_cast<const u32x4*>(wsrc + (long long)i * 32 * F);                   \
    const int seg = (S) / slabs_per_seg;                                                           \
    const int fo = ((S) - seg * slabs_per_seg) * kScSlab;                                          \
    const unsigned short* xs = seg == 0 ? x0 : (seg == 1 ? x1 : x2);                               \
    const unsigned short* xsrc = xs + (long long)tokc * ld_x + fo + 8 * g;                         \
    _Pragma("unroll") for (int kk = 0; kk < 4; ++kk)                                               \
        xreg[kk] = *reinterpret_cast<const bf16x8*>(xsrc + kk * 16);                               \
  } while (0)
#define PAFU_STORE_SLAB(BUF)                                                                       \
  do {                                                                                             \
    unsigned char* dst = lds + (BUF) * kScBufBytes + w_row * kScRowBytes + w_chunk * 16;           \
    _Pragma("unroll") for (int i = 0; i < kScMBlocks; ++i)                                         \
        *reinterpret_cast<u32x4*>(dst + i * 32 * kScRowBytes) = wreg[i];                           \
  } while (0)

    PAFU_LOAD_SLAB(0);
    // The second layer's weights and the biases of this pass, once per workgroup and while the first slab is on its way.
    // (Read by every lane where they are used, they were 16 rounds of loads, each n_out long: 6 layers of 7210 tokens, 512
    // features, 128 units and 4 output rows 23.7 us, now 16.3.)
    float4 second = make_float4(0.f, 0.f, 0.f, 0.f);
    if (mp == 0) b2 = folded_b2(L.b2, A.n_out, A.inv_out);
    const int unit = 4 * (tid & 127);
    if (unit < kScMBlocks * 32) {
      if (tid < 128) second = A.n_out == 1 ? *reinterpret_cast<const float4*>(L.W2 + mp + unit)
                                           : averaged_w2(L.W2, M, A.n_out, A.inv_out, mp + unit);
      else if (b1 != nullptr) second = *reinterpret_cast<const float4*>(b1 + mp + unit);
    }
    __syncthreads();  // every wave is done with the LDS contents of the previous pass
    if (unit < kScMBlocks * 32) *reinterpret_cast<float4*>(w2s + (tid < 128 ? 0 : kScMBlocks * 32) + unit) = second;
    PAFU_STORE_SLAB(0);
    __syncthreads();
#pragma unroll 1
    for (int s = 0; s < n_slabs; ++s) {
      bf16x8 xcur[4];
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) xcur[kk] = xreg[kk];
      if (s + 1 < n_slabs) PAFU_LOAD_SLAB(s + 1);
      const unsigned char* buf = lds + (s & 1) * kScBufBytes + c * kScRowBytes + g * 16;
      // Fragments are read two matrix instructions ahead.  (With the order left to the compiler, which keeps registers free for a
      // third wave per SIMD, each one waited for its own: 4680 tokens of 1536 features, 128 units 24.5 us, now 20.8.)
      bf16x8 a[2];
      auto frag = [&](int i) {  // fragment i of the slab: k-step i / MB, block i % MB
        return *reinterpret_cast<const bf16x8*>(buf + (i % kScMBlocks) * 32 * kScRowBytes + (i / kScMBlocks) * 32);
      };
      a[0] = frag(0);
      a[1] = frag(1);
#pragma unroll
      for (int i = 0; i < 4 * kScMBlocks; ++i) {
        const int b = i % kScMBlocks, kk = i / kScMBlocks;
        acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i & 1], xcur[kk], acc[b], 0, 0, 0);
        if (i + 2 < 4 * kScMBlocks) a[i & 1] = frag(i + 2);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (s + 1 < n_slabs) PAFU_STORE_SLAB((s + 1) & 1);
      __syncthreads();
    }
    // activation and second layer for this pass's hidden units; lane holds token c, units
    // mp + 32 b + 8 (r/4) + 4 g + (r%4)
    // (One branch for all of it: with one per four units each waited for its own LDS reads, 37440 tokens of 1536 features, 64
    // units 31.5 us, now 29.2.)
    auto second_layer = [&](auto activation) {
#pragma unroll
      for (int b = 0; b < kScMBlocks; ++b) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int m0 = 32 * b + 8 * q + 4 * g;
          const float4 w = *reinterpret_cast<const float4*>(w2s + m0);
          const float4 bb = *reinterpret_cast<const float4*>(w2s + kScMBlocks * 32 + m0);
          partial = fmaf(w.x, activation(acc[b][4 * q + 0] + bb.x), partial);
          partial = fmaf(w.y, activation(acc[b][4 * q + 1] + bb.y), partial);
          partial = fmaf(w.z, activation(acc[b][4 * q + 2] + bb.z), partial);
          partial = fmaf(w.w, activation(acc[b][4 * q + 3] + bb.w), partial);
          asm volatile("" : "+v"(partial));  // (or all activations are kept for later: spills)
        }
      }
    };
    if (act == PAFU_ACT_SILU) second_layer([](float h) { return fast_silu(h); });
    else second_layer([&](float h) { return act_accurate(h, act); });
  }
#undef PAFU_LOAD_SLAB
#undef PAFU_STORE_SLAB
  partial += __shfl_xor(partial, 32);
  if (g == 0 && tok < T) L.out[tok] = partial + b2;
}

// ---------------------------------------------------------------------------------- streaming MFMA path
// For M % 256 == 0 and Fs % 64 == 0.  With a 256-wide hidden layer the head sits near the ridge of the roofline
// (about 256 flop per byte of features), and every CU has to pull all of W1 through its L1 once per token group, so
// the kernel must keep the matrix cores and the memory pipe busy at the same time: an even spread of MFMA work over
// the 1024 SIMDs, few LDS bytes per MFMA, and many bytes in flight without spending registers on them.
//  - A workgroup owns TT 32-token tiles (TT picked at launch so that the grid needs as few rounds over the 256 CUs
//    as possible) and one pass of 128 NB hidden units at a time.  Its 8 waves split the hidden units four
//    ways and the reduction axis two ways: wave (hq, kh) accumulates NB 32-unit blocks for all TT
//    tiles over half of the k-steps of every slab, so one W1 fragment feeds TT MFMAs and one feature fragment NB.
//    The two reduction halves sit on the same SIMD (waves w and w + 4) and are added through LDS at the end of a pass.
//  - W1 and the features stream global -> LDS with global_load_lds through a ring of slabs (no staging registers,
//    all but one slab of the ring in flight), rows XOR-swizzled in 16-byte chunks for conflict-free b128 reads.
//  - A CU takes in about 45 bytes per clock, and a slab's W1 part (32 KB at NB = 2) costs more than its TT feature tiles.
//    A hidden layer may therefore be shared by `splits` workgroups (SPLIT), which makes room for a larger TT: 4680
//    tokens of 4608 features and 1024 units took 128 us with one token tile per workgroup and all four passes in it, and
//    take 62 us with five tiles and an eighth of the units (10800 tokens, 5120 features, 512 units: 123 -> 80 us).
//    What the workgroups leave in scratch are activations, not partial sums: one more launch (6.5 us in both) then takes them through
//    the second layer in the order of the unsplit kernel, so that a score's bits do not depend on the launch.
//  - Layers of one geometry share a launch: the token groups of one (57 at 7210 tokens) leave most of the chip idle
//    (six of 128 units: 6 x 12.9 us one by one, 24 us together, in the kernel above).
constexpr int kS3Slab = 64;                      // features per slab (full 128-byte lines per row)
constexpr int kS3RowB = kS3Slab * 2;             // bytes per slab row
constexpr int kS3Chunks = kS3RowB / 16;          // 16-byte chunks per row
constexpr int kS3RowsPerLoad = 1024 / kS3RowB;   // rows covered by one wave-wide 16-byte-per-lane load
constexpr int kS3Stages = 3;                     // ring depth: 3 x (32 KB + 4 TT KB) <= 156 KB
constexpr int s3_w_bytes(int NB) { return 128 * NB * kS3RowB; }  // W1 part of a stage (128 NB hidden units)
constexpr int kS3MaxTT = 5;
constexpr int kS3RedBytes = 65536;               // two 32 KB regions for the end-of-pass reduction
constexpr int s3_stage_bytes(int TT, int NB) { return s3_w_bytes(NB) + 32 * TT * kS3RowB; }
constexpr int s3_lds_bytes(int TT, int NB) {
  return kS3Stages * s3_stage_bytes(TT, NB) > kS3RedBytes ? kS3Stages * s3_stage_bytes(TT, NB) : kS3RedBytes;
}
static_assert(s3_lds_bytes(1, 2) >= kS3RedBytes + 256 * 4, "room for a pass's averaged second layer behind the two regions");
// chunk q of row r lives in slot q ^ swz(r): 16 consecutive rows of one chunk then cover all 64 banks
__device__ __forceinline__ int s3_swz(int row) {
  return kS3RowB == 64 ? (row >> 2) & 3 : (row >> 1) & 7;
}

// 64 x 16 bytes global -> LDS: lane l's bytes at (uniform base + its byte offset) land at lds_addr + 16 l
__device__ __forceinline__ void s3_dma(const void* base_uniform, unsigned byte_off, unsigned lds_addr_uniform) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :
               : "s"(lds_addr_uniform), "v"(byte_off), "s"(base_uniform)
               : "memory");
}
template <int N>
__device__ __forceinline__ void s3_wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// SELW > 0: workgroup 0 of the launch does not score but runs a top-k selection (SELW key words per thread, 512
// threads) on a list that does not depend on this launch's scores: the stored score list of a rollout step.  A
// selection keeps one CU busy for about as long as the scoring of a chunk takes the others, so carried along it
// costs nothing, where a launch of its own would leave the rest of the chip idle meanwhile.
// OWN_ROWS: the kernel averages the rows of the second layer (n_out > 1).  A variant of its own, because the choice at run
// time kept the one row's loads from overlapping the activations (1 us of 13.5).
template <int TT, int NB, bool SPLIT, bool OWN_ROWS, int SELW>
__global__ __launch_bounds__(512, 1) void score_stream_kernel(ScoreArgs A) {
  static_assert(SPLIT || NB == 2, "the order of a score's sums is that of passes of 256 units");
  int id = blockIdx.x;
  if constexpr (SELW > 0) {
    if (id == 0) {
      select_bitslice_body<SELW, 512>(A.ride);
      return;
    }
    --id;
  }
  // Workgroups are handed to the 8 XCDs in turn: the splits of a token group are 8 apart, so that one L2 serves its
  // features to all of them.
  // (no divisions in front of the first load where one layer and no splits make them needless)
  ScoreLayer L = layer_args(A, 0);
  const int per_layer = A.groups * A.splits;
  int li = 0;
  if (A.n_layers > 1) li = id / per_layer;
  int group = id - li * per_layer, split = 0;
  if constexpr (SPLIT) {
    const int w = id - li * per_layer, band = 8 * A.splits, full = A.groups / 8 * 8;
    if (w < full * A.splits) {
      const int r = w % band;
      group = w / band * 8 + r % 8;
      split = r / 8;
    } else {
      const int r = w - full * A.splits, left = A.groups - full;
      group = full + r % left;
      split = r / left;
    }
  }
  if (A.n_layers > 1) L = A.layer[li];
  const unsigned short* const x0 = static_cast<const unsigned short*>(L.x[0]);
  const unsigned short* const x1 = static_cast<const unsigned short*>(L.x[1]);
  const unsigned short* const x2 = static_cast<const unsigned short*>(L.x[2]);
  const unsigned short* const W1 = static_cast<const unsigned short*>(L.W1);
  const float* const b1 = L.b1;
  const int T = A.T, Fs = A.Fs, F = A.F, act = A.act;
  const long long ld_x = A.ld_x;
  constexpr int MP = 128 * NB;                         // hidden units per pass
  constexpr int kWBytes = s3_w_bytes(NB);
  constexpr int kStageB = s3_stage_bytes(TT, NB);
  constexpr int WU = MP / kS3RowsPerLoad;              // wave-wide loads that fill the W1 part of a stage
  constexpr int XU = 32 * TT / kS3RowsPerLoad;         // ... and the feature part
  constexpr int LW = WU / 8;                           // W1 loads per wave per slab
  constexpr int LX = (XU + 7) / 8;                     // feature loads per wave per slab
  constexpr int LPW = LW + LX;
  constexpr int KS = kS3Slab / 32;                     // k-steps (16 features) per wave per slab
  static_assert(KS % 2 == 0, "the two fragment sets alternate per k-step and must line up across slabs");
  typedef __attribute__((address_space(3))) unsigned char lds_byte;
  typedef __attribute__((address_space(3))) bf16x8 lds_frag;
  typedef float f32x4_t __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) f32x4_t lds_f4;
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds_raw[];
  lds_byte* const ring = (lds_byte*)lds_raw;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // said to be uniform: LDS addresses of the loads stay scalar
  const int hq = wave & 3, kh = wave >> 2;
  const int g = lane >> 5, c = lane & 31;
  const int tok_base = group * (32 * TT);
  const int n_slabs = F / kS3Slab;
  const int slabs_per_seg = Fs / kS3Slab;

  // ---- loads.  One wave-wide load covers kS3RowsPerLoad slab rows: lane -> (row, LDS slot); the slot receives chunk
  // slot ^ swz(row) of the row.  Addresses are a uniform base plus a 32-bit per-lane byte offset.  Surplus feature
  // loads repeat a unit (same bytes, same place) so that every wave issues the same number of loads.
  const int d_row = lane / kS3Chunks, d_slot = lane % kS3Chunks;
  unsigned w_off[LW], x_off[LX];
#pragma unroll
  for (int j = 0; j < LW; ++j) {
    const int row = (wave + 8 * j) * kS3RowsPerLoad + d_row;
    w_off[j] = (unsigned)((row * F + (d_slot ^ s3_swz(row)) * 8) * 2);
  }
#pragma unroll
  for (int j = 0; j < LX; ++j) {
    const int row = ((wave + 8 * j) % XU) * kS3RowsPerLoad + d_row;
    const int rel = tok_base + row < T ? row : T - 1 - tok_base;
    x_off[j] = (unsigned)(rel * ld_x * 2) + (d_slot ^ s3_swz(row)) * 16;
  }
  const long long x_wg_off = (long long)tok_base * ld_x;
  // ---- fragment reads inside a stage: k-step ks = KS kh + j of the slab, lane half g -> chunk 2 ks + g.
  // swz(row) only depends on c for the rows a lane reads (row = 32-row block + c).
  int rd[KS];
#pragma unroll
  for (int j = 0; j < KS; ++j) rd[j] = c * kS3RowB + (((2 * (KS * kh + j) + g) ^ s3_swz(c)) << 4);

  float partial[TT];
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) partial[tt] = 0.f;

  const int m_share = SPLIT ? A.M / A.splits : A.M;
#pragma unroll 1
  for (int mp = split * m_share; mp < (split + 1) * m_share; mp += MP) {
    f32x16 acc[TT][NB];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[tt][b][r] = 0.f;
    const unsigned short* const w_pass = W1 + (long long)mp * F;  // uniform

    // Slabs go to the stages of the ring in turn; their addresses move on from one to the next.  (Slabs past the end re-read the
    // last one; they are never consumed.  Worked out from the slab's number, with a division for its segment and one for the
    // stage, and with the output rows below averaged one load after the other, 4680 tokens of 4608 features, 1024 units and
    // 12 rows took 55.7 us, now 48.6; 21840 tokens of 1536 features and 1024 units 83.2, now 79.3.)
    const unsigned short *w_next = w_pass, *x_next = x0 + x_wg_off;
    int to_come = n_slabs, seg_next = 0, seg_left = slabs_per_seg, stage_next = 0;
    auto issue_slab = [&] {
      lds_byte* const st = ring + stage_next;
#pragma unroll
      for (int j = 0; j < LW; ++j) s3_dma(w_next, w_off[j], (unsigned)(uintptr_t)(st + (wave + 8 * j) * 1024));
#pragma unroll
      for (int j = 0; j < LX; ++j)
        s3_dma(x_next, x_off[j], (unsigned)(uintptr_t)(st + kWBytes + ((wave + 8 * j) % XU) * 1024));
      stage_next = stage_next == (kS3Stages - 1) * kStageB ? 0 : stage_next + kStageB;
      if (--to_come > 0) {
        w_next += kS3Slab;
        x_next += kS3Slab;
        if (--seg_left == 0) {
          seg_left = slabs_per_seg;
          x_next = (++seg_next == 1 ? x1 : x2) + x_wg_off;
        }
      }
    };

    // Fragments of k-step j of a slab: two W1 blocks and TT feature tiles, into fragment set B (0 or 1).
#define PAFU_S3_READ(B, ST, J)                                                                                  \
  do {                                                                                                          \
    _Pragma("unroll") for (int nb = 0; nb < NB; ++nb)                                                           \
        fw[B][nb] = *(const lds_frag*)((ST) + (hq * 32 * NB + 32 * nb) * kS3RowB + rd[J]);                      \
    _Pragma("unroll") for (int tt = 0; tt < TT; ++tt)                                                           \
        fx[B][tt] = *(const lds_frag*)((ST) + kWBytes + tt * 32 * kS3RowB + rd[J]);                           \
  } while (0)
#define PAFU_S3_MMA(B)                                                                                          \
  do {                                                                                                          \
    _Pragma("unroll") for (int tt = 0; tt < TT; ++tt)                                                           \
        _Pragma("unroll") for (int nb = 0; nb < NB; ++nb)                                                       \
            acc[tt][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[B][nb], fx[B][tt], acc[tt][nb], 0, 0, 0);  \
  } while (0)

    // Software pipeline.  The fragments of the next k-step are read while the matrix instructions of the current one
    // run, also across slabs: the barrier sits before the LAST k-step of slab s, where every wave has its last
    // fragments of slab s in registers (so the slab's stage can be refilled) and where slab s+1 must have landed (so
    // its first fragments can be fetched under the last k-step of slab s).  Ring: stage of slab s being refilled
    // with slab s+3, slab s+1 ready, slab s+2 in flight.
    bf16x8 fw[2][NB], fx[2][TT];
    const bool kh_first = kh == 0;
    __syncthreads();  // every wave is done with the LDS contents of the previous pass
#pragma unroll
    for (int s = 0; s < kS3Stages; ++s) issue_slab();
    s3_wait_vmcnt<(kS3Stages - 1) * LPW>();
    __builtin_amdgcn_s_barrier();  // slab 0 visible to all
    PAFU_S3_READ(0, ring, 0);
#pragma unroll 1
    for (int s = 0, stage = 0; s < n_slabs; ++s) {
      const lds_byte* st = ring + stage;
      const lds_byte* st_next = ring + (stage == (kS3Stages - 1) * kStageB ? 0 : stage + kStageB);
#pragma unroll
      for (int j = 0; j < KS; ++j) {
        if (j + 1 < KS) {
          PAFU_S3_READ((j + 1) & 1, st, j + 1);
        } else {
          // own fragment reads of slab s complete (they must be before the stage is handed back), then the loads
          // of slab s+1 (issued two barriers ago; only the slab after it may still be in flight)
          __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0), other counters left alone
          s3_wait_vmcnt<(kS3Stages - 2) * LPW>();
          __builtin_amdgcn_s_barrier();
          // refill the stage of slab s.  A wave cannot issue anything else while its loads queue up behind a busy
          // memory pipe, so the two waves of a SIMD (kh = 0, 1) take turns: one issues its loads before this
          // k-step's matrix instructions, the other after them.
          if (kh_first) issue_slab();
          PAFU_S3_READ((j + 1) & 1, st_next, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        PAFU_S3_MMA(j & 1);
        __builtin_amdgcn_sched_barrier(0);
        if (j + 1 == KS && !kh_first) issue_slab();
      }
      stage = stage == (kS3Stages - 1) * kStageB ? 0 : stage + kStageB;
    }
#undef PAFU_S3_READ
#undef PAFU_S3_MMA
    // ---- add the two halves of the reduction axis through LDS, one token tile at a time, alternating between two
    // 32 KB regions so that one barrier per tile is enough.  The two waves (hq, 0) and (hq, 1) swap half of their units
    // (a 32-unit block, or 16 units of the only one): wave kh ends up with the complete sums of the kh-th half and applies
    // bias, activation and second layer to it, so that both waves of a SIMD share that work.
    s3_wait_vmcnt<0>();
    __syncthreads();  // all loads have landed and all fragment reads are done: the ring can be reused
    constexpr int KQ = 2 * NB;  // quadruples of units that a wave keeps (and sends)
    const int m_wave = mp + 32 * NB * hq + 16 * NB * kh + 4 * g;  // quadruple q of the lane: units m_wave + 8 q ..
    // the pass's averaged second layer, behind the two regions (the first barrier below shows it to all waves); every wave
    // averaging what it needs took 2 us more (256 units, 12 rows)
    typedef __attribute__((address_space(3))) float lds_float;
    if (OWN_ROWS && tid < MP && (!SPLIT || (A.n_out > 1 && group == 0))) {
      float w = 0.f;
#pragma unroll 4
      for (int o = 0; o < A.n_out; ++o) w += L.W2[(long long)o * A.M + mp + tid];
      w *= A.inv_out;
      if (SPLIT) A.w2bar[(long long)li * A.M + mp + tid] = w;
      else ((lds_float*)(ring + kS3RedBytes))[tid] = w;
    }
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
      lds_f4* reg = (lds_f4*)(ring + (tt & 1) * 32768) + (hq * 2 + kh) * KQ * 64 + lane;       // what this wave sends
      const lds_f4* got = (const lds_f4*)(ring + (tt & 1) * 32768) + (hq * 2 + (kh ^ 1)) * KQ * 64 + lane;
      // element e of quadruple q of half HALF (NB = 2: block HALF; NB = 1: the upper or lower rows of the block)
#define PAFU_S3_HALF(HALF, Q, E) (NB == 2 ? acc[tt][NB - 1 ? (HALF) : 0][4 * (Q) + (E)] : acc[tt][0][4 * (2 * (HALF) + (Q)) % 16 + (E)])
#pragma unroll
      for (int q = 0; q < KQ; ++q) {
        if (kh == 0) reg[q * 64] = f32x4_t{PAFU_S3_HALF(1, q, 0), PAFU_S3_HALF(1, q, 1), PAFU_S3_HALF(1, q, 2), PAFU_S3_HALF(1, q, 3)};
        else reg[q * 64] = f32x4_t{PAFU_S3_HALF(0, q, 0), PAFU_S3_HALF(0, q, 1), PAFU_S3_HALF(0, q, 2), PAFU_S3_HALF(0, q, 3)};
      }
      __syncthreads();
      // the lane holds token c of tile tt and hidden units m_wave + 8 q + e
      float hsum[4 * KQ];
#pragma unroll
      for (int q = 0; q < KQ; ++q) {
        const f32x4_t o = got[q * 64];
        float4 bb = make_float4(0.f, 0.f, 0.f, 0.f);
        if (b1 != nullptr) bb = *reinterpret_cast<const float4*>(b1 + m_wave + 8 * q);
        const float ov[4] = {o.x, o.y, o.z, o.w}, bv[4] = {bb.x, bb.y, bb.z, bb.w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
          hsum[4 * q + e] = (kh == 0 ? PAFU_S3_HALF(0, q, e) : PAFU_S3_HALF(1, q, e)) + ov[e] + bv[e];
      }
#undef PAFU_S3_HALF
      if (act == PAFU_ACT_SILU) {
#pragma unroll
        for (int i = 0; i < 4 * KQ; ++i) hsum[i] = fast_silu(hsum[i]);
      } else {
#pragma unroll
        for (int i = 0; i < 4 * KQ; ++i) hsum[i] = act_accurate(hsum[i], act);
      }
      if constexpr (SPLIT) {
        const int tok = tok_base + 32 * tt + c;
        float* const acts = A.acts + ((long long)li * A.M + m_wave) * A.ld_acts + tok;
        if (tok < T) {
#pragma unroll
          for (int i = 0; i < 4 * KQ; ++i) acts[(8 * (i >> 2) + (i & 3)) * A.ld_acts] = hsum[i];
        }
        continue;
      }
#pragma unroll
      for (int q = 0; q < KQ; ++q) {
        const f32x4_t w = OWN_ROWS ? *(const lds_f4*)(ring + kS3RedBytes + (m_wave - mp + 8 * q) * 4)
                                   : *reinterpret_cast<const f32x4_t*>(L.W2 + m_wave + 8 * q);
        partial[tt] = fmaf(w.x, hsum[4 * q], partial[tt]);
        partial[tt] = fmaf(w.y, hsum[4 * q + 1], partial[tt]);
        partial[tt] = fmaf(w.z, hsum[4 * q + 2], partial[tt]);
        partial[tt] = fmaf(w.w, hsum[4 * q + 3], partial[tt]);
      }
    }
  }
  if (SPLIT) return;
  // ---- add the two lane halves, then the eight waves (each holds the part of its 32-unit blocks)
  __syncthreads();
  float* red = reinterpret_cast<float*>(lds_raw);
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) {
    partial[tt] += __shfl_xor(partial[tt], 32);
    if (g == 0) red[wave * (32 * TT) + tt * 32 + c] = partial[tt];
  }
  __syncthreads();
  for (int i = tid; i < 32 * TT; i += 512) {
    const int tok = tok_base + i;
    if (tok < T) {
      float v = folded_b2(L.b2, A.n_out, A.inv_out);
#pragma unroll
      for (int w = 0; w < 8; ++w) v += red[w * (32 * TT) + i];
      L.out[tok] = v;
    }
  }
}

// Scratch of pafu_score_static: the output-averaged second layer (M weights + 1 bias) that pafu_score keeps in its
// caller-provided workspace.  One copy per GPU, held until the process ends; every call on a GPU shares it.
static __device__ __align__(256) float scratch[PAFU_SCORE_STATIC_MAX_M + 1];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
float* g_scratch_ptr[kMaxDevices] = {};  // device address of `scratch` on each GPU (the array's name is only a
                                         // host-side handle: kernels are given these addresses)

// Device address of `scratch` on the current GPU, looked up once per device.
int score_scratch(float** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return record_hip_error(e);
  if (dev < 0 || dev >= kMaxDevices) return PAFU_ERR_SHAPE;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return record_hip_error(e);
    if (ptr == nullptr) return record_hip_error(hipErrorInvalidSymbol);
    g_scratch_ptr[dev] = static_cast<float*>(ptr);
  }
  *out = g_scratch_ptr[dev];
  return PAFU_OK;
}

}  // namespace

int launch_score_static(hipStream_t st, const ScoreShape& s, const ScoreLayer& layer) {
  if (s.M > PAFU_SCORE_STATIC_MAX_M) return PAFU_ERR_WORKSPACE;
  float* ws = nullptr;
  const int rc = score_scratch(&ws);
  if (rc != PAFU_OK) return rc;
  return launch_score(st, s, &layer, 1, ws);
}

namespace {

// What one slab of 64 features takes a workgroup, in clocks: its matrix instructions or its fragment reads from LDS (128 TT
// and 64 (TT + 2) per 32 features and 256 units), or the copies into LDS (W1 and TT token tiles at 45 bytes per clock),
// whichever is longer; plus the barrier and the exposed first reads.
long long slab_cost(int tt, int nb) {
  const int mfma = 128 * tt * nb, lds = nb == 2 ? 128 * (tt + 2) : 128 * (tt + 1);
  const int copies = (16 * nb + 4 * tt) * 1024 / 45 - 100;
  const int most = mfma > lds ? mfma : lds;
  return (most > copies ? most : copies) + 100;
}

// How the streaming kernel cuts its work: tt 32-token tiles per workgroup, nb (units per pass / 128), and how many
// workgroups share the hidden units of a token group.
struct ScorePlan {
  int tt, nb, splits;
};
ScorePlan plan_score(int T, int F, int M, int n_layers, bool may_split) {
  ScorePlan best{1, 2, 1};
  long long best_cost = 1ll << 60;
  const long long cus = compute_units();
  const int tiles = (T + 31) / 32, slabs = F / kS3Slab;
  for (int nb = 1; nb <= 2; ++nb) {
    const int passes = M / (128 * nb);
    for (int splits = 1; splits <= passes && splits <= kScoreSplitMax; ++splits) {
      if (passes % splits != 0 || (splits == 1 ? nb == 1 : !may_split)) continue;
      for (int tt = 1; tt <= kS3MaxTT; ++tt) {
        const long long wgs = (long long)((tiles + tt - 1) / tt) * splits * n_layers;
        // (a pass ends with about 1500 + 500 tt clocks of sums and activations; the launch that takes shared units through
        // the second layer costs about 18000, the wait for it included: 60 tokens of 768 features and 512 units, 23700
        // clocks by this sum, lose 3 us when shared, 300 of 1536 features, 43300 clocks, gain 4)
        const long long cost = (wgs + cus - 1) / cus * (passes / splits) * (slabs * slab_cost(tt, nb) + 1500 + 500 * tt) +
                               (splits > 1 ? 18000 + (long long)T * M * n_layers / 1000 : 0);
        if (cost <= best_cost) { best_cost = cost; best = ScorePlan{tt, nb, splits}; }
      }
    }
  }
  return best;
}
// scratch of shared hidden units: the activations, rounded up to whole tiles of tokens, and the averaged second layers
long long split_ld(int T) { return ((long long)T + 31) / 32 * 32; }
size_t split_scratch_bytes(int T, int M, int n_layers) {
  return (size_t)n_layers * M * ((size_t)split_ld(T) + 1) * sizeof(float);
}

template <int TT, int NB, bool SPLIT, bool OWN_ROWS, int SELW>
int launch_stream(hipStream_t st, const ScoreArgs& a, int n_layers) {
  static LdsLimit lds_limit;
  int lds = s3_lds_bytes(TT, NB);
  if (SELW > 0 && lds < select_bitslice_lds_bytes(512)) lds = select_bitslice_lds_bytes(512);
  const int rc = set_lds_limit(lds_limit, score_stream_kernel<TT, NB, SPLIT, OWN_ROWS, SELW>, lds);
  if (rc != PAFU_OK) return rc;
  hipLaunchKernelGGL((score_stream_kernel<TT, NB, SPLIT, OWN_ROWS, SELW>),
                     dim3(a.groups * a.splits * n_layers + (SELW > 0 ? 1 : 0)), dim3(512), lds, st, a);
  if (SPLIT) hipLaunchKernelGGL(score_sum_kernel, dim3((a.T + 31) / 32, n_layers), dim3(512), 0, st, a);
  return check_launch();
}
template <int TT, int NB, bool SPLIT, bool OWN_ROWS>
int launch_stream_sel(hipStream_t st, const ScoreArgs& a, int n_layers, int selw) {
  if (selw == 2) return launch_stream<TT, NB, SPLIT, OWN_ROWS, 2>(st, a, n_layers);
  if (selw == 4) return launch_stream<TT, NB, SPLIT, OWN_ROWS, 4>(st, a, n_layers);
  return launch_stream<TT, NB, SPLIT, OWN_ROWS, 0>(st, a, n_layers);
}
// (with shared units the rows are averaged by one token group on the side: no variant of its own)
template <int TT, int NB, bool SPLIT>
int launch_stream_rows(hipStream_t st, const ScoreArgs& a, int n_layers, int selw) {
  return SPLIT || a.n_out > 1 ? launch_stream_sel<TT, NB, SPLIT, true>(st, a, n_layers, selw)
                              : launch_stream_sel<TT, NB, SPLIT, SPLIT>(st, a, n_layers, selw);
}
template <int NB, bool SPLIT>
int launch_stream_tt(hipStream_t st, const ScoreArgs& a, int n_layers, int tt, int selw) {
  switch (tt) {
    case 1: return launch_stream_rows<1, NB, SPLIT>(st, a, n_layers, selw);
    case 2: return launch_stream_rows<2, NB, SPLIT>(st, a, n_layers, selw);
    case 3: return launch_stream_rows<3, NB, SPLIT>(st, a, n_layers, selw);
    case 4: return launch_stream_rows<4, NB, SPLIT>(st, a, n_layers, selw);
    default: return launch_stream_rows<5, NB, SPLIT>(st, a, n_layers, selw);
  }
}

// the streaming kernel addresses rows by 32-bit byte offsets from a per-workgroup base
bool stream_takes(const ScoreShape& s) {
  const long long F = (long long)s.n_seg * s.Fs;
  return s.x_dtype == PAFU_BF16 && s.Fs % kS3Slab == 0 && s.M % 256 == 0 && s.ld_x % 8 == 0 &&
         32ll * kS3MaxTT * s.ld_x * 2 < (1ll << 31) && 256ll * F * 2 < (1ll << 31);
}

bool mfma_takes(const ScoreShape& s) {
  return s.x_dtype == PAFU_BF16 && s.Fs % kScSlab == 0 && s.M % 32 == 0 && s.ld_x % 8 == 0;
}
// (rows are 16-byte aligned by the entry points' checks)
bool f32_takes(const ScoreShape& s) { return s.x_dtype == PAFU_F32 && s.Fs % 4 == 0; }

template <int MB>
int launch_mfma(hipStream_t st, const ScoreArgs& a, int n_layers) {
  static LdsLimit lds_limit;
  const int rc = set_lds_limit(lds_limit, score_mfma_kernel<MB>, sc_lds_bytes(MB));
  if (rc != PAFU_OK) return rc;
  hipLaunchKernelGGL(score_mfma_kernel<MB>, dim3((a.T + kScTokPerWg - 1) / kScTokPerWg, n_layers), dim3(kScThreads),
                     sc_lds_bytes(MB), st, a);
  return check_launch();
}

}  // namespace

bool score_batchable(const ScoreShape& s) {
  return s.n_out <= kScoreFoldMax && (stream_takes(s) || mfma_takes(s) || f32_takes(s));
}

int launch_score(hipStream_t st, const ScoreShape& s, const ScoreLayer* layers, int n_layers, void* fold_ws, void* scratch,
                 size_t scratch_bytes, const SelectJob* ride, bool* rode) {
  if (rode != nullptr) *rode = false;
  if (s.T <= 0 || n_layers <= 0) return PAFU_OK;
  if (n_layers > 1 && (n_layers > kScoreBatchMax || !score_batchable(s))) return PAFU_ERR_SHAPE;  // callers ask first
  ScoreArgs a;
  a.T = s.T; a.Fs = s.Fs; a.F = s.n_seg * s.Fs; a.ld_x = s.ld_x; a.M = s.M; a.act = s.act; a.n_out = s.n_out;
  a.inv_out = 1.0f / (float)s.n_out;
  for (int l = 0; l < n_layers; ++l) a.layer[l] = layers[l];
  a.n_layers = n_layers;
  a.groups = 0;
  a.splits = 1;
  a.acts = a.w2bar = nullptr;
  a.ld_acts = 0;
  a.ride = SelectJob{nullptr, nullptr, nullptr, 0, 0, 0};
  const bool stream = stream_takes(s);
  ScorePlan plan{1, 2, 1};
  if (stream) {
    const bool may_split = scratch != nullptr && aligned16(scratch) && scratch_bytes >= split_scratch_bytes(s.T, s.M, n_layers);
    plan = plan_score(s.T, a.F, s.M, n_layers, may_split);
  }
  // Who averages the output rows.  A kernel does it at the end of a pass, about 3 us for 12 rows, a launch of its own takes
  // 4.7 us: in the kernel for several layers, for a single pass per workgroup, for shared units (where one token group does
  // it for all) and for the few units of the fp32 kernel (21840 tokens of 4608 features and 1024 units: 249 us with it in
  // all four passes, 235 with the launch).
  const bool own_rows = n_layers > 1 || (stream ? plan.splits > 1 || s.M == 256 : f32_takes(s));
  if (s.n_out > 1 && !(own_rows && score_batchable(s))) {
    float* w = static_cast<float*>(fold_ws);
    ScoreLayer& first = a.layer[0];
    hipLaunchKernelGGL(fold_w2_kernel, dim3((s.M + 1 + 255) / 256), dim3(256), 0, st, first.W2, first.b2, s.M, s.n_out, w);
    int rc = check_launch();
    if (rc != PAFU_OK) return rc;
    first.W2 = w;
    first.b2 = w + s.M;
    a.n_out = 1;
    a.inv_out = 1.f;
  }
  if (stream) {
    a.groups = ((s.T + 31) / 32 + plan.tt - 1) / plan.tt;
    a.splits = plan.splits;
    if (a.splits > 1) {
      a.acts = static_cast<float*>(scratch);
      a.ld_acts = split_ld(s.T);
      a.w2bar = a.acts + (long long)n_layers * s.M * a.ld_acts;
    }
    int selw = 0;
    // a selection rides along when the last round of workgroups leaves a CU for it (one more workgroup would otherwise be
    // a round of its own) and the list fits the 512-thread bit-sliced selection
    if (ride != nullptr && (long long)a.groups * a.splits % compute_units() != 0 && ride->n > 0 && ride->n <= 512 * 32 * 4) {
      a.ride = *ride;
      if (a.ride.n_pinned < 0) a.ride.n_pinned = 0;
      selw = a.ride.n <= 512 * 32 * 2 ? 2 : 4;
      if (rode != nullptr) *rode = true;
    }
    if (plan.splits == 1) return launch_stream_tt<2, false>(st, a, n_layers, plan.tt, selw);
    return plan.nb == 2 ? launch_stream_tt<2, true>(st, a, n_layers, plan.tt, selw)
                        : launch_stream_tt<1, true>(st, a, n_layers, plan.tt, selw);
  }
  if (mfma_takes(s)) {
    if (s.M % 128 == 0) return launch_mfma<4>(st, a, n_layers);
    return s.M % 64 == 0 ? launch_mfma<2>(st, a, n_layers) : launch_mfma<1>(st, a, n_layers);
  }
  if (f32_takes(s)) {
    hipLaunchKernelGGL(score_f32_kernel, dim3((s.T + 15) / 16, n_layers), dim3(256), 0, st, a);
    return check_launch();
  }
  const ScoreLayer& L = a.layer[0];
  const dim3 grid((s.T + 15) / 16);
  if (s.x_dtype == PAFU_BF16)
    hipLaunchKernelGGL(score_generic_kernel<true>, grid, dim3(256), 0, st, L.x[0], L.x[1], L.x[2], s.n_seg, s.T, s.Fs, s.ld_x,
                       L.W1, L.b1, L.W2, L.b2, s.M, s.act, L.out);
  else
    hipLaunchKernelGGL(score_generic_kernel<false>, grid, dim3(256), 0, st, L.x[0], L.x[1], L.x[2], s.n_seg, s.T, s.Fs, s.ld_x,
                       L.W1, L.b1, L.W2, L.b2, s.M, s.act, L.out);
  return check_launch();
}

}  // namespace pafu
