// 8-bit storage of the K/V cache: bf16 rows <-> E4M3 codes with one power-of-two scale per tensor.
// (Beyond the paper, which states no storage precision: App. A.)  E4M3 = 1 sign, 4 exponent bits with bias 7,
// 3 mantissa bits, no infinities, S.1111.111 = NaN; round to nearest even; magnitudes beyond 448 saturate.
//
// Both directions use the hardware's conversions: to nearest even after saturation (the cache must match a reference
// bit for bit, and does for every bf16 value), and exact for every code and scale on the way back.
#include "pafu_internal.h"
#include "quant_body.h"

namespace pafu {
namespace {

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;

// Both kernels walk the (row, 8-element chunk) list with the whole grid, one chunk of K and of V per thread at a time.
// Row and chunk advance by the grid's stride, which the host has divided by the chunks of a row: a division per chunk
// takes as many instructions as its conversion.  Bound by HBM: 32760 rows of 12 x 128 to codes and back 130 -> 111 us on
// new inputs (5.4 TB/s; 125 -> 102 us when the same ones are repeated, some of them then in the caches), 80000 of 40 x 128
// 1050 us before and after.  On repeated inputs two or four chunks per thread were slower (104, 108 us); stores that bypass
// the caches leave more of the codes there for whoever reads them next (118 us without).
struct Walk {
  unsigned rows, chunks;    // 8-element chunks per row
  unsigned step_r, step_c;  // grid stride = step_r rows and step_c chunks
};
struct WalkAt {
  unsigned r, c;
  __device__ __forceinline__ explicit WalkAt(const Walk& w) {
    const unsigned i = blockIdx.x * 256u + threadIdx.x;
    r = i / w.chunks;
    c = i - r * w.chunks;
  }
  __device__ __forceinline__ void next(const Walk& w) {
    r += w.step_r;
    c += w.step_c;
    if (c >= w.chunks) { c -= w.chunks; ++r; }
  }
};

__global__ __launch_bounds__(256) void quantize_rows_kernel(const char* __restrict__ K, const char* __restrict__ V,
                                                            long long ld_in, Walk w, float inv_k, float inv_v,
                                                            char* __restrict__ Kq, char* __restrict__ Vq,
                                                            long long ld_out) {
  for (WalkAt at(w); at.r < w.rows; at.next(w)) {
    const long long src = at.r * ld_in + at.c * 16ll, dst = at.r * ld_out + at.c * 8ll;
    const u32x4 in[2] = {*reinterpret_cast<const u32x4*>(K + src), *reinterpret_cast<const u32x4*>(V + src)};
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const unsigned words[4] = {in[t][0], in[t][1], in[t][2], in[t][3]};
      unsigned codes[2];
      e4m3_codes8(words, t ? inv_v : inv_k, codes);
      u32x2 o;
      o[0] = codes[0];
      o[1] = codes[1];
      __builtin_nontemporal_store(o, reinterpret_cast<u32x2*>((t ? Vq : Kq) + dst));
    }
  }
}

__global__ __launch_bounds__(256) void dequantize_rows_kernel(const char* __restrict__ Kq, const char* __restrict__ Vq,
                                                              long long ld_in, Walk w, float k_scale, float v_scale,
                                                              char* __restrict__ K, char* __restrict__ V,
                                                              long long ld_out) {
  for (WalkAt at(w); at.r < w.rows; at.next(w)) {
    const long long src = at.r * ld_in + at.c * 8ll, dst = at.r * ld_out + at.c * 16ll;
    const u32x2 in[2] = {*reinterpret_cast<const u32x2*>(Kq + src), *reinterpret_cast<const u32x2*>(Vq + src)};
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const float scl = t ? v_scale : k_scale;
      u32x4 o;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        o[2 * e] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(in[t][e], scl, false));
        o[2 * e + 1] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(in[t][e], scl, true));
      }
      __builtin_nontemporal_store(o, reinterpret_cast<u32x4*>((t ? V : K) + dst));
    }
  }
}

// grid and its walk over `rows` rows of `chunks` chunks, at most 16 workgroups per CU
int walk_grid(int rows, int chunks, Walk& w) {
  long long blocks = ((long long)rows * chunks + 255) / 256;
  if (blocks > 256 * 16) blocks = 256 * 16;
  if (blocks < 1) blocks = 1;
  w.rows = (unsigned)rows;
  w.chunks = (unsigned)chunks;
  w.step_r = (unsigned)(blocks * 256 / chunks);
  w.step_c = (unsigned)(blocks * 256 % chunks);
  return (int)blocks;
}

}  // namespace

int launch_quantize(hipStream_t st, const void* K, const void* V, long long ld_in_bytes, int rows, int row_elems,
                    int k_scale_log2, int v_scale_log2, void* Kq, void* Vq, long long ld_out_bytes) {
  if (rows <= 0) return PAFU_OK;
  Walk w;
  const int blocks = walk_grid(rows, row_elems / 8, w);
  hipLaunchKernelGGL(quantize_rows_kernel, dim3(blocks), dim3(256), 0, st,
                     static_cast<const char*>(K), static_cast<const char*>(V), ld_in_bytes, w,
                     ldexpf(1.0f, -k_scale_log2), ldexpf(1.0f, -v_scale_log2), static_cast<char*>(Kq),
                     static_cast<char*>(Vq), ld_out_bytes);
  return check_launch();
}

int launch_dequantize(hipStream_t st, const void* Kq, const void* Vq, long long ld_in_bytes, int rows, int row_elems,
                      int k_scale_log2, int v_scale_log2, void* K, void* V, long long ld_out_bytes) {
  if (rows <= 0) return PAFU_OK;
  Walk w;
  const int blocks = walk_grid(rows, row_elems / 8, w);
  hipLaunchKernelGGL(dequantize_rows_kernel, dim3(blocks), dim3(256), 0, st,
                     static_cast<const char*>(Kq), static_cast<const char*>(Vq), ld_in_bytes, w,
                     ldexpf(1.0f, k_scale_log2), ldexpf(1.0f, v_scale_log2), static_cast<char*>(K),
                     static_cast<char*>(V), ld_out_bytes);
  return check_launch();
}

}  // namespace pafu
