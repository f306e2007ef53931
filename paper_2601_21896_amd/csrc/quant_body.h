// E4M3 quantisation of bf16 values (8-bit storage of the K/V cache; beyond the paper, which states no storage
// precision: App. A), shared by the quantisation kernel and by the compaction kernel that quantises the chunk's rows
// behind the retained ones.  E4M3 = 1 sign, 4 exponent bits with bias 7, 3 mantissa bits, no infinities,
// S.1111.111 = NaN; round to nearest even; magnitudes beyond 448 saturate.  The hardware's conversion rounds so; the
// saturation is done before it.  (The same in integer arithmetic was 15 vector instructions per value instead of 4.)
#pragma once
#include "pafu_internal.h"

namespace pafu {
namespace {

// x * inv_scale (exact: inv_scale is a power of two), within the format's range (a NaN stays one)
__device__ __forceinline__ float e4m3_range(float x, float inv_scale) {
  return __builtin_elementwise_minimum(__builtin_elementwise_maximum(x * inv_scale, -448.0f), 448.0f);
}

__device__ __forceinline__ float bf16_lo(unsigned w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(unsigned w) { return __uint_as_float(w & 0xffff0000u); }

// 8 bf16 values (four 32-bit words) -> 8 codes (two words)
__device__ __forceinline__ void e4m3_codes8(const unsigned (&w)[4], float inv, unsigned (&o)[2]) {
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const unsigned a = w[2 * e], b = w[2 * e + 1];
    int c = __builtin_amdgcn_cvt_pk_fp8_f32(e4m3_range(bf16_lo(a), inv), e4m3_range(bf16_hi(a), inv), 0, false);
    c = __builtin_amdgcn_cvt_pk_fp8_f32(e4m3_range(bf16_lo(b), inv), e4m3_range(bf16_hi(b), inv), c, true);
    // the signs are the inputs' (the conversion loses that of a NaN): their upper bytes, in the codes' order
    const unsigned upper = __builtin_amdgcn_perm(b, a, 0x07050301u);
    o[e] = ((unsigned)c & 0x7f7f7f7fu) | (upper & 0x80808080u);
  }
}

}  // namespace
}  // namespace pafu
