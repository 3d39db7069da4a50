// Exact dequantization of NVFP4 and HiF4 codes to 16-bit MFMA operands on
// gfx950, shared by the GEMM kernels of those formats.
//
// NVFP4: every product q * d of an E2M1 code and an E4M3 scale is exact in
// fp16: q has at most 2 significant bits and |q| <= 6, d has at most 4 and
// lies in [2^-9, 448], so q d has at most 6 significant bits and lies in
// [2^-10, 2688], inside fp16's normal range.  A pair of codes is decoded to
// fp16 and scaled by one packed multiply: 2 instructions per pair.
//
// HiF4: every value E6M2 * 2^(E1_8 + E1_16) * S1P2 has at most 6 significant
// bits and an exponent in [-50, 17]: exact in bf16 (fp16's range is too
// small).
#pragma once

#include "sharq_device.hpp"

namespace sharq {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 q) { return __builtin_bit_cast(bf16x8, q); }
__device__ __forceinline__ f16x8 as_f16x8(uint4 q) { return __builtin_bit_cast(f16x8, q); }

// Place of the 16-byte parts of a row of 32 staged 16-bit values (64 bytes)
__device__ __forceinline__ int swz_nv(int row) { return ((row >> 1) ^ (row >> 3)) & 3; }

// an E4M3 scale as an fp16 pair (exact)
__device__ __forceinline__ f16x2 nv_scale2(uint32_t code) {
  const _Float16 h = (_Float16)e4m3_value(code);
  return f16x2{h, h};
}

// codes byte SEL (two E2M1 values, lower position in the low nibble) times
// the scale pair d -> one packed fp16 pair
template <int SEL>
__device__ __forceinline__ uint32_t f16_pair(uint32_t codes, f16x2 d) {
  const f16x2 v = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(codes, 1.0f, SEL);
  return __builtin_bit_cast(uint32_t, v * d);
}

// eight codes -> eight fp16 values
__device__ __forceinline__ uint4 nv_dequant8(uint32_t codes, f16x2 d) {
  return make_uint4(f16_pair<0>(codes, d), f16_pair<1>(codes, d), f16_pair<2>(codes, d), f16_pair<3>(codes, d));
}

// Eight codes times scale d -> eight bf16 values.  The fp32 products have at
// most 6 significant bits, so dropping the low 16 bits is exact.
__device__ __forceinline__ uint4 dequant8_bf16(uint32_t codes, float d) {
  uint32_t o[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v2f v;
    switch (i) {
      case 0: v = fp4x2_decode<0>(codes); break;
      case 1: v = fp4x2_decode<1>(codes); break;
      case 2: v = fp4x2_decode<2>(codes); break;
      default: v = fp4x2_decode<3>(codes); break;
    }
    const float a = v.x * d, b = v.y * d;
    o[i] = __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
  }
  return make_uint4(o[0], o[1], o[2], o[3]);
}

// The two scales E6M2 * 2^(E1_8 + E1_16) of dword t (positions 8 t .. 8 t + 7,
// two groups of 4) of half hb of a HiF4 unit, from its metadata word [E6M2,
// E1_8, E1_16 low, E1_16 high].  An E6M2 code's fields are the top of a float
// (exponent bias 48 against 127, 2 mantissa bits), so scale and exponents are
// integer adds.
struct HfScales {
  float lo, hi;   // positions 0-3, 4-7 of the dword
};
__device__ __forceinline__ HfScales hf_scales(uint32_t word, int hb, int t) {
  const uint32_t e8 = word >> (8 + 4 * hb + t), e16 = word >> (16 + 8 * hb + 2 * t);
  const uint32_t base = (word & 0xFFu) + 4u * (127u - 48u) + 4u * (e8 & 1u);
  HfScales s;
  s.lo = __uint_as_float((base + 4u * (e16 & 1u)) << 21);
  s.hi = __uint_as_float((base + 2u * (e16 & 2u)) << 21);
  return s;
}

// Eight S1P2 codes times their scales -> eight bf16 values, in the order of
// positions 0, 2, 1, 3, 4, 6, 5, 7 (both operands of a product use the same
// one, so the K order inside a dword is free).  A code's magnitude m / 4 is
// looked up as an E4M3 byte by one byte permute for four codes, decoded in
// pairs and scaled in fp32; the products have at most 6 significant bits, so
// dropping the low 16 bits is exact.  24 instructions for 8 values.
__device__ __forceinline__ uint4 hf_dequant8(uint32_t codes, HfScales s) {
  constexpr uint32_t kLo = 0x34302800u, kHi = 0x3E3C3A38u;   // E4M3 of 0, .25, .5, .75 and 1, 1.25, 1.5, 1.75
  const uint32_t ev = __builtin_amdgcn_perm(kHi, kLo, codes & 0x07070707u) | ((codes << 4) & 0x80808080u);
  const uint32_t od = __builtin_amdgcn_perm(kHi, kLo, (codes >> 4) & 0x07070707u) | (codes & 0x80808080u);
  const v2f a = __builtin_amdgcn_cvt_pk_f32_fp8((int)ev, false), b = __builtin_amdgcn_cvt_pk_f32_fp8((int)od, false);
  const v2f c = __builtin_amdgcn_cvt_pk_f32_fp8((int)ev, true), d = __builtin_amdgcn_cvt_pk_f32_fp8((int)od, true);
  const auto pack = [](float x, float y) {
    return __builtin_amdgcn_perm(__float_as_uint(y), __float_as_uint(x), 0x07060302u);
  };
  return make_uint4(pack(a.x * s.lo, a.y * s.lo), pack(b.x * s.lo, b.y * s.lo), pack(c.x * s.hi, c.y * s.hi),
                    pack(d.x * s.hi, d.y * s.hi));
}

}  // namespace sharq
