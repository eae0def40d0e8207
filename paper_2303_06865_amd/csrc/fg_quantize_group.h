// The group-wise 4-bit quantizer of Section 5, for the kernels that store groups: the quantizer and cache append
// (fg_quant.hip) and the decode attention, which stores the token's own row (fg_attn_decode.hip).  Codes and {min, scale}
// are bit-exact functions of the input: binary32, one rounding per operation, IEEE division.
#pragma once
#include "fg_common.h"

namespace fg {

// Eight lanes cooperate on one group of 64 FP16 values (16 bytes per lane), so a wavefront
// covers eight groups per pass: 1 KiB of coalesced input, 256 B of codes, 64 B of meta.
// H16: the 4.5-bit variant whose {min, scale} pair is stored as two FP16 numbers.  min is an FP16
// input value and needs no rounding; scale becomes the smallest FP16 number >= (max-min)/15, and it
// is that stored scale the codes are computed with (so they still lie in [0, 15] unclamped).
// What bounds the quantizer once its loads are wide and many is the vector ALU, so the per-element work is
// kept to seven instructions: the extrema are taken on FP16 pairs (FP16 -> binary32 is exact and monotone) and
// exchanged between the eight lanes with DPP operands, x - min is one mixed-precision FMA, and the codes are
// converted and gathered a byte at a time.
template <bool H16>
__device__ __forceinline__ void quantize_group_8lanes(const h8_t v, uint32_t& packed, float& mn_out,
                                                      float& scale_out) {
#pragma clang fp contract(off)
  const h2_t v0 = {v[0], v[1]}, v1 = {v[2], v[3]}, v2 = {v[4], v[5]}, v3 = {v[6], v[7]};
  const h2_t mn2 = __builtin_elementwise_min(__builtin_elementwise_min(v0, v1), __builtin_elementwise_min(v2, v3));
  const h2_t mx2 = __builtin_elementwise_max(__builtin_elementwise_max(v0, v1), __builtin_elementwise_max(v2, v3));
  float mn = fminf((float)mn2.x, (float)mn2.y), mx = fmaxf((float)mx2.x, (float)mx2.y);
  mn = fminf(mn, dpp_f32<kDppXor1>(mn));
  mx = fmaxf(mx, dpp_f32<kDppXor1>(mx));
  mn = fminf(mn, dpp_f32<kDppXor2>(mn));
  mx = fmaxf(mx, dpp_f32<kDppXor2>(mx));
  mn = fminf(mn, dpp_f32<kDppHalfMirror>(mn));   // quads are uniform by now: the mirror brings the other quad
  mx = fmaxf(mx, dpp_f32<kDppHalfMirror>(mx));
  const float range = mx - mn;
  float scale = range / 15.0f;  // IEEE-rounded division (see build flags)
  if (H16) {
    half_t hs = (half_t)scale;                         // round to nearest ...
    if ((float)hs < scale) {                           // ... then up, if that fell below
      const uint16_t b = __builtin_bit_cast(uint16_t, hs);
      hs = __builtin_bit_cast(half_t, (uint16_t)(b + 1));
    }
    scale = (float)hs;
  }
  uint32_t p = 0;
  if (scale > 0.0f) {
    // The code is rint(Q), Q = the correctly rounded quotient (x - min) / scale.  An IEEE division per
    // element makes this kernel VALU-bound, so the quotient is first taken as (x - min) * rcp(scale):
    // rcp is good to 1 ulp and the product adds half an ulp, so it is within 15 * 1.5 * 2^-23 < 3e-6
    // of the exact quotient, as is Q (half an ulp of 15 = 5e-7).  Both therefore round to the same
    // integer unless the fast quotient lies within 1e-4 of a half-integer; only then (2e-4 of all
    // elements, and every exact tie) the lane redoes its eight elements with the exact division.
    const float inv = __builtin_amdgcn_rcpf(scale);
    float one = 1.0f;
    asm("" : "+v"(one));   // keeps x * 1 - min one mixed-precision FMA (a single rounding, like the subtraction)
    float d[8], r[8], far = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) d[i] = __builtin_fmaf((float)v[i], one, -mn);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float t = d[i] * inv;
      r[i] = rintf(t);  // ties to even
      far = fmaxf(far, fabsf(t - r[i]));
    }
    if (far > 0.4999f) {
#pragma unroll
      for (int i = 0; i < 8; ++i) r[i] = rintf(d[i] / scale);
    }
    // No clamp is needed: d >= 0 and d / scale <= 15 (1 + 2^-22) for finite inputs.  An infinite range has inv = 0, so
    // every r is 0 or NaN, and the conversion takes NaN to 0.
    uint32_t even = 0, odd = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      even = __builtin_amdgcn_cvt_pk_u8_f32(r[2 * i], i, even);
      odd = __builtin_amdgcn_cvt_pk_u8_f32(r[2 * i + 1], i, odd);
    }
    p = even | (odd << 4);
  }
  packed = p;
  mn_out = mn;
  scale_out = scale;
}

}  // namespace fg
