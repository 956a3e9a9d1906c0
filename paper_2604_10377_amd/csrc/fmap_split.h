// Float32 products on the float16 matrix cores (gfx950).
//
// A float32 operand x is scaled by a power of two and split into two float16
// parts, h = f16(s x) and l = f16(s x - h), both round-to-nearest-even: 22
// significant bits and a sign on the residual, so |s x - h - l| <= 2^-23 |s x|
// for values within 2^-17 of the largest one that shares the scale, and at most
// 2^-25 in units where that largest value is 2^13 or more (the short forward:
// 2^9).  Smaller values lose bits to the largest; an entry of the product shows
// it only where that one meets zeros, or values as small, in the other operand.
// (A chunk could be sent to float32 products whenever a group of values lies that
// low, but features with compact or Gaussian support do so as a rule, and their
// tails do not reach the results.)  Of the four part
// products, hh, hl and lh are accumulated in float32 (v_mfma_f32_16x16x32_f16);
// the dropped ll is below 2^-22 relative and random in sign.
//
// Float16 has 5 exponent bits, so each row and each column of a product carries
// its own power-of-two scale: exact to apply, exact to remove from the float32
// sums (ldexp), and lowered together with the sums when a later value would not
// fit.
#pragma once

#include "fmap_device.h"

namespace fmap {

typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// Scaled values of this magnitude or more do not fit (the largest float16 is 65504).
constexpr float kSplitLimit = 65000.f;
// The least that the largest scaled magnitude of a row or column may be: the parts resolve 2^-25, 2^-29 of it, where
// float32 keeps 2^-24.
constexpr float kSplitLeast = 16.f;

// Power-of-two shift that brings values of magnitude <= |m| (given as float bits, sign clear) below 2^(TOP + 1):
// [2^TOP, 2^(TOP + 1)) for normal m.  With TOP = 13 values up to 4 |m| fit, with TOP = 9 up to 64 |m| (values below
// 2^-11 |m| then keep fewer than 22 bits, to 2^-34 |m|).  Clamped so that both 2^shift and 2^-shift are normal numbers;
// zero gives the largest shift.
template <int TOP = 13>
__device__ __forceinline__ int split_shift(uint32_t mbits)
{
    const int e = (int)(mbits >> 23) - 127;
    return max(-126, min(126, TOP - e));
}
__device__ __forceinline__ float split_scale(int shift) { return __uint_as_float((uint32_t)(shift + 127) << 23); }

// x0, x1 times the power of two s, as packed float16 parts.  Each part is one fused multiply-add with a
// float16 result (s x is exact, so nothing is rounded before the float16 rounding); the parts are pinned so
// that the residual takes the packed high parts instead of converting again.
__device__ __forceinline__ void split_pair(float x0, float x1, float s, uint32_t &h, uint32_t &l)
{
    const f16x2_t hv = {(_Float16)__builtin_fmaf(x0, s, 0.f), (_Float16)__builtin_fmaf(x1, s, 0.f)};
    h = __builtin_bit_cast(uint32_t, hv);
    asm("" : "+v"(h));
    const f16x2_t hp = __builtin_bit_cast(f16x2_t, h);
    const f16x2_t lv = {(_Float16)__builtin_fmaf(x0, s, -(float)hp[0]), (_Float16)__builtin_fmaf(x1, s, -(float)hp[1])};
    l = __builtin_bit_cast(uint32_t, lv);
}

__device__ __forceinline__ f32x4 mfma16x16x32f16(u32x4_t a, u32x4_t b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0,
                                                   0, 0);
}

}  // namespace fmap
