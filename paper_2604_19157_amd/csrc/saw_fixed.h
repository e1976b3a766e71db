// Fixed-point operands of the INT4 decode kernels: 31-bit numbers as four signed byte digits (base 256), one tile row per digit, so
// that v_mfma_i32_16x16x64_i8 multiplies them by 4-bit codes exactly and the sums over channels or tokens are exact as well.
// Rows of a tile are 4 head + digit: lane group grp of a result tile holds the four digits of head grp, column lane % 16.
#pragma once

#include "saw_wave_util.h"

namespace saw {

typedef int i32x4 __attribute__((ext_vector_type(4)));

constexpr int kDigitRow = 80;                  // bytes of a row in LDS: 64 contraction steps and 16 that spread the banks
constexpr int kDigitTile = 16 * kDigitRow;     // four heads

__device__ __forceinline__ i32x4 mfma_i8(i32x4 a, i32x4 b, i32x4 c) { return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0); }

// Weights p s as fixed-point numbers: relative to a reference that puts the largest one met when it was set at kWeightTop, and set anew
// when one outgrows kWeightMost, the most that four digits hold.  So every weight is rounded to 2^-30 of the largest or finer, and
// where the n weights of a range fall short of that altogether its result is off by n 2^-30 at most; the matrix cores' fp32 sums, cut off at 2^-23
// twice a batch, made that up to n 2^-28.  A reference further up would have to be set anew more often.
constexpr float kWeightTop = 536870912.f, kWeightMost = 2.1e9f;
constexpr float kLeastLog = -100.f;            // log2 of the smallest scale that counts for the reference: p stays finite
constexpr int kFlushAfter = 1024;              // batches whose digits, 64 x 128 x 128 at most, add up to less than 2^31

// u = d0 + 256 d1 + 65536 d2 + 2^24 d3 with -128 <= d0, d1, d2 < 128, |u| <= 2.13e9: the digits as bytes
__device__ __forceinline__ uint32_t digit_bytes(int u) { return ((uint32_t)u + 0x00808080u) ^ 0x00808080u; }
// the nearest integer of a number below 2^31 (halves up)
__device__ __forceinline__ int nearest_int(float x) {
  int u;
  asm("v_cvt_rpi_i32_f32 %0, %1" : "=v"(u) : "v"(x));
  return u;
}
// digit l of four numbers as the bytes of out[l]
__device__ __forceinline__ void transpose_digits(uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t (&out)[4]) {
  const uint32_t ab0 = __builtin_amdgcn_perm(b, a, 0x05010400u), ab2 = __builtin_amdgcn_perm(b, a, 0x07030602u);
  const uint32_t cd0 = __builtin_amdgcn_perm(d, c, 0x05010400u), cd2 = __builtin_amdgcn_perm(d, c, 0x07030602u);
  out[0] = __builtin_amdgcn_perm(cd0, ab0, 0x05040100u);
  out[1] = __builtin_amdgcn_perm(cd0, ab0, 0x07060302u);
  out[2] = __builtin_amdgcn_perm(cd2, ab2, 0x05040100u);
  out[3] = __builtin_amdgcn_perm(cd2, ab2, 0x07060302u);
}
// the number that a sum's four digits make, below 2^22 each
__device__ __forceinline__ float digits_value(i32x4 d) {
  return fmaf((float)((d[3] << 8) + d[2]), 65536.f, (float)((d[1] << 8) + d[0]));
}
// the same of long sums, whose digits may fill 31 bits
__device__ __forceinline__ float long_digits_value(i32x4 d) {
  return fmaf(fmaf(fmaf((float)d[3], 256.f, (float)d[2]), 256.f, (float)d[1]), 256.f, (float)d[0]);
}
// the largest of |x|, |y|, .. with a NaN winning
__device__ __forceinline__ float max_or_nan(float a, float b) { return __builtin_elementwise_maximum(a, b); }
// The exponent e that takes a row whose largest element is mx to below 2^30; the row's unit 2^-e (NaN if mx is: an infinity or NaN has
// no digits, the unit carries it on into everything that is made of the row)
__device__ __forceinline__ int fixed_exponent(float mx) { return 30 - __builtin_amdgcn_frexp_expf(mx); }
__device__ __forceinline__ float fixed_unit(float mx, int e) { return mx <= 3.402823466e38f ? __builtin_amdgcn_ldexpf(1.f, -e) : __builtin_nanf(""); }

// Eight nibbles n0 .. n7 -> bytes (n0, n2, n4, n6) and (n1, n3, n5, n7)
__device__ __forceinline__ u32x2 code_bytes(uint32_t w) { return u32x2{w & 0x0F0F0F0Fu, (w >> 4) & 0x0F0F0F0Fu}; }
// ... as 16 (n - 8): codes that count from the middle of their range
__device__ __forceinline__ u32x2 centred_bytes(uint32_t w) {
  return u32x2{((w << 4) & 0xF0F0F0F0u) ^ 0x80808080u, (w & 0xF0F0F0F0u) ^ 0x80808080u};
}
__device__ __forceinline__ i32x4 operand(u32x2 a, u32x2 b) { return i32x4{(int)a.x, (int)a.y, (int)b.x, (int)b.y}; }

}  // namespace saw
