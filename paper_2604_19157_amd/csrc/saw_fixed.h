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

// Weights w = 2^u p s as fixed-point numbers: p = 2^(logit - m) with a reference m per head, the largest logit met when it was set, rounded
// up to a whole number so that sums are scaled by exact powers of two when it moves; and a unit 2^-u per head that puts the largest p s met
// then at 2^(kWeightBits - 1) to 2^kWeightBits.  Both are set anew when a weight outgrows kWeightMost, the most that four digits hold.
// So every weight is rounded to 2^-28 of the largest or finer, and where the n weights of a range fall short of that altogether its
// result is off by n 2^-28 at most; the matrix cores' fp32 sums, cut off at 2^-23 twice a batch, made that up to n 2^-28 too.  A unit
// further up has to be set anew more often; one further down rounds to 2^-27 (64 ragged sequences x 8 single 64-channel heads, eight query
// heads: 26.9 us and 26.7).
// The unit is the head's own, and the scales are in it and not in the reference: scales of other heads cannot reach a head's weights, and
// denominators, sums of p, are at least 1/2 however far apart the scales of ranges, partitions and batches are.
constexpr int kWeightBits = 28;
constexpr float kWeightMost = 2.1e9f;
constexpr float kLeastLogit = -3.402823466e38f;  // references are finite: a logit of -infinity is a weight of 0
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
// ... and a number below 2^54 as such a sum, rounded to a whole one
__device__ __forceinline__ i32x4 long_digits(float x) {
  const int hi = (int)__builtin_rintf(x * 0x1p-24f);
  return i32x4{(int)__builtin_rintf(fmaf((float)hi, -0x1p24f, x)), 0, 0, hi};
}
// the largest of |x|, |y|, .. with a NaN winning
__device__ __forceinline__ float max_or_nan(float a, float b) { return __builtin_elementwise_maximum(a, b); }
// The exponent e that takes a row whose largest element is mx to below 2^30, as far as its unit 2^-e is a number: with 2^-149 every element
// is a whole one as it is (NaN if mx is: an infinity or NaN has no digits, the unit carries it on into everything that is made of the row)
__device__ __forceinline__ int fixed_exponent(float mx) { return min(30 - __builtin_amdgcn_frexp_expf(mx), 149); }
__device__ __forceinline__ float fixed_unit(float mx, int e) { return mx <= 3.402823466e38f ? __builtin_amdgcn_ldexpf(1.f, -e) : __builtin_nanf(""); }

// Eight nibbles n0 .. n7 -> bytes (n0, n2, n4, n6) and (n1, n3, n5, n7)
__device__ __forceinline__ u32x2 code_bytes(uint32_t w) { return u32x2{w & 0x0F0F0F0Fu, (w >> 4) & 0x0F0F0F0Fu}; }
// ... as 16 (n - 8): codes that count from the middle of their range
__device__ __forceinline__ u32x2 centred_bytes(uint32_t w) {
  return u32x2{((w << 4) & 0xF0F0F0F0u) ^ 0x80808080u, (w & 0xF0F0F0F0u) ^ 0x80808080u};
}
__device__ __forceinline__ i32x4 operand(u32x2 a, u32x2 b) { return i32x4{(int)a.x, (int)a.y, (int)b.x, (int)b.y}; }

// The u of weights whose largest p s is big >= 0 (an exponent, because 2^u may be no fp32 number).  0 counts as the smallest number, so that
// whatever follows moves it; of an infinity or NaN any will do.
__device__ __forceinline__ int unit_exponent(float big) {
  return kWeightBits - __builtin_amdgcn_frexp_expf(__uint_as_float((uint32_t)max((int)__float_as_uint(big), 1)));
}

// A head's reference and unit set anew for a batch's logits lg and pairs vm of this lane's four tokens, whose p and w it returns;
// alpha, beta <= 1: what that makes of sums of p and of w.  none: there are no sums yet.  lower: beta is 1/2 at most.
// (The weights as 2^u (p s): 2^u s may overflow where p is small, p s is in range of the unit.)
__device__ __forceinline__ void set_reference(const float (&lg)[4], const f32x2 (&vm)[4], bool none, bool lower, float& m, int& unit,
                                              float (&p)[4], float (&w)[4], float& alpha, float& beta) {
  const float mx = row_allmax(fmaxf(fmaxf(lg[0], lg[1]), fmaxf(lg[2], lg[3])));
  const float mnew = fmaxf(fmaxf(m, kLeastLogit), ceilf(mx));
  float big = 0.f;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    p[q] = fast_exp2(lg[q] - mnew);                           // exp2(-inf) = 0 for masked tokens
    w[q] = p[q] * vm[q].x;
    big = fmaxf(big, fabsf(w[q]));
  }
  int e = unit_exponent(row_allmax_positive(big));
  const int up = (int)fminf(mnew - m, 1000.f);
  if (!none) e = min(e, unit + up - (lower ? 1 : 0));
  alpha = __builtin_amdgcn_ldexpf(1.f, -up);
  beta = __builtin_amdgcn_ldexpf(1.f, e - unit - up);
  m = mnew;
  unit = e;
#pragma unroll
  for (int q = 0; q < 4; ++q) w[q] = __builtin_amdgcn_ldexpf(w[q], e);
}

// The running state of a range: NT tiles of four heads, a lane's head in tile t being 4 t + grp, NC column tiles of 16 channels.
// Accumulators hold 16 times the sum of w (c - 8) as digits.  When the unit or the reference moves they are scaled as fp32 numbers and put
// back as whole numbers; every kFlushAfter batches by a half at least, so that they stay below 2^31: a half of what 1024 batches
// can make of what was there, and 1024 batches' 2^30 on top.
template <int NT, int NC>
struct FixedState {
  // (references to arrays of the kernel's: as members of one object some of them end up in memory)
  i32x4 (&digits)[NT][NC];
  float (&m_ref)[NT];
  int (&unit)[NT];
  float (&lsum)[NT], (&zs)[NT];                               // ... lsum, zs: of the p and of the w (z - 8), of this lane's tokens
  int& room;                                                  // batches until the digits could fill up

  __device__ __forceinline__ void clear() {
    room = kFlushAfter;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      m_ref[t] = -INFINITY; unit[t] = 0; lsum[t] = 0.f; zs[t] = 0.f;
#pragma unroll
      for (int c = 0; c < NC; ++c) digits[t][c] = i32x4{0, 0, 0, 0};
    }
  }

  // The state of tile t opens with one token: its logit, its pair, the codes (c - 8) of this lane's channels 16 c + row16; one: this
  // lane counts it for the head.  Pairs that are not finite carry on into lsum and zs.
  __device__ __forceinline__ void open(int t, float lg, f32x2 m, const float (&code)[NC], bool one) {
    room = kFlushAfter - 1;                                   // (there is something to be scaled)
    m_ref[t] = fmaxf(ceilf(lg), kLeastLogit);
    const float p = fast_exp2(lg - m_ref[t]), ps = p * m.x;
    unit[t] = unit_exponent(fabsf(ps));
    const float w = __builtin_amdgcn_ldexpf(ps, unit[t]);
    lsum[t] = one ? p : 0.f;
    zs[t] = one ? w * (m.y - 8.f) : 0.f;
#pragma unroll
    for (int c = 0; c < NC; ++c) digits[t][c] = long_digits(16.f * w * code[c]);
  }

  // A batch's logits (-infinity: masked; then its scale is 0) of this lane's four tokens and its heads become weights, whose
  // digits go to rows 4 grp + l of tile t.  vm: the tokens' pairs, NM = 1 for all tiles or one set for each.
  // (Sums of the p are checked with the weights: where the scales are small or 0 they would grow without a weight that shows it.)
  template <int NM>
  __device__ __forceinline__ void weigh(const float (&lg)[NT][4], const f32x2 (&vm)[NM][4], uint8_t* pw) {
    float w[NT][4], p[NT][4], sum[NT];
    const bool first = room == kFlushAfter;                   // (wavefront-uniform; nothing is in the state yet)
    bool move = first || room == 0;
    if (!move) {
      float most = 0.f;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          p[t][q] = fast_exp2(lg[t][q] - m_ref[t]);           // exp2(-inf) = 0 for masked tokens
          w[t][q] = p[t][q] * __builtin_amdgcn_ldexpf(vm[t * (NM - 1)][q].x, unit[t]);
          most = max_or_nan(most, fabsf(w[t][q]));
        }
        sum[t] = (p[t][0] + p[t][1]) + (p[t][2] + p[t][3]);
        most = max_or_nan(most, sum[t]);
      }
      move = __any(!(most <= kWeightMost));
    }
    if (move) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        float alpha, beta;
        set_reference(lg[t], vm[t * (NM - 1)], first, room == 0, m_ref[t], unit[t], p[t], w[t], alpha, beta);
        if (!first) {
          lsum[t] *= alpha;
          zs[t] *= beta;
#pragma unroll
          for (int c = 0; c < NC; ++c) digits[t][c] = long_digits(long_digits_value(digits[t][c]) * beta);
        }
        sum[t] = (p[t][0] + p[t][1]) + (p[t][2] + p[t][3]);
      }
      if (room == 0) room = kFlushAfter;
    }
    --room;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      uint32_t u[4], d[4];
      const f32x2 (&m)[4] = vm[t * (NM - 1)];
      float z = w[t][0] * (m[0].y - 8.f);
#pragma unroll
      for (int q = 1; q < 4; ++q) z = fmaf(w[t][q], m[q].y - 8.f, z);
      zs[t] += z;                                             // (one addition a batch to each running sum)
      lsum[t] += sum[t];
#pragma unroll
      for (int q = 0; q < 4; ++q) u[q] = digit_bytes(nearest_int(w[t][q]));
      transpose_digits(u[0], u[1], u[2], u[3], d);
#pragma unroll
      for (int l = 0; l < 4; ++l) *(uint32_t*)(pw + t * kDigitTile + l * kDigitRow) = d[l];
    }
  }

  // the lanes' sums of a head together, in all of its lanes
  __device__ __forceinline__ void sum_lanes() {
#pragma unroll
    for (int t = 0; t < NT; ++t) { lsum[t] = row_allsum(lsum[t]); zs[t] = row_allsum(zs[t]); }
  }
  // ... and then channel 16 c + row16 of this lane's head, not normalised
  __device__ __forceinline__ float value(int t, int c) const {
    return __builtin_amdgcn_ldexpf(fmaf(long_digits_value(digits[t][c]), 1.f / 16.f, -zs[t]), -unit[t]);
  }
};

}  // namespace saw
