// Wavefront-level helpers shared by the MFMA decode kernels (gfx950): operand types, bf16 hi/lo splitting,
// lane-row exchanges, DPP row reductions, barrier-free LDS hand-over inside one wavefront, and an LDS Walsh-Hadamard transform.
#pragma once

#include "saw_common.h"

namespace saw {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

#define LDS_AS __attribute__((address_space(3)))
#define GLOBAL_AS __attribute__((address_space(1)))

// x = hi + lo with hi a truncated bf16 and lo a rounded bf16 of the remainder.
__device__ __forceinline__ void split_bf16(float x, uint32_t& hi16, uint32_t& lo16, float& sum) {
  const uint32_t u = __float_as_uint(x);
  const float hf = __uint_as_float(u & 0xffff0000u);
  hi16 = u >> 16;
  uint32_t r = __float_as_uint(x - hf);
  r += 0x7fffu + ((r >> 16) & 1u);
  lo16 = r >> 16;
  sum = hf + __uint_as_float(r & 0xffff0000u);
}

// v_permlane16_swap: x <- rows (a0, b0, a2, b2), y <- rows (a1, b1, a3, b3)   (row = 16 lanes)
__device__ __forceinline__ void swap16(float a, float b, float& x, float& y) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  x = __uint_as_float(r[0]);
  y = __uint_as_float(r[1]);
}
// v_permlane32_swap: x <- rows (a0, a1, b0, b1), y <- rows (a2, a3, b2, b3)
__device__ __forceinline__ void swap32(float a, float b, float& x, float& y) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  x = __uint_as_float(r[0]);
  y = __uint_as_float(r[1]);
}

// v + (v of the lane 16 / 32 away, index xor), as two register permutes instead of a trip through
// the LDS crossbar (ds_bpermute)
__device__ __forceinline__ float add_xor16(float v) {
  float x, y;
  swap16(v, v, x, y);              // x rows (v0, v0, v2, v2), y rows (v1, v1, v3, v3)
  return x + y;
}
__device__ __forceinline__ float add_xor32(float v) {
  float x, y;
  swap32(v, v, x, y);              // x rows (v0, v1, v0, v1), y rows (v2, v3, v2, v3)
  return x + y;
}
__device__ __forceinline__ float max_xor16(float v) {
  float x, y;
  swap16(v, v, x, y);
  return fmaxf(x, y);
}
__device__ __forceinline__ float max_xor32(float v) {
  float x, y;
  swap32(v, v, x, y);
  return fmaxf(x, y);
}

// (every lane has a source in the rotations, mirrors and permutations used here; with bound_ctrl the move is folded into its user)
template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true); }
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) { return __uint_as_float(dpp_i<CTRL>((int)__float_as_uint(v))); }
// max over the 16 lanes of each row (rotations by 1, 2, 4, 8)
__device__ __forceinline__ float row_allmax(float v) {
  v = fmaxf(v, dpp_f<0x121>(v));
  v = fmaxf(v, dpp_f<0x122>(v));
  v = fmaxf(v, dpp_f<0x124>(v));
  v = fmaxf(v, dpp_f<0x128>(v));
  return v;
}
// the same of numbers from 0 on, as integers: no instructions to quiet NaNs, one of which may be the result
__device__ __forceinline__ float row_allmax_positive(float v) {
  int u = (int)__float_as_uint(v);
  u = max(u, dpp_i<0x121>(u));
  u = max(u, dpp_i<0x122>(u));
  u = max(u, dpp_i<0x124>(u));
  u = max(u, dpp_i<0x128>(u));
  return __uint_as_float((uint32_t)u);
}
__device__ __forceinline__ float row_allsum(float v) {
  v += dpp_f<0x121>(v);
  v += dpp_f<0x122>(v);
  v += dpp_f<0x124>(v);
  v += dpp_f<0x128>(v);
  return v;
}

// The block is one wavefront: LDS operations of a wave execute in order, so exchanging data
// between lanes through LDS needs no barrier and no wait, only a point the compiler will not
// move memory accesses across.  (A workgroup barrier would also wait for every LDS-DMA transfer
// in flight, which is exactly what the prefetch must not do.)
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// In-place un-normalised block Walsh-Hadamard transform (block size h = 16, 32, 64 or 128) of NVEC
// vectors of 128 floats in LDS (16-byte aligned), run by one wavefront.  Three passes with eight
// values per lane in registers: strides 1-2-4 inside chunks of eight contiguous values, strides
// 8-16-32 over values eight apart (as far as h reaches), and stride 64 when h = 128.
template <int NVEC>
__device__ __forceinline__ void wave_lds_fwht128(float* x, int h, int lane) {
  // (compile-time trip counts: every loop below is unrolled, there is no loop-carried address)
#pragma unroll
  for (int it = 0; it < (NVEC * 16 + 63) / 64; ++it) {
    const int ch = lane + 64 * it;
    if (NVEC * 16 % 64 == 0 || ch < NVEC * 16) {
      f32x4* const p = (f32x4*)(x + 8 * ch);
      const f32x4 a = p[0], b = p[1];
      float e[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
      for (int st = 1; st < 8; st <<= 1)
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (!(k & st)) { const float u = e[k], v = e[k + st]; e[k] = u + v; e[k + st] = u - v; }
      p[0] = f32x4{e[0], e[1], e[2], e[3]};
      p[1] = f32x4{e[4], e[5], e[6], e[7]};
    }
  }
  wave_sync();
#pragma unroll
  for (int it = 0; it < (NVEC * 16 + 63) / 64; ++it) {
    const int g = lane + 64 * it;
    if (NVEC * 16 % 64 == 0 || g < NVEC * 16) {
      float* const p = x + (g >> 4) * 128 + ((g >> 3) & 1) * 64 + (g & 7);
      float e[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) e[k] = p[8 * k];
#pragma unroll
      for (int st = 1; st < 8; st <<= 1) {
        if (8 * st < h) {                                    // wavefront-uniform
#pragma unroll
          for (int k = 0; k < 8; ++k)
            if (!(k & st)) { const float u = e[k], v = e[k + st]; e[k] = u + v; e[k + st] = u - v; }
        }
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) p[8 * k] = e[k];
    }
  }
  wave_sync();
  if (h > 64) {
#pragma unroll
    for (int v = 0; v < NVEC; ++v) {
      float* const b = x + lane;
      const float a = b[v * 128], c = b[v * 128 + 64];
      b[v * 128] = a + c;
      b[v * 128 + 64] = a - c;
    }
    wave_sync();
  }
}

// In-place x <- x M for NV vectors of 128 floats in LDS, run by one wavefront: out[v][j] =
// sum_i x[v][i] M[i][j] with M a global fp32 [128][128] row-major matrix (the learned rotation of
// App. A.3 or its transpose).  Lane l takes four consecutive columns 4 (l % 32) .. + 3 and the rows of
// half l / 32 (rows 64 h .. 64 h + 63): every load is 16 bytes, a load instruction covers two whole rows
// of M, and the 64 loads of a lane go out in four rounds of 16 (what bounds this routine is the latency
// of M coming from L2 while every wavefront of the chip asks for it, so few, wide rounds matter).  Two
// partial sums per output and half (rows of even and odd index), added pairwise at the end, keep the
// rounding error near that of a pairwise sum.  LOADS: of a round, 8 where registers are short (the same sums).
template <int NV, int LOADS = 16>
__device__ __forceinline__ void wave_lds_matvec128(float* x, const float* __restrict__ M, int lane) {
  const int half = lane >> 5, cq = lane & 31;
  float acc[NV][2][4];
#pragma unroll
  for (int v = 0; v < NV; ++v)
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[v][e][c] = 0.f;
  const float* const mbase = M + (64 * half) * 128 + 4 * cq;
#pragma unroll 1
  for (int t = 0; t < 64 / LOADS; ++t) {
    f32x4 m[LOADS];
#pragma unroll
    for (int u = 0; u < LOADS; ++u) m[u] = *(const f32x4*)(mbase + (LOADS * t + u) * 128);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const float* xr = x + v * 128 + 64 * half + LOADS * t;
#pragma unroll
      for (int u4 = 0; u4 < LOADS / 4; ++u4) {
        const f32x4 xv = *(const f32x4*)(xr + 4 * u4);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int u = 4 * u4 + k;
#pragma unroll
          for (int c = 0; c < 4; ++c) acc[v][u & 1][c] = fmaf(xv[k], m[u][c], acc[v][u & 1][c]);
        }
      }
    }
  }
  wave_sync();                                               // every read of x is done
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    f32x4 r;
#pragma unroll
    for (int c = 0; c < 4; ++c) r[c] = add_xor32(acc[v][0][c] + acc[v][1][c]);   // the two halves of the rows
    if (half == 0) *(f32x4*)(x + v * 128 + 4 * cq) = r;
  }
  wave_sync();
}

// Products x[v] M of vectors in LDS by a block of NW (2, 4 or 8) wavefronts: wavefront `wave` takes 128 / NW columns, so that the
// block reads M (64 KiB, from L2) once and not once per wavefront.  A lane's part of M, four columns of ROWS rows, is requested by
// block_columns_load: early, in front of transfers from HBM, because loads return in order.
// Which rows: a sum of wave_lds_matvec128 is four chains of 32 terms, the rows of even and of odd index in either half.  Each row
// of 16 lanes takes one of the chains, SEQ neighbouring groups of lanes the parts of it one after the other, so that
// block_columns_ordered can add up in that very order.
template <int NW>
struct BlockColumns {
  static constexpr int QUADS = 32 / NW;                       // column quads of a wavefront, one per lane of a group
  static constexpr int SEQ = 16 / QUADS;                      // groups that share a chain
  static constexpr int ROWS = 32 / SEQ;                       // rows of M a lane multiplies: row0, row0 + 2, ...
  f32x4 m[ROWS];
  int col, row0;
};
template <int NW>
__device__ __forceinline__ void block_columns_load(const float* __restrict__ M, int wave, int lane, BlockColumns<NW>& k) {
  using K = BlockColumns<NW>;
  k.col = 4 * (K::QUADS * wave + (lane & (K::QUADS - 1)));
  k.row0 = 64 * (lane >> 5) + ((lane >> 4) & 1) + 2 * K::ROWS * ((lane & 15) / K::QUADS);
#pragma unroll
  for (int u = 0; u < K::ROWS; ++u) k.m[u] = *(const f32x4*)(M + (k.row0 + 2 * u) * 128 + k.col);
}
// y[v] = x[v] M in this wavefront's columns, v < NV (x and y are different memory; the caller's barriers)
template <int NV, int NW>
__device__ __forceinline__ void block_columns_product(const float* __restrict__ x, float* __restrict__ y, const BlockColumns<NW>& k, int lane) {
  using K = BlockColumns<NW>;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    float acc[2][4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int u = 0; u < K::ROWS; ++u) {
      const float xu = x[v * 128 + k.row0 + 2 * u];
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[u & 1][c] = fmaf(xu, k.m[u][c], acc[u & 1][c]);
    }
    f32x4 r;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      float t = acc[0][c] + acc[1][c];
      if (K::QUADS <= 4) t += dpp_f<0x124>(t);                // row_ror:4, 8: the row's other lanes of the same columns
      if (K::QUADS <= 8) t += dpp_f<0x128>(t);
      r[c] = add_xor32(add_xor16(t));
    }
    if (lane < K::QUADS) *(f32x4*)(y + v * 128 + k.col) = r;
  }
}
// The same for one or two vectors with every sum in the order of wave_lds_matvec128, bit for bit, whatever NW is: a new token's
// stored scale, zero-point and codes must not depend on which block rotated it.  A chain's running sum goes from group to group; the
// second vector follows the first a group behind.  (Fused step, the new token in any order before: 34 x 120 tokens 14.4 -> 15.3 us, 4 x 256
// 11.5 -> 11.9, 64 ragged up to 4000 45.7 -> 46.3.)
template <int NV, int NW>
__device__ __forceinline__ void block_columns_ordered(const float* __restrict__ x, float* __restrict__ y, const BlockColumns<NW>& k, int lane) {
  using K = BlockColumns<NW>;
  const int seq = (lane & 15) / K::QUADS;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < K::SEQ + NV - 1; ++t) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if constexpr (K::SEQ > 1) acc[c] = dpp_f<0x110 + K::QUADS>(acc[c]);         // row_shr: from the group before; the first gets 0
      else acc[c] = 0.f;
    }
    const float* const xv = x + 128 * min(max(t - seq, 0), NV - 1) + k.row0;
#pragma unroll
    for (int u = 0; u < K::ROWS; ++u) {
      const float xu = xv[2 * u];
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[c] = fmaf(xu, k.m[u][c], acc[c]);
    }
    if (t >= K::SEQ - 1) {                                    // the last group has the whole chain of vector t - (SEQ - 1)
      f32x4 r;
#pragma unroll
      for (int c = 0; c < 4; ++c) r[c] = add_xor32(add_xor16(acc[c]));            // even + odd rows, then the two halves
      if (lane < 16 && seq == K::SEQ - 1) *(f32x4*)(y + 128 * (t - (K::SEQ - 1)) + k.col) = r;
    }
  }
}
// a barrier that waits for this wavefront's LDS accesses only, not for transfers in flight
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_s_waitcnt(0xC07F);                         // lgkmcnt(0)
  wave_sync();
  __builtin_amdgcn_s_barrier();
  wave_sync();
}

}  // namespace saw
