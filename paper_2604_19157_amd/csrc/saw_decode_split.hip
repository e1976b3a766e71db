// INT4 paged decode attention, one 64-channel head at a time, on the gfx950 matrix cores: the head_dim 64 shapes
// whose heads the head-pair kernel cannot take two at a time (an odd number of kv heads, eight query heads per kv head).
// Paper: Sec. 2 (decode step), Sec. 4.1 / App. A.4 (rotated-space attention), App. A.1.
//
// A wavefront walks its share of one (sequence, kv head) in batches of four pages (64 tokens: 512 bytes of K and of
// V codes and 128 bytes of (scale, zero) pairs a page).  Everything is loaded into registers, two batches ahead:
//   * K codes: lane (token = lane % 16, k-group = lane / 16) loads the 16 codes it feeds to the logit MFMA;
//   * V codes: 16 bytes per lane, two pages a load; written to LDS when their batch is due and read back by
//     ds_read_b64_tr_b4 (a 16x16 nibble transpose) with tokens along the contraction;
//   * the pairs: each lane loads those of its own token(s) of the softmax layout.
// With a fifth of the bytes of an LDS-DMA double buffer per wavefront in LDS, registers set the occupancy: three
// wavefronts per SIMD with two batches each in flight, which is what a 5 KiB batch needs to keep HBM busy.
//
// Numerics.  A nibble c, as a byte, is the fp8 (e4m3) number c 2^-9: codes 0-7 are the format's subnormals and 8-15 its
// first binade, which has the same spacing.  One v_cvt_scalef32_pk_bf16_fp8 with scale 2^9 therefore makes two bf16
// integers of two nibbles, without an offset whose removal would cost bits (128 + c, or 16 + c, in the mantissa of a
// constant: twice to three times the error).  The query and the weights p s are
// carried in three bf16 limbs, whose sum is the fp32 value: first and second limbs in separate rows of one tile, third
// limbs in a second product that adds into the first limbs' rows.  So the results are those of fp32 arithmetic.
#include "saw_decode.h"
#include "saw_wave_util.h"
#include "saw_rank.h"
#include "saw_cut.h"

namespace saw {

namespace split64 {

constexpr int D = 64;
constexpr int kTile = 512;                     // one (page, head) code tile: 16 tokens x 32 B
constexpr int kProw = 72;                      // P row stride in bf16 (64 tokens + 8 pad)
constexpr float kLazyTau = 8.0f;               // the reference maximum may lag the true one by 2^8

template <int G>
struct Lds {
  static constexpr int LO = (G > 4) ? 8 : 4;                 // first row of the second limbs
  static constexpr int kV = 4 * kTile;
  static constexpr int kP = 3 * LO * kProw * 2;
  static constexpr int kWave = kV + kP;
};

// Eight nibbles -> eight bf16 integers in k-order (n0, n2, n4, n6, n1, n3, n5, n7)
__device__ __forceinline__ bf16x8 unpack8f(uint32_t w) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const uint32_t even = w & 0x0F0F0F0Fu, odd = (w >> 4) & 0x0F0F0F0Fu;
  u32x4 r;
  r.x = __builtin_bit_cast(uint32_t, (bf16x2)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(even, 512.f, false));
  r.y = __builtin_bit_cast(uint32_t, (bf16x2)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(even, 512.f, true));
  r.z = __builtin_bit_cast(uint32_t, (bf16x2)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(odd, 512.f, false));
  r.w = __builtin_bit_cast(uint32_t, (bf16x2)__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(odd, 512.f, true));
  return as_bf16x8(r);
}
// x = hi + mid + lo, three bf16 values (two truncations; the eight bits that remain are exact)
__device__ __forceinline__ void split3(float x, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
  hi = __float_as_uint(x) >> 16;
  const float r = x - __uint_as_float(hi << 16);
  mid = __float_as_uint(r) >> 16;
  lo = __float_as_uint(r - __uint_as_float(mid << 16)) >> 16;
}

template <int NS>
struct Batch {                                 // one batch as loaded
  u32x2 k[4];                                  // channels 16 grp .. + 15 of token row16 of page q
  u32x4 v[2];                                  // chunk lane % 32 of pages 2 i and 2 i + 1
  f32x2 km[NS], vm[NS];                        // (scale, zero) of this lane's token(s)
};

}  // namespace split64

// NW wavefronts share a partition: wavefront w takes its batches w, w + NW, ...
// p.cut: block x is slot x of the batch cut by its own lengths (saw_cut.h); otherwise partition x of sequence z.
template <int G, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(3, 3)))
void decode_int4_split64_kernel(DecodeParams p) {
  using namespace split64;
  constexpr int LO = Lds<G>::LO;
  constexpr int NS = (G > 4) ? 2 : 1;          // tokens per lane in the softmax layout
  constexpr int NH = (G > 4) ? 4 : G;          // heads per lane in the softmax layout
  constexpr int kWave = Lds<G>::kWave;
  const int kvh = blockIdx.y;
  const int lane = threadIdx.x & 63;
  const int wave = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row16 = lane & 15, grp = lane >> 4;
  __shared__ __attribute__((aligned(16))) uint8_t lds_all[NW * kWave];
  uint8_t* const vbuf = lds_all + wave * kWave;
  uint8_t* const pbuf = vbuf + 4 * kTile;

  // ---- which tokens ----
  int b, part = 0, parts = 1, slot;
  int first, end;                              // batches of the sequence
  int len;
  if (p.cut) {
    const BatchCut cut = cut_batch(p, lane);
    slot = blockIdx.x;
    cut_slot(cut, slot, b, len, part, parts);
    if (b < 0) return;                                        // block-uniform
    if (part == 0 && kvh == 0 && threadIdx.x == 0) p.cut_of[b] = make_int2(slot, parts);
    cut_range((len + 63) >> 6, part, parts, first, end);
  } else {
    // (the partition index is rotated by kv head and sequence, so that no XCD serves a fixed set of partitions)
    slot = (blockIdx.x + blockIdx.y + blockIdx.z) % gridDim.x;
    b = blockIdx.z;
    // (blocks are dispatched in index order: with the caller's order, longest first)
    if (p.sorted) b = min(max(p.order[blockIdx.z], 0), p.batch - 1);
    len = max(min(p.seq_lens[b], p.bound), 0);
    first = slot * (p.chunk_tokens >> 6);
    end = min((len + 63) >> 6, first + (p.chunk_tokens >> 6));
    part = slot;
    parts = 0;                                                // (with an append the first partition takes the token)
    if (first >= end && !(p.append && slot == 0)) {           // block-uniform
      if (p.num_splits == 1)
        for (int i = threadIdx.x; i < G * D; i += 64 * NW)
          store_elem(p.out, p.out_dtype, ((int64_t)b * p.n_q_heads + kvh * G) * D + i, 0.f);
      return;
    }
  }
  b = __builtin_amdgcn_readfirstlane(b);
  len = __builtin_amdgcn_readfirstlane(len);
  first = __builtin_amdgcn_readfirstlane(first);
  end = __builtin_amdgcn_readfirstlane(end);
  const int nb = max(end - first, 0);
  const int t_begin = 64 * first, t_end = min(len, 64 * end);
  // the step's new token goes to a partition with the fewest batches, and there to the wavefront with the fewest
  const bool takes_new = p.append && (p.cut ? part == parts - 1 : part == 0) && wave == NW - 1;

  // ---- page ids: lane l holds that of page 64 window + l of the range; the next window is loaded one ahead ----
  const int64_t pt_row = (int64_t)b * p.max_pages;
  const int pg_first = 4 * first;
  auto load_pids = [&](int at) { return p.page_table[pt_row + min(pg_first + at + lane, p.max_pages - 1)]; };
  auto clamp_pid = [&](int id) { return (id < 0 || id >= p.num_pages) ? 0 : id; };
  int window = 0;
  int pidv = load_pids(0), pidv_nx = load_pids(64);

  // ---- query and new token, requested with the page ids ----
  float qraw[G];                               // channel `lane` of head g
  {
    const int64_t qoff = ((int64_t)b * p.n_q_heads + kvh * G) * D + lane;
    uint32_t bits[G];
    if (p.q_dtype == SAW_F32) {
#pragma unroll
      for (int g = 0; g < G; ++g) bits[g] = ((const uint32_t*)p.q)[qoff + D * g];
    } else {
#pragma unroll
      for (int g = 0; g < G; ++g) bits[g] = ((const uint16_t*)p.q)[qoff + D * g];
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      qraw[g] = p.q_dtype == SAW_F32 ? __uint_as_float(bits[g]) : p.q_dtype == SAW_BF16 ? __uint_as_float(bits[g] << 16)
                                                                                       : f16_to_f32(bits[g] & 0xffffu);
      if (p.rot_k && p.has_signs) qraw[g] = apply_sign(p.signs, lane, qraw[g]);
    }
  }
  uint32_t new_wk = 0, new_wv = 0;             // channels 2 (lane % 32), + 1 of the new K and V (both halves of the wavefront)
  int new_pid = -1;
  if (takes_new) {
    const int64_t e = ((int64_t)b * p.n_kv_heads + kvh) * (D / 2) + (lane & 31);
    new_wk = ((const uint32_t*)p.k_new)[e];
    new_wv = ((const uint32_t*)p.v_new)[e];
    // (a length beyond the caller's bound was clamped for the attention; storing at the clamped
    // position would overwrite a cached token, so such a token is attended to but not stored; nor is one of a length below
    // zero, whose position is no position)
    if ((len >> 4) < p.max_pages && (uint32_t)p.seq_lens[b] <= (uint32_t)p.bound) new_pid = p.page_table[pt_row + (len >> 4)];
  }
  pidv = clamp_pid(pidv);

  // ---- fetch ----
  const int64_t page_stride = (int64_t)p.n_kv_heads * kTile, head_tile = (int64_t)kvh * kTile;
  const int64_t page_meta = (int64_t)p.n_kv_heads * 32, head_meta = (int64_t)kvh * 32;       // floats
  auto fetch = [&](int bi, Batch<NS>& r) __attribute__((always_inline)) {
    if ((bi >> 4) != window) {
      window = bi >> 4;
      pidv = clamp_pid(pidv_nx);
      pidv_nx = load_pids(64 * window + 64);
    }
    int id[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) id[q] = __builtin_amdgcn_readlane(pidv, 4 * (bi & 15) + q);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      r.k[q] = __builtin_nontemporal_load((const u32x2*)(p.k_codes + (int64_t)id[q] * page_stride + head_tile + 32 * row16 + 8 * grp));
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int pid = lane < 32 ? id[2 * i] : id[2 * i + 1];
      r.v[i] = __builtin_nontemporal_load((const u32x4*)(p.v_codes + (int64_t)pid * page_stride + head_tile + 16 * (lane & 31)));
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int pid = (G > 4) ? (lane < 32 ? id[2 * s] : id[2 * s + 1])
                              : (grp == 0 ? id[0] : grp == 1 ? id[1] : grp == 2 ? id[2] : id[3]);
      const int64_t m = (int64_t)pid * page_meta + head_meta + 2 * row16;
      r.km[s] = __builtin_nontemporal_load((const f32x2*)(p.k_meta + m));
      r.vm[s] = __builtin_nontemporal_load((const f32x2*)(p.v_meta + m));
    }
  };
  const int mine = (nb > wave) ? (nb - wave + NW - 1) / NW : 0;         // this wavefront's batches
  Batch<NS> ra, rb;
  if (mine > 0) fetch(wave, ra);
  if (mine > 1) fetch(wave + NW, rb);

  // ---- q~ = (q R) sm_scale log2(e) as A operands ----
  // lane (row16, grp) holds channels 16 grp + 8 kk + {0, 2, 4, 6, 1, 3, 5, 7} of head row16 % LO
  u32x4 a_q[2], a_q3[2];
  float qsum[NH];
  {
    float* const qs = (float*)vbuf;
#pragma unroll
    for (int g = 0; g < G; ++g) qs[D * g + lane] = qraw[g];
    wave_sync();
    float qmul = p.q_scale;
    if (p.rot_k) {
      wave_lds_fwht128<(G + 1) / 2>(qs, p.had_block, lane);  // two 64-channel rows are one 128-channel vector (G = 1: half of one)
      qmul *= had_norm(p.had_block);
    }
    const bool second = (row16 & LO) != 0;
    const int head = row16 & (LO - 1);
    const float qm = (row16 < 2 * LO && head < G) ? qmul : 0.f;
    const float* const qrow = qs + (head < G ? head : 0) * D + 16 * grp;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const f32x4 va = *(const f32x4*)(qrow + 8 * kk), vb = *(const f32x4*)(qrow + 8 * kk + 4);
      uint32_t w[4], w3[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        uint32_t h0, m0, l0, h1, m1, l1;
        // dword j packs channels 4 (j & 1) + (j >> 1) and that + 2
        split3((j & 1 ? vb : va)[j >> 1] * qm, h0, m0, l0);
        split3((j & 1 ? vb : va)[(j >> 1) + 2] * qm, h1, m1, l1);
        w[j] = second ? (m0 | (m1 << 16)) : (h0 | (h1 << 16));
        w3[j] = second ? 0u : (l0 | (l1 << 16));
      }
      a_q[kk] = u32x4{w[0], w[1], w[2], w[3]};
      a_q3[kk] = u32x4{w3[0], w3[1], w3[2], w3[3]};
    }
    // qsum = sum over channels of q~: row sums by a product with a matrix of ones
    f32x4 rs = f32x4{0.f, 0.f, 0.f, 0.f};
    const bf16x8 ones = as_bf16x8(u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u});
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      rs = mfma_bf16(as_bf16x8(a_q3[kk]), ones, rs);
      rs = mfma_bf16(as_bf16x8(a_q[kk]), ones, rs);
    }
#pragma unroll
    for (int i = 0; i < NH; ++i) {
      float t = rs[i];
      if (G <= 4) t = add_xor16(t);
      qsum[i] = add_xor32(t);
    }
    wave_sync();
  }

  // ---- per-lane constants ----
  // V in LDS: 16-byte chunk Q of token t at chunk 2 t + (Q ^ (t / 8)) of the page's tile, which spreads the rows that
  // share a bank; the transpose read of channels 16 c .. + 15 takes half c & 1 of chunk c >> 1
  const int vw_off = kTile * (lane >> 5) + 16 * (((lane & 31) & ~1) + ((lane & 1) ^ ((lane >> 4) & 1)));
  int vr_off[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) vr_off[c] = grp * kTile + 16 * (2 * row16 + ((c >> 1) ^ (row16 >> 3))) + 8 * (c & 1);
  // P column of token t of a page: 16 page + 8 (t / 8) + perm^-1(t % 8), the k-order of the unpacked nibbles
  const int pcol_t = (row16 & 8) + (((row16 & 1) << 2) | ((row16 >> 1) & 3));
  const int head0 = (G > 4) ? 4 * (grp & 1) : 0;              // first head of this lane
  const uint16_t* const pa = (const uint16_t*)pbuf + (row16 & (2 * LO - 1)) * kProw + 16 * grp;
  const uint16_t* const pa3 = (const uint16_t*)pbuf + (2 * LO + (row16 & (LO - 1))) * kProw + 16 * grp;
  const uint32_t third_rows = (row16 < LO) ? 0xffffffffu : 0u;

  f32x4 oacc[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) oacc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_ref[NH], lsum[NH], zs[NH];
#pragma unroll
  for (int i = 0; i < NH; ++i) { m_ref[i] = -INFINITY; lsum[i] = 0.f; zs[i] = 0.f; }

  // One batch whose first token is position tok0; tokens from t_lim on are masked.  `next` requests the batch
  // that takes these registers next, as soon as they are consumed.
  auto body = [&](Batch<NS>& r, int tok0, int t_lim, auto&& next) __attribute__((always_inline)) {
    f32x4 dq[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const bf16x8 kb = unpack8f(r.k[q][kk]);
        acc = mfma_bf16(as_bf16x8(a_q3[kk]), kb, acc);
        acc = mfma_bf16(as_bf16x8(a_q[kk]), kb, acc);
      }
      dq[q] = acc;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) *(u32x4*)(vbuf + 2 * kTile * i + vw_off) = r.v[i];
    f32x2 km[NS], vm[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) { km[s] = r.km[s]; vm[s] = r.vm[s]; }
    next(r);
    // ---- gather: limbs added, lane = token of the batch, registers = heads ----
    float lg[NS][NH];
    bool valid[NS];
    bool need = false;
#pragma unroll
    for (int s = 0; s < NS; ++s) valid[s] = tok0 + 16 * ((G > 4) ? 2 * s + (lane >> 5) : grp) + row16 < t_lim;
#pragma unroll
    for (int i = 0; i < NH; ++i) {
      float raw[NS];
      if constexpr (G > 4) {        // tile rows: first limbs of heads 0-3 | 4-7 | second limbs of 0-3 | 4-7
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          float hi, lo;
          swap32(dq[2 * s][i], dq[2 * s + 1][i], hi, lo);
          raw[s] = hi + lo;
        }
      } else {                      // first limbs | second limbs | idle | idle
        float h01, l01, h23, l23, hi, lo, junk;
        swap16(dq[0][i], dq[1][i], h01, l01);
        swap16(dq[2][i], dq[3][i], h23, l23);
        swap32(h01, h23, hi, junk);
        swap32(l01, l23, lo, junk);
        raw[0] = hi + lo;
      }
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const float v = km[s].x * fmaf(-km[s].y, qsum[i], raw[s]);
        lg[s][i] = valid[s] ? v : -INFINITY;
        need |= lg[s][i] > m_ref[i] + kLazyTau;
      }
    }
    if (__any(need)) {
#pragma unroll
      for (int i = 0; i < NH; ++i) {
        float mx = lg[0][i];
        if (NS > 1) mx = fmaxf(mx, lg[NS - 1][i]);
        mx = row_allmax(mx);
        if (G <= 4) mx = max_xor16(mx);                       // eight heads: lanes 32 apart share the head group
        mx = max_xor32(mx);
        const float mnew = fmaxf(m_ref[i], mx);
        const float alpha = fast_exp2(m_ref[i] - mnew);       // 0 on the first batch
        lsum[i] *= alpha;
        zs[i] *= alpha;
#pragma unroll
        for (int c = 0; c < 4; ++c) oacc[c][i] *= alpha;
        m_ref[i] = mnew;
      }
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int col = 16 * ((G > 4) ? 2 * s + (lane >> 5) : grp) + pcol_t;
      const float vs = valid[s] ? vm[s].x : 0.f;
      const float vz = valid[s] ? vm[s].y - 8.f : 0.f;                 // (codes count from 8: see below)
#pragma unroll
      for (int i = 0; i < NH; ++i) {
        const float pr = fast_exp2(lg[s][i] - m_ref[i]);      // exp2(-inf) = 0 for masked tokens
        lsum[i] += pr;
        const float w = pr * vs;
        zs[i] = fmaf(w, vz, zs[i]);
        uint32_t h, m, l;
        split3(w, h, m, l);
        uint16_t* const pw = (uint16_t*)pbuf + (head0 + i) * kProw + col;
        pw[0] = (uint16_t)h;
        pw[LO * kProw] = (uint16_t)m;
        pw[2 * LO * kProw] = (uint16_t)l;
      }
    }
    wave_sync();
    // ---- O[row][channel] += P (rows x 64 tokens) . V codes ----
    const u32x4 p0 = *(const u32x4*)pa, p1 = *(const u32x4*)(pa + 8);
    u32x4 q0 = *(const u32x4*)pa3, q1 = *(const u32x4*)(pa3 + 8);
    q0 &= u32x4{third_rows, third_rows, third_rows, third_rows};
    q1 &= u32x4{third_rows, third_rows, third_rows, third_rows};
    // The batch's sums start at -8 sum w (a product with a matrix of -8) and are then added to the running ones: the
    // codes count from the middle of their range, so that the running sums stay as small as the values they stand
    // for (a range of 5000 tokens: 3e-5 of the output off without this, 3e-6 with it).
    const bf16x8 eights = as_bf16x8(u32x4{0xc100c100u, 0xc100c100u, 0xc100c100u, 0xc100c100u});
    f32x4 mid = f32x4{0.f, 0.f, 0.f, 0.f};
    mid = mfma_bf16(as_bf16x8(q0), eights, mid);
    mid = mfma_bf16(as_bf16x8(q1), eights, mid);
    mid = mfma_bf16(as_bf16x8(p0), eights, mid);
    mid = mfma_bf16(as_bf16x8(p1), eights, mid);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const i32x2 tv = __builtin_amdgcn_ds_read_tr4_b64_v2i32((LDS_AS i32x2*)(vbuf + vr_off[c]));
      const bf16x8 v0 = unpack8f((uint32_t)tv.x), v1 = unpack8f((uint32_t)tv.y);
      f32x4 t = mfma_bf16(as_bf16x8(q0), v0, mid);
      t = mfma_bf16(as_bf16x8(q1), v1, t);
      t = mfma_bf16(as_bf16x8(p0), v0, t);
      t = mfma_bf16(as_bf16x8(p1), v1, t);
      oacc[c] += t;
    }
    wave_sync();                                              // V and P are rewritten by the next batch
  };
  for (int n = 0; n < mine; n += 2) {
    const int bi = wave + NW * n;
    body(ra, t_begin + 64 * bi, t_end, [&](Batch<NS>& r) { if (n + 2 < mine) fetch(bi + 2 * NW, r); });
    if (n + 1 < mine)
      body(rb, t_begin + 64 * (bi + NW), t_end, [&](Batch<NS>& r) { if (n + 3 < mine) fetch(bi + 3 * NW, r); });
  }

  // ---- fused append: the step's new token as one more batch in which only token 0 is valid ----
  // Rotated, quantised (Sec. 3 eqs. 1-3, App. A.1) and stored as the store kernel would; what attends to it
  // comes from LDS, nothing this launch writes to the cache is read back by it.
  if (takes_new) {
    float* const yb = (float*)vbuf;                           // [2][64]: K, V
    uint8_t* const cb = vbuf + 1024;                          // code bytes of K, V
    const bool rot[2] = {p.rot_k != 0, p.rot_v != 0};
    float x[2][2];
    if (p.kv_new_dtype == SAW_BF16) { widen2<SAW_BF16>(new_wk, x[0][0], x[0][1]); widen2<SAW_BF16>(new_wv, x[1][0], x[1][1]); }
    else                            { widen2<SAW_F16>(new_wk, x[0][0], x[0][1]);  widen2<SAW_F16>(new_wv, x[1][0], x[1][1]); }
    const int c2 = 2 * (lane & 31);
    if (rot[0] || rot[1]) {
      if (p.has_signs) {
#pragma unroll
        for (int w = 0; w < 2; ++w)
          if (rot[w]) {
            x[w][0] = apply_sign(p.signs, c2, x[w][0]);
            x[w][1] = apply_sign(p.signs, c2 + 1, x[w][1]);
          }
      }
      // K and V are one 128-channel vector of two blocks; a tensor that is not rotated keeps its values
      const int w = lane >> 5;
      *(f32x2*)(yb + D * w + c2) = f32x2{x[w][0], x[w][1]};
      wave_sync();
      wave_lds_fwht128<1>(yb, p.had_block, lane);
#pragma unroll
      for (int t = 0; t < 2; ++t)
        if (rot[t]) {
          const f32x2 y = *(const f32x2*)(yb + D * t + c2);
          x[t][0] = y.x; x[t][1] = y.y;
        }
      wave_sync();
    }
    uint32_t byte[2];
    f32x2 meta[2];
#pragma unroll
    for (int w = 0; w < 2; ++w) {
      const float mx = max_xor16(row_allmax(fmaxf(x[w][0], x[w][1])));       // over the 32 lanes of a half
      const float mn = -max_xor16(row_allmax(-fminf(x[w][0], x[w][1])));
      const float norm = rot[w] ? had_norm(p.had_block) : 1.0f;
      const float range = mx - mn;
      float inv, zq, s_store, z_store;
      if (range > 0.0f) {
        inv = 15.0f / range;
        s_store = range * (norm * (1.0f / 15.0f));
        zq = rintf(-mn * inv);
        z_store = zq;
      } else {  // constant vector
        inv = 0.0f;
        zq = 0.0f;
        s_store = (mn != 0.0f) ? fabsf(mn) * norm : 1.0f;
        z_store = (mn > 0.0f) ? -1.0f : ((mn < 0.0f) ? 1.0f : 0.0f);
      }
      const float q0 = __builtin_amdgcn_fmed3f(rintf(x[w][0] * inv) + zq, 0.0f, 15.0f);
      const float q1 = __builtin_amdgcn_fmed3f(rintf(x[w][1] * inv) + zq, 0.0f, 15.0f);
      byte[w] = (uint32_t)q0 | ((uint32_t)q1 << 4);
      meta[w] = f32x2{s_store, z_store};
      if (lane < 32) cb[32 * w + lane] = (uint8_t)byte[w];
    }
    wave_sync();
    Batch<NS> r;
#pragma unroll
    for (int q = 0; q < 4; ++q) r.k[q] = u32x2{0u, 0u};
    r.k[0] = *(const u32x2*)(cb + 8 * grp);                   // (rows other than token 0 are masked)
    r.v[0] = *(const u32x4*)(cb + 32 + 16 * (lane & 1));
    r.v[1] = r.v[0];
#pragma unroll
    for (int s = 0; s < NS; ++s) { r.km[s] = meta[0]; r.vm[s] = meta[1]; }
    wave_sync();
    body(r, 0, 1, [](Batch<NS>&) {});
    // (nobody waits for these stores)
    if (new_pid >= 0 && new_pid < p.num_pages && lane < 32) {
      const int64_t vec = ((int64_t)new_pid * p.n_kv_heads + kvh) * 16 + (len & 15);
      const_cast<uint8_t*>(p.k_codes)[vec * (D / 2) + lane] = (uint8_t)byte[0];
      const_cast<uint8_t*>(p.v_codes)[vec * (D / 2) + lane] = (uint8_t)byte[1];
      if (lane == 0) {
        *(f32x2*)(const_cast<float*>(p.k_meta) + vec * 2) = meta[0];
        *(f32x2*)(const_cast<float*>(p.v_meta) + vec * 2) = meta[1];
      }
    }
  }

  // ---- this wavefront's record in its own LDS: acc[G][64] un-normalised, then (max, sum) per head ----
#pragma unroll
  for (int i = 0; i < NH; ++i) {
    lsum[i] = row_allsum(lsum[i]);
    zs[i] = row_allsum(zs[i]);
    if (G <= 4) { lsum[i] = add_xor16(lsum[i]); zs[i] = add_xor16(zs[i]); }
    lsum[i] = add_xor32(lsum[i]);
    zs[i] = add_xor32(zs[i]);
  }
  const bool writer = (G > 4) ? (grp < 2) : (grp == 0);
  float* const rec = (float*)vbuf;
#pragma unroll
  for (int i = 0; i < NH; ++i) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float o = (G > 4) ? add_xor32(oacc[c][i]) : add_xor16(oacc[c][i]);
      if (writer) rec[(head0 + i) * D + 16 * c + row16] = o - zs[i];
    }
    if (writer && row16 == 0) { rec[G * D + 2 * (head0 + i)] = m_ref[i]; rec[G * D + 2 * (head0 + i) + 1] = lsum[i]; }
  }
  if (NW > 1) __syncthreads(); else wave_sync();

  // ---- combine the block's records, a few heads per wavefront ----
  constexpr int HPW = (G + NW - 1) / NW;
  const int h0 = wave * HPW;
  const bool alone = !p.cut && p.num_splits == 1;
  float val[HPW], mm[HPW], den[HPW];
#pragma unroll
  for (int j = 0; j < HPW; ++j) {
    const int h = min(h0 + j, G - 1);
    float mw[NW], m = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      mw[w] = ((const float*)(lds_all + w * kWave))[G * D + 2 * h];
      m = fmaxf(m, mw[w]);
    }
    float v = 0.f, l = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float* const rw = (const float*)(lds_all + w * kWave);
      const float a = NW == 1 ? 1.f : fast_exp2(mw[w] - m);   // 0 for a wavefront without a batch
      v = fmaf(a, rw[h * D + lane], v);
      l = fmaf(a, rw[G * D + 2 * h + 1], l);
    }
    val[j] = v; mm[j] = m; den[j] = l;
  }
  if (!alone) {
#pragma unroll
    for (int j = 0; j < HPW; ++j)
      if (h0 + j < G) {
        const int head = kvh * G + h0 + j;
        float* const dst = p.ws + (p.cut ? (int64_t)head * p.cut + slot
                                         : ((int64_t)b * p.n_q_heads + head) * p.num_splits + slot) * (D + 2);
        dst[2 + lane] = val[j];
        if (lane == 0) { dst[0] = mm[j]; dst[1] = den[j]; }
      }
    return;
  }
  if (NW > 1) __syncthreads(); else wave_sync();              // every record has been read: the regions are free
  if (h0 >= G) return;
  // normalise, rotate back once for V (App. A.4), write
  float* const fb = (float*)vbuf;
#pragma unroll
  for (int j = 0; j < HPW; ++j) fb[D * j + lane] = val[j] / den[j];
  wave_sync();
  float onorm = 1.0f;
  if (p.rot_v) {
    wave_lds_fwht128<(HPW + 1) / 2>(fb, p.had_block, lane);
    onorm = had_norm(p.had_block);
  }
#pragma unroll
  for (int j = 0; j < HPW; ++j)
    if (h0 + j < G) {
      float o = fb[D * j + lane] * onorm;
      if (p.rot_v && p.has_signs) o = apply_sign(p.signs, lane, o);          // (o~ H_blk) diag(sigma) = o~ R^T
      store_elem(p.out, p.out_dtype, ((int64_t)b * p.n_q_heads + kvh * G + h0 + j) * D + lane, o);
    }
}

template <int G>
static void launch_split64_g(const DecodeParams& p, int nw, dim3 grid, hipStream_t st) {
  if (nw >= 8) decode_int4_split64_kernel<G, 8><<<grid, dim3(512), 0, st>>>(p);
  else if (nw >= 2) decode_int4_split64_kernel<G, 4><<<grid, dim3(256), 0, st>>>(p);
  else decode_int4_split64_kernel<G, 1><<<grid, dim3(64), 0, st>>>(p);
}

int launch_decode_int4_split64(const DecodeParams& p, int G, int nw, dim3 grid, hipStream_t st) {
  switch (G) {
    case 1: launch_split64_g<1>(p, nw, grid, st); return SAW_OK;
    case 2: launch_split64_g<2>(p, nw, grid, st); return SAW_OK;
    case 4: launch_split64_g<4>(p, nw, grid, st); return SAW_OK;
    case 8: launch_split64_g<8>(p, nw, grid, st); return SAW_OK;
    default: return SAW_EINVAL;
  }
}

}  // namespace saw
