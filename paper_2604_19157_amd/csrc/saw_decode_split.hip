// INT4 paged decode attention, one 64-channel head at a time, on the gfx950 matrix cores: the head_dim 64 shapes
// whose heads the head-pair kernel cannot take two at a time (an odd number of kv heads, eight query heads per kv head).
// Paper: Sec. 2 (decode step), Sec. 4.1 / App. A.4 (rotated-space attention), App. A.1.
//
// A wavefront walks its share of one (sequence, kv head) in batches of four pages (64 tokens: 512 bytes of K and of
// V codes and 128 bytes of (scale, zero) pairs a page).  Everything is loaded into registers, two batches ahead:
//   * K codes: lane (token = lane % 16, k-group = lane / 16) loads the 16 codes it feeds to the logit product;
//   * V codes: 16 bytes per lane, two pages a load; written to LDS when their batch is due and read back by
//     ds_read_b64_tr_b4 (a 16x16 nibble transpose) with tokens along the contraction;
//   * the pairs: each lane loads those of one token; LDS hands them to the lanes that have its logits.
// With a fifth of the bytes of an LDS-DMA double buffer per wavefront in LDS, registers set the occupancy: three
// wavefronts per SIMD with two batches each in flight, which is what a 5 KiB batch needs to keep HBM busy.
//
// Numerics: both products are integer (v_mfma_i32_16x16x64_i8; saw_fixed.h).  The query and the weights p s are 31-bit
// fixed-point numbers, four signed byte digits each, and the codes are bytes as they are, so the products and their sums
// are exact; what is rounded is the query, to 2^-31 of its row's largest element, and each weight, to 2^-28 of the largest weight
// the wavefront had met of its head when it set the unit.
// What bounds it is the vector ALU, i.e. instructions: a nibble becomes a byte with 1.5 operations on eight of them where bf16 operands
// take seven, and the digits of a number need two operations, whatever their count.  Tile rows are 4 head + digit, so that a lane
// holds all four digits of a head's results and of one head only: no exchange between lanes in front of the softmax, one running
// state per tile.  (As bf16 products with three limbs: 370 vector-ALU and matrix instructions a batch of eight heads, now 245; 64 ragged
// sequences of 300 to 3000 tokens x 8 kv heads, 8 query heads each: kernel 28.4 -> 24.9 us, fused step 32.9 -> 30.4; error against
// 64 bits with fp32 outputs 7.2e-7 -> 4.4e-7.)
#include "saw_decode.h"
#include "saw_wave_util.h"
#include "saw_rank.h"
#include "saw_cut.h"
#include "saw_fixed.h"

namespace saw {

namespace split64 {

constexpr int D = 64;
constexpr int kTile = 512;                     // one (page, head) code tile: 16 tokens x 32 B

template <int G>
struct Lds {
  static constexpr int NT = (G > 4) ? 2 : 1;                 // row tiles of four heads
  static constexpr int kV = 4 * kTile;
  static constexpr int kP = NT * kDigitTile;
  static constexpr int kMeta = 1024;                         // a batch's pairs: K [page][token], then V
  static constexpr int kWave = kV + kP + kMeta;
};

struct Batch {                                 // one batch as loaded
  u32x2 k[4];                                  // channels 16 grp .. + 15 of token row16 of page q
  u32x4 v[2];                                  // chunk lane % 32 of pages 2 i and 2 i + 1
  f32x2 km, vm;                                // (scale, zero) of token row16 of page grp
};
}  // namespace split64

// NW wavefronts share a partition: wavefront w takes its batches w, w + NW, ...
// p.cut: block x is slot x of the batch cut by its own lengths (saw_cut.h); otherwise partition x of sequence z.
template <int G, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(3, 3)))
void decode_int4_split64_kernel(DecodeParams p) {
  using namespace split64;
  constexpr int NT = Lds<G>::NT;               // row tiles: lane group grp has head 4 t + grp of tile t
  constexpr int kWave = Lds<G>::kWave;
  const int kvh = blockIdx.y;
  const int lane = threadIdx.x & 63;
  const int wave = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row16 = lane & 15, grp = lane >> 4;
  __shared__ __attribute__((aligned(16))) uint8_t lds_all[NW * kWave];
  uint8_t* const vbuf = lds_all + wave * kWave;
  uint8_t* const pbuf = vbuf + Lds<G>::kV;
  uint8_t* const mbuf = pbuf + Lds<G>::kP;

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
  auto fetch = [&](int bi, Batch& r) __attribute__((always_inline)) {
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
    const int pid = grp == 0 ? id[0] : grp == 1 ? id[1] : grp == 2 ? id[2] : id[3];
    const int64_t m = (int64_t)pid * page_meta + head_meta + 2 * row16;
    r.km = __builtin_nontemporal_load((const f32x2*)(p.k_meta + m));
    r.vm = __builtin_nontemporal_load((const f32x2*)(p.v_meta + m));
  };
  const int mine = (nb > wave) ? (nb - wave + NW - 1) / NW : 0;         // this wavefront's batches
  Batch ra, rb;
  if (mine > 0) fetch(wave, ra);

  // ---- q~ = (q R) sm_scale log2(e) as A operands: digits of 31-bit fixed-point numbers, one exponent per row ----
  i32x4 a_q[NT];                               // 16 channels: even and odd ones of each eight in turn, as unpack_codes has them
  float qsum[NT], qunit[NT];                   // this lane's heads: sum over channels in the row's unit; the unit
  {
    float* const qs = (float*)vbuf;
#pragma unroll
    for (int g = 0; g < G; ++g) qs[D * g + lane] = qraw[g];
    if (G % 4 != 0) {                                         // rows of heads there are none of
#pragma unroll
      for (int i = 0; i < kDigitTile / 256; ++i) ((uint32_t*)pbuf)[lane + 64 * i] = 0u;
    }
    wave_sync();
    float qmul = p.q_scale;
    if (p.rot_k) {
      wave_lds_fwht128<(G + 1) / 2>(qs, p.had_block, lane);  // two 64-channel rows are one 128-channel vector (G = 1: half of one)
      qmul *= had_norm(p.had_block);
    }
    float* const units = (float*)mbuf;
    const int head = lane >> 3, ch8 = lane & 7;               // eight lanes a head, eight channels a lane
    if (G == 8 || head < G) {
      const f32x4 va = *(const f32x4*)(qs + D * head + 8 * ch8), vb = *(const f32x4*)(qs + D * head + 8 * ch8 + 4);
      const float x[8] = {va.x * qmul, va.y * qmul, va.z * qmul, va.w * qmul, vb.x * qmul, vb.y * qmul, vb.z * qmul, vb.w * qmul};
      float mx = 0.f;
#pragma unroll
      for (int k = 0; k < 8; ++k) mx = max_or_nan(mx, fabsf(x[k]));
      mx = max_or_nan(mx, dpp_f<0x141>(mx));                  // the eight lanes of the head: row_half_mirror,
      mx = max_or_nan(mx, dpp_f<0xB1>(mx));                   // quad_perm 1 0 3 2 and
      mx = max_or_nan(mx, dpp_f<0x4E>(mx));                   // 2 3 0 1
      const int e = fixed_exponent(mx);
      uint32_t even[4], odd[4];
      uint32_t u[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) u[k] = digit_bytes(nearest_int(__builtin_amdgcn_ldexpf(x[k], e)));
      transpose_digits(u[0], u[2], u[4], u[6], even);
      transpose_digits(u[1], u[3], u[5], u[7], odd);
#pragma unroll
      for (int l = 0; l < 4; ++l)
        *(u32x2*)(pbuf + (head >> 2) * kDigitTile + (4 * (head & 3) + l) * kDigitRow + 8 * ch8) = u32x2{even[l], odd[l]};
      if (ch8 == 0) units[head] = fixed_unit(mx, e);
    }
    wave_sync();
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      a_q[t] = *(const i32x4*)(pbuf + t * kDigitTile + row16 * kDigitRow + 16 * grp);
      qunit[t] = (G % 4 == 0 || grp < G) ? units[4 * t + grp] : 0.f;
      const i32x4 ones = i32x4{0x01010101, 0x01010101, 0x01010101, 0x01010101};
      qsum[t] = digits_value(mfma_i8(a_q[t], ones, i32x4{0, 0, 0, 0}));
    }
    wave_sync();
  }
  // ---- per-lane constants ----
  // V in LDS: 16-byte chunk Q of token t at chunk 2 t + (Q ^ (page & 1)) of the page's tile.  A lane group's transpose reads take
  // tokens 4 grp .. + 3 of all four pages, page innermost: lane 8 i + 2 page + j supplies token 4 grp + 2 i + j, so that contraction
  // step 16 grp + 4 r + page is token 4 grp + r, and the four weights of a lane of the softmax are four steps in a row.
  const int vw_off = kTile * (lane >> 5) + 16 * (((lane & 31) & ~1) + ((lane & 1) ^ (lane >> 5)));
  const int v_page = (row16 >> 1) & 3, v_tok = 4 * grp + 2 * (row16 >> 3) + (row16 & 1);
  const int vr_off = v_page * kTile + 32 * v_tok;
  const int vr_flip = 16 * (v_page & 1);
  uint8_t* const pw = pbuf + 4 * grp * kDigitRow + 4 * row16;  // digit l of this lane's head: row 4 grp + l
  const uint8_t* const pr = pbuf + row16 * kDigitRow + 16 * grp;

  // Running state: reference and unit (saw_fixed.h), sum of the p and of the w (z - 8) of this lane's tokens, and sum of the w (c - 8) as
  // 16 times that in digits, and what was moved out of the digits.
  i32x4 oacc[NT][4];
  float otop[NT][4], m_ref[NT], lsum[NT], zs[NT];
  int unit[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    m_ref[t] = -INFINITY; unit[t] = 0; lsum[t] = 0.f; zs[t] = 0.f;
#pragma unroll
    for (int c = 0; c < 4; ++c) { oacc[t][c] = i32x4{0, 0, 0, 0}; otop[t][c] = 0.f; }
  }
  int room = kFlushAfter;                      // (batches until the digits are moved out; all of them: nothing is in them yet)

  // (the second batch only here: requested with the first, 20 loads a wavefront filled the compute unit's memory pipeline in front of the
  // page ids and queries of wavefronts that had started later, which then ended last: 27.7 -> 26.3 us)
  if (mine > 1) fetch(wave + NW, rb);

  // ---- fused append: the step's new token ----
  // Rotated, quantised (Sec. 3 eqs. 1-3, App. A.1) and stored as the store kernel would; what attends to it
  // comes from LDS, nothing this launch writes to the cache is read back by it.  It opens the running state while the first batches
  // travel: as one more batch behind the last it made its wavefronts the last ones of the launch.
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
    // its one logit of each head (the same in every column of the tile), and its weight times its codes in fp32
    const u32x2 kc = *(const u32x2*)(cb + 8 * grp);
    const i32x4 kb = operand(code_bytes(kc.x), code_bytes(kc.y));
    float vc[4];                                              // channels 16 c + row16
#pragma unroll
    for (int c = 0; c < 4; ++c) vc[c] = (float)((cb[32 + 8 * c + (row16 >> 1)] >> (4 * (row16 & 1))) & 15) - 8.f;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const float lg = (meta[0].x * qunit[t]) * fmaf(-meta[0].y, qsum[t], digits_value(mfma_i8(a_q[t], kb, i32x4{0, 0, 0, 0})));
      m_ref[t] = fmaxf(ceilf(lg), kLeastLogit);
      const float pr = fast_exp2(lg - m_ref[t]), ps = pr * meta[1].x;
      unit[t] = unit_exponent(fabsf(ps));
      const float w = __builtin_amdgcn_ldexpf(ps, unit[t]);
      lsum[t] = row16 == 0 ? pr : 0.f;
      zs[t] = row16 == 0 ? w * (meta[1].y - 8.f) : 0.f;
#pragma unroll
      for (int c = 0; c < 4; ++c) otop[t][c] = 16.f * w * vc[c];
    }
    room = kFlushAfter - 1;                                   // (there is something to be scaled)
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
    wave_sync();                                              // (the first batch's codes and pairs take the place)
  }

  // One batch whose first token is position tok0; tokens from t_lim on are masked.  `next` requests the batch
  // that takes these registers next, as soon as they are consumed.
  auto body = [&](Batch& r, int tok0, int t_lim, auto&& next) __attribute__((always_inline)) {
    i32x4 dq[NT][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const i32x4 kb = operand(code_bytes(r.k[q].x), code_bytes(r.k[q].y));
#pragma unroll
      for (int t = 0; t < NT; ++t) dq[t][q] = mfma_i8(a_q[t], kb, i32x4{0, 0, 0, 0});
    }
    *(f32x2*)(mbuf + 8 * lane) = r.km;
    *(f32x2*)(mbuf + 512 + 8 * lane) = r.vm;
#pragma unroll
    for (int i = 0; i < 2; ++i) *(u32x4*)(vbuf + 2 * kTile * i + vw_off) = r.v[i];
    next(r);
    wave_sync();
    // ---- this lane's tokens are row16 of the four pages, its heads grp and 4 + grp ----
    f32x2 vm[4];
    float lg[NT][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x2 km = *(const f32x2*)(mbuf + 128 * q + 8 * row16);
      vm[q] = *(const f32x2*)(mbuf + 512 + 128 * q + 8 * row16);
#pragma unroll
      for (int t = 0; t < NT; ++t) lg[t][q] = (km.x * qunit[t]) * fmaf(-km.y, qsum[t], digits_value(dq[t][q]));
    }
    if (tok0 + 64 > t_lim) {                                  // wavefront-uniform
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool valid = tok0 + 16 * q + row16 < t_lim;
        vm[q] = valid ? vm[q] : f32x2{0.f, 0.f};
#pragma unroll
        for (int t = 0; t < NT; ++t) lg[t][q] = valid ? lg[t][q] : -INFINITY;
      }
    }
    float w[NT][4], pr_[NT][4], sum[NT], most = 0.f;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        pr_[t][q] = fast_exp2(lg[t][q] - m_ref[t]);           // exp2(-inf) = 0 for masked tokens
        w[t][q] = pr_[t][q] * __builtin_amdgcn_ldexpf(vm[q].x, unit[t]);
        most = max_or_nan(most, fabsf(w[t][q]));
      }
      sum[t] = (pr_[t][0] + pr_[t][1]) + (pr_[t][2] + pr_[t][3]);
      most = max_or_nan(most, sum[t]);
    }
    if (__any(!(most <= kWeightMost)) || room == 0) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        float alpha, beta;
        set_reference(lg[t], vm, room == kFlushAfter, false, m_ref[t], unit[t], pr_[t], w[t], alpha, beta);
        if (room != kFlushAfter) {
          lsum[t] *= alpha;
          zs[t] *= beta;
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            otop[t][c] = (otop[t][c] + long_digits_value(oacc[t][c])) * beta;
            oacc[t][c] = i32x4{0, 0, 0, 0};
          }
        }
        sum[t] = (pr_[t][0] + pr_[t][1]) + (pr_[t][2] + pr_[t][3]);
      }
      room = kFlushAfter;
    }
    --room;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      uint32_t u[4], d[4];
      float z = w[t][0] * (vm[0].y - 8.f);
#pragma unroll
      for (int q = 1; q < 4; ++q) z = fmaf(w[t][q], vm[q].y - 8.f, z);
      zs[t] += z;                                             // (one addition a batch to each running sum)
      lsum[t] += sum[t];
#pragma unroll
      for (int q = 0; q < 4; ++q) u[q] = digit_bytes(nearest_int(w[t][q]));
      transpose_digits(u[0], u[1], u[2], u[3], d);
#pragma unroll
      for (int l = 0; l < 4; ++l) *(uint32_t*)(pw + t * kDigitTile + l * kDigitRow) = d[l];
    }
    wave_sync();
    // ---- O[row][channel] += P (rows x 64 tokens) . V codes ----
    i32x4 pa[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) pa[t] = *(const i32x4*)(pr + t * kDigitTile);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const i32x2 tv = __builtin_amdgcn_ds_read_tr4_b64_v2i32((LDS_AS i32x2*)(vbuf + vr_off + ((16 * (c >> 1)) ^ vr_flip) + 8 * (c & 1)));
      const i32x4 vb = operand(centred_bytes((uint32_t)tv.x), centred_bytes((uint32_t)tv.y));
#pragma unroll
      for (int t = 0; t < NT; ++t) oacc[t][c] = mfma_i8(pa[t], vb, oacc[t][c]);
    }
    wave_sync();                                              // V, P and the pairs are rewritten by the next batch
  };
  for (int n = 0; n < mine; n += 2) {
    const int bi = wave + NW * n;
    body(ra, t_begin + 64 * bi, t_end, [&](Batch& r) { if (n + 2 < mine) fetch(bi + 2 * NW, r); });
    if (n + 1 < mine)
      body(rb, t_begin + 64 * (bi + NW), t_end, [&](Batch& r) { if (n + 3 < mine) fetch(bi + 3 * NW, r); });
  }

  const bool alone = !p.cut && p.num_splits == 1;
  const auto value = [&](int t, int c, float z) {              // channel 16 c + row16 of this lane's head, not normalised
    return __builtin_amdgcn_ldexpf(fmaf(otop[t][c] + long_digits_value(oacc[t][c]), 1.f / 16.f, -z), -unit[t]);
  };
  if (NW == 1 && !alone) {                                    // a record of its own, straight from the registers
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int head = 4 * t + grp;
      const float l = row_allsum(lsum[t]), z = row_allsum(zs[t]);
      if (G % 4 == 0 || head < G) {
        const int at = kvh * G + head;
        float* const dst = p.ws + (p.cut ? (int64_t)at * p.cut + slot : ((int64_t)b * p.n_q_heads + at) * p.num_splits + slot) * (D + 2);
#pragma unroll
        for (int c = 0; c < 4; ++c)
          dst[2 + 16 * c + row16] = value(t, c, z);
        if (row16 == 0) *(f32x2*)dst = f32x2{m_ref[t], l};
      }
    }
    return;
  }
  // ---- this wavefront's record in its own LDS: acc[G][64] un-normalised, then (max, sum) per head ----
  float* const rec = (float*)vbuf;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int head = 4 * t + grp;
    lsum[t] = row_allsum(lsum[t]);
    zs[t] = row_allsum(zs[t]);
    if (G % 4 == 0 || head < G) {
#pragma unroll
      for (int c = 0; c < 4; ++c)
        rec[head * D + 16 * c + row16] = value(t, c, zs[t]);
      if (row16 == 0) { rec[G * D + 2 * head] = m_ref[t]; rec[G * D + 2 * head + 1] = lsum[t]; }
    }
  }
  if (NW > 1) __syncthreads(); else wave_sync();

  // ---- combine the block's records, a few heads per wavefront ----
  constexpr int HPW = (G + NW - 1) / NW;
  const int h0 = wave * HPW;
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
