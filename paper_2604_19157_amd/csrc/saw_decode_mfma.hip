// INT4 paged decode attention for head_dim 128 on the gfx950 matrix cores.
// Paper: Sec. 2 (decode step), Sec. 4.1 / App. A.4 (rotated-space attention), App. A.1.
//
// A wavefront walks a range of one (sequence, kv head)'s tokens in batches of four pages (64
// tokens); which ranges a wavefront gets (a whole partition, every NW-th batch of one, or an even
// share of a long/short sequence pair) is described at the kernel.  Per batch:
//   * the four K and four V code tiles (1 KiB each, contiguous in HBM) and the tokens' (scale,
//     zero) pairs go straight from global memory into LDS (global_load_lds_dwordx4, no staging
//     registers): V and the metadata one batch ahead into double buffers, K into a single buffer
//     that is refilled as soon as its operand reads are done.  Each lane fetches the 16-byte chunk that belongs at its LDS
//     position under the swizzle pos(t, Q) = 4t + ((Q + t/4) & 3) (V: (Q + t/4 + page) & 3), which makes every later
//     LDS read bank-conflict free while a lane quad still reads one whole 64-byte row;
//   * logits: D[4 head + digit][token] = q~ . codes with v_mfma_i32_16x16x64_i8: q~ is a 31-bit fixed-point number, four signed
//     byte digits in neighbouring rows of the tile, and a nibble becomes a byte with 1.5 ALU operations on eight of them
//     (saw_fixed.h).  A lane's four results are the digits of one head and token: no exchange between lanes in front of the softmax;
//   * reference and unit of the running state only move (with a rescale of the accumulators) when a weight outgrows the digits, 2^4 above
//     the largest weight met when they were set;
//   * P.V needs tokens along the contraction: ds_read_b64_tr_b4 hands each lane 16 tokens of one channel (a 16x16 nibble
//     transpose inside LDS); the weights p s go through LDS once as digit rows; O[4 head + digit][channel] adds up exactly in 32-bit
//     integers.
// Integers because instructions in front of and between the transfers are what short and middle-sized calls wait for: as bf16 products
// with hi and lo limbs a batch of four query heads took 506 vector-ALU and matrix instructions, now 191 (eight heads 573, now 287).  Fused steps:
// 4 x 256 tokens 8.1 -> 6.9 us, 16 x 4096 22.4 -> 21.0, 48 ragged 32.6 -> 30.3, 256 ragged x 8 kv heads 121.5 -> 115.6, 64 ragged with a
// learned rotation 46.4 -> 41.9; one sequence of 131072 tokens with eight query heads 34.5 -> 33.5.  The error against 64 bits with fp32
// outputs fell from 2.4e-5 to 4e-7.
// Zero-points never enter the loops:  q~.k^ = s (q~.c - z sum q~),  sum_t w_t v^_t = sum_t w_t (c_t - 8) - sum_t w_t (z_t - 8),  w_t = p_t s_t.
// When one partition covers the sequence the kernel also normalises, rotates the output back and
// writes it (no merge launch), and it can append the step's new token itself (append_token).
#include "saw_decode.h"
#include "saw_wave_util.h"
#include "saw_rank.h"
#include "saw_cut.h"
#include "saw_fixed.h"

namespace saw {

constexpr int kTileBytes = 1024;               // one (page, head) code tile: 16 tokens x 64 B
template <int G> constexpr int kTiles = (G > 4) ? 2 : 1;        // row tiles of four heads
// Loads of a learned rotation's matrix at once (wave_lds_matvec128) for the query and the new token, and for the output: pair blocks of eight
// query heads are short of registers, and what they spill is reloaded behind transfers.  256 ragged sequences x 8 kv heads: 16, 16 and
// 16 loads 161 us, 8 each 150, 4 each with 8 for the token 143, 8 and 4 for the output 142.
template <int G, bool PAIR> constexpr int kLoads = (PAIR && G > 4) ? 8 : 16;
template <int G, bool PAIR> constexpr int kLoadsOut = (PAIR && G > 4) ? 4 : 16;
// Of a head pair with two row tiles a tile is one of the heads: it needs the 64 channels of that head only, one k-step of logits
template <int G, bool HP> constexpr int kSteps = (HP && G > 4) ? 1 : 2;
// ... and four column tiles of 16 output channels.  (Half the products: see the kernel.)
template <int G, bool HP> constexpr int kColumns = (HP && G > 4) ? 4 : 8;
template <int G, bool HP> using RangeState = FixedState<kTiles<G>, kColumns<G, HP>>;
constexpr int kQueryTile = 2048;               // digit rows of the query's four heads in LDS, 128 channels each: where their fp32 rows were
// (chunk of 16 channels: turned by the row, so that a column of chunks is spread over the banks)
__device__ __forceinline__ int query_at(int row, int chunk) { return 128 * row + 16 * (chunk ^ (row & 7)); }
// the P buffer: weights as digit rows, [tile][16 rows]; at the start of a range also one tile of the query's
template <int G> constexpr int kPbufBytes = (G > 4) ? kTiles<G> * kDigitTile : kQueryTile;

// Tile t of the query from the rows of q R (in LDS, 128 floats each), in two steps with a wave_sync between them, so that the digits may
// take the rows' place: lane (grp, row16) reads channels 8 row16 .. + 7 of head 4 t + grp and leaves their digits, even channels
// of each eight in front of the odd ones, as code_bytes has them.  Heads there are none of get rows of zeros.
struct QueryPart {
  float x[8];
};
template <int G>
__device__ __forceinline__ QueryPart q_part(const float* rows, int t, float qmul, int lane) {
  const int head = 4 * t + (lane >> 4);
  const float* const row = rows + 128 * min(head, G - 1) + 8 * (lane & 15);
  const f32x4 va = *(const f32x4*)row, vb = *(const f32x4*)(row + 4);
  const bool live = G % 4 == 0 || head < G;
  QueryPart r;
#pragma unroll
  for (int k = 0; k < 4; ++k) { r.x[k] = live ? va[k] * qmul : 0.f; r.x[4 + k] = live ? vb[k] * qmul : 0.f; }
  return r;
}
__device__ __forceinline__ void q_digits(const QueryPart& r, int lane, uint8_t* dig, float& unit) {
  float mx = 0.f;
#pragma unroll
  for (int k = 0; k < 8; ++k) mx = max_or_nan(mx, fabsf(r.x[k]));
  mx = max_or_nan(mx, dpp_f<0x121>(mx));                     // over the row of lanes: rotations by 1, 2, 4, 8
  mx = max_or_nan(mx, dpp_f<0x122>(mx));
  mx = max_or_nan(mx, dpp_f<0x124>(mx));
  mx = max_or_nan(mx, dpp_f<0x128>(mx));
  const int e = fixed_exponent(mx);
  uint32_t u[8], even[4], odd[4];
#pragma unroll
  for (int k = 0; k < 8; ++k) u[k] = digit_bytes(nearest_int(__builtin_amdgcn_ldexpf(r.x[k], e)));
  transpose_digits(u[0], u[2], u[4], u[6], even);
  transpose_digits(u[1], u[3], u[5], u[7], odd);
#pragma unroll
  for (int l = 0; l < 4; ++l)
    *(u32x2*)(dig + query_at(4 * (lane >> 4) + l, (lane & 15) >> 1) + 8 * (lane & 1)) = u32x2{even[l], odd[l]};
  unit = fixed_unit(mx, e);
}
// the A operands of tile t: k-step kk has channels 32 grp + 16 kk .. + 15, a single one 64 t + 16 grp .. + 15; and the sum over
// channels of this lane's head, in its unit
template <int KS>
__device__ __forceinline__ void q_operands(const uint8_t* dig, int t, int lane, i32x4 (&a_q)[KS], float& qsum) {
  i32x4 sum = i32x4{0, 0, 0, 0};
  const i32x4 ones = i32x4{0x01010101, 0x01010101, 0x01010101, 0x01010101};
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) {
    a_q[kk] = *(const i32x4*)(dig + query_at(lane & 15, KS == 2 ? 2 * (lane >> 4) + kk : 4 * t + (lane >> 4)));
    sum = mfma_i8(a_q[kk], ones, sum);
  }
  qsum = digits_value(sum);
}

// ---------------------------------------------------------------------------------------
// q~ = (q H_blk) sm_scale log2(e) for the G query heads of one kv head, in the lane layout of the
// logit MFMA's A operand, as digits of 31-bit fixed-point numbers with one unit per row (Sec. 4.1: the query is rotated once and
// consumed by the q.K loop).  qsum[t], qunit[t]: sum over channels and unit of this lane's head of tile t.
// `qraw` holds this lane's share of q (element lane + 64 j), loaded by the caller ahead of time;
// `qs` is LDS scratch of G*128 floats, `dig` of one tile's digits (up to G = 4 they take the rows' place).  These are
// __restrict__ parameters on purpose: that keeps
// these LDS accesses in an alias scope of their own, so the compiler does not make them wait for
// the LDS-DMA transfers the caller already has in flight into other buffers.
// HP (two 64-channel heads per row, see the kernel): `qraw[j]`, j < G, is channel `lane` of the j-th
// query head of the pair; its row gets the 64 values in the half of its own kv head and zeros in
// the other half, so that the 128-channel products below are the 64-channel ones.
// DN: a learned rotation R_l follows the Hadamard (App. A.3); a compile-time flag, so that the kernels
// of caches without one carry none of its code.
template <int G, bool HP, bool DN, int LOADS>
__device__ __forceinline__ void prepare_q(const DecodeParams& p, const float (&qraw)[2 * G], int lane, float* __restrict__ qs,
                                          uint8_t* __restrict__ dig, i32x4 (&a_q)[kTiles<G>][kSteps<G, HP>], float (&qsum)[kTiles<G>],
                                          float (&qunit)[kTiles<G>]) {
  constexpr int D = 128;
  if (HP) {
#pragma unroll
    for (int j = 0; j < G; ++j) {
      const int kv = j / (G / 2 > 0 ? G / 2 : 1);
      qs[j * D + 64 * kv + lane] = qraw[j];
      qs[j * D + 64 * (1 - kv) + lane] = 0.f;
    }
  } else {
    // a lane holds channels `lane` and `lane + 64` of every head: the butterflies of stride 64
    // (h = 128) are done here, in registers, and the LDS transform only goes up to order 64
    const bool top = p.rot_k && p.had_block > 64;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const float a = qraw[2 * g], b = qraw[2 * g + 1];
      qs[lane + 128 * g] = top ? a + b : a;
      qs[lane + 128 * g + 64] = top ? a - b : b;
    }
  }
  wave_sync();
  float qmul = p.q_scale;
  if (p.rot_k) {
    wave_lds_fwht128<G>(qs, min(p.had_block, 64), lane);
    qmul *= had_norm(p.had_block);
  }
  // learned rotation after the Hadamard (App. A.3: q^ = (q H_b) R_l)
  if constexpr (DN) {
    if (p.dense_k) wave_lds_matvec128<G, LOADS>(qs, p.dense, lane);
  }
  uint8_t* const d = (G > 4) ? dig : (uint8_t*)qs;
#pragma unroll
  for (int t = 0; t < kTiles<G>; ++t) {
    const QueryPart part = q_part<G>(qs, t, qmul, lane);
    wave_sync();
    q_digits(part, lane, d, qunit[t]);
    wave_sync();
    q_operands(d, t, lane, a_q[t], qsum[t]);
    wave_sync();
  }
}

constexpr int kMetaBytesOf(bool hp) { return hp ? 2048 : 1024; }   // one batch's (scale, zero) pairs: K, then V

// (what append_token leaves for append_store: four codes and the (scale, zero) pair of this lane's vector, its
// index in the pools, and whether its page is mapped)
struct NewToken {
  uint32_t codes;
  f32x2 meta;
  int64_t vec;
  bool place;
};
// The stores of the new token to the cache pools.  They are issued after the batch that attends to the
// token (which needs nothing from memory), so that no part of the step waits for them.
template <bool HP>
__device__ __forceinline__ void append_store(const DecodeParams& p, int lane, const NewToken& nt) {
  constexpr int DH = HP ? 64 : 128, LANES = DH / 4;          // lanes of a head
  if (!nt.place) return;
  uint8_t* const codes = const_cast<uint8_t*>(lane < 32 ? p.k_codes : p.v_codes);
  float* const meta = const_cast<float*>(lane < 32 ? p.k_meta : p.v_meta);
  *(uint16_t*)(codes + nt.vec * (DH / 2) + 2 * (lane & (LANES - 1))) = (uint16_t)nt.codes;
  if ((lane & (LANES - 1)) == 0) *(f32x2*)(meta + nt.vec * 2) = nt.meta;
}
// The rotation of the new token's K and V vectors by one wavefront, four channels per lane, K in the lower half (a block that prepares
// its range together has them from there); w: the channels as loaded; scr: LDS scratch of 256 floats (16-byte aligned).
template <bool HP, bool DN, int LOADS>
__device__ __forceinline__ void rotate_token(const DecodeParams& p, int lane, u32x2 w, float* __restrict__ scr, float (&x)[4]) {
  constexpr int DH = HP ? 64 : 128;
  const bool second = lane >= 32;
  const bool rot = second ? p.rot_v : p.rot_k;
  const bool dns[2] = {DN && p.dense_k != 0, DN && p.dense_v != 0};
  if (p.kv_new_dtype == SAW_BF16) { widen2<SAW_BF16>(w.x, x[0], x[1]); widen2<SAW_BF16>(w.y, x[2], x[3]); }
  else                            { widen2<SAW_F16>(w.x, x[0], x[1]);  widen2<SAW_F16>(w.y, x[2], x[3]); }
  if (p.has_signs) {                                         // x diag(sigma), as the store kernel does
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = rot ? apply_sign(p.signs, (4 * lane + e) & (DH - 1), x[e]) : x[e];
  }
  if (p.rot_k || p.rot_v || dns[0] || dns[1]) {
    *(f32x4*)(scr + 4 * lane) = f32x4{x[0], x[1], x[2], x[3]};             // [2][128]: K, V
    wave_sync();
    if (p.rot_k && p.rot_v) wave_lds_fwht128<2>(scr, p.had_block, lane);
    else if (p.rot_k) wave_lds_fwht128<1>(scr, p.had_block, lane);
    else if (p.rot_v) wave_lds_fwht128<1>(scr + 128, p.had_block, lane);
    if constexpr (DN) {                                      // k^ = (k H_b) R_l, the same for V (App. A.3)
      if (dns[0] && dns[1]) wave_lds_matvec128<2, LOADS>(scr, p.dense, lane);
      else if (dns[0]) wave_lds_matvec128<1, LOADS>(scr, p.dense, lane);
      else if (dns[1]) wave_lds_matvec128<1, LOADS>(scr + 128, p.dense, lane);
    }
    const f32x4 y = *(const f32x4*)(scr + 4 * lane);
    x[0] = y.x; x[1] = y.y; x[2] = y.z; x[3] = y.w;
    wave_sync();
  }
}
// The decode step's own token (fused append, Sec. 4.1's "new KV entries are rotated, quantised
// and written" folded into the attention launch): rotate and quantise the new K and V vectors of
// (sequence b, kv head kvh) for position L exactly as the store kernel would (Sec. 3 eqs. 1-3,
// App. A.1; append_store writes them to the pools), and place its codes and (scale, zero) pairs in LDS as token 0 of page 0 of a
// batch, in the layout the transfers produce; nothing this launch writes to the cache is read back by it.
// In pair blocks and single wavefronts the caller then runs one more batch in which only that token is valid, at the END of the range that
// starts the sequence, when every transfer of the range has landed and the buffers are idle: those launches fill the chip, every
// wavefront starts at once, bound by instructions, and in the middle of the loop, where wavefronts have no slack, it costs 1-2 us.  The
// rotation in front of it runs there too (rotate_token).  Blocks that share a range open the last wavefront's state with it
// instead (open_with_token); theirs is rotated with the query where they prepare it together (block_prepare).
// One wavefront, K in lanes 0-31 and V in lanes 32-63, four channels per lane: one chain of reductions and one division for both.
// (It is on the critical path of the range's last wavefront: with two channels of both vectors in every lane, 4 x 256 tokens took 8.6 us
// and take 8.1, 16 x 4096 22.6 and 22.1, 64 ragged with a learned rotation 46.3 and 45.0.)
//   pid, x  page id of position L and this lane's channels 4 (lane % 32) .. + 3, rotated
//   kdst, vdst, mdst  the K buffer, a V buffer and its metadata buffer
// HP: the 128 values are the new vectors of two neighbouring 64-channel kv heads (16 lanes each),
// quantised and stored per head; `kvh` counts pairs.
template <bool HP>
__device__ __forceinline__ void append_token(const DecodeParams& p, int kvh, int lane, int L, int pid, const float (&x)[4],
                                             uint8_t* __restrict__ kdst, uint8_t* __restrict__ vdst,
                                             uint8_t* __restrict__ mdst, NewToken& nt) {
  constexpr int DH = HP ? 64 : 128, LANES = DH / 4;
  const bool second = lane >= 32;
  nt.place = pid >= 0 && pid < p.num_pages;                  // otherwise attended to but not stored
  const int head = HP ? 2 * kvh + ((lane >> 4) & 1) : kvh;   // kv head of this lane's channels
  nt.vec = ((int64_t)pid * p.n_kv_heads + head) * 16 + (L & 15);
  // max and -min over the head's lanes, rows first (DPP)
  float mx = row_allmax(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])));
  float nmn = row_allmax(-fminf(fminf(x[0], x[1]), fminf(x[2], x[3])));
  if (!HP) {
    mx = max_xor16(mx);
    nmn = max_xor16(nmn);
  }
  const float norm = (second ? p.rot_v : p.rot_k) ? had_norm(p.had_block) : 1.0f;
  const float mn = -nmn;
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
  nt.codes = 0u;
#pragma unroll
  for (int e = 0; e < 4; ++e) nt.codes |= (uint32_t)__builtin_amdgcn_fmed3f(rintf(x[e] * inv) + zq, 0.0f, 15.0f) << (4 * e);
  nt.meta = f32x2{s_store, z_store};
  // token 0 of page 0 of the batch: its 64 code bytes are the first 64 bytes of the tile (chunk Q of
  // token 0 sits at chunk position Q), its pairs the first of the metadata block (head pair: one per head)
  *(uint16_t*)((second ? vdst : kdst) + 2 * (lane & 31)) = (uint16_t)nt.codes;
  if ((lane & (LANES - 1)) == 0) *(f32x2*)(mdst + (second ? kMetaBytesOf(HP) / 2 : 0) + (HP ? 128 * ((lane >> 4) & 1) : 0)) = nt.meta;
  wave_sync();
}

// Blocks of several wavefronts over one range (not pair blocks): the new token is quantised and opens the running state of the last
// wavefront, which has the fewest batches, while the first batch travels.  scr: 2 KiB of LDS that no transfer in flight targets.
// As one more batch behind the last it made the range longer by a microsecond (fused steps, at the end and here: 96 x 200 tokens x 8 kv
// heads 11.4 -> 10.2 us, 64 x 700 14.8 -> 13.7, 40 ragged 22.7 -> 21.6, 64 ragged 28.7 -> 27.6, one sequence of 300 7.2 -> 6.7).
template <int G, bool HP>
__device__ __forceinline__ void open_with_token(const DecodeParams& p, int kvh, int lane, int L, int pid, const float (&x)[4],
                                                uint8_t* __restrict__ scr, const i32x4 (&a_q)[kTiles<G>][kSteps<G, HP>],
                                                const float (&qsum)[kTiles<G>], const float (&qunit)[kTiles<G>], RangeState<G, HP> st,
                                                NewToken& nt) {
  constexpr int NT = kTiles<G>, NC = kColumns<G, HP>, KS = kSteps<G, HP>;
  constexpr int GK = HP ? G / 2 : G;
  const int row16 = lane & 15, grp = lane >> 4;
  uint8_t* const kdst = scr;                                 // token 0 of a page: 64 bytes; then its V codes and its pairs
  uint8_t* const vdst = scr + 64;
  uint8_t* const mdst = scr + 128;                           // [K, V][kv head]
  append_token<HP>(p, kvh, lane, L, pid, x, kdst, vdst, mdst, nt);
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const i32x4 none = i32x4{0, 0, 0, 0};
    i32x4 dq;
    if constexpr (KS == 2) {
      const u32x4 kw = *(const u32x4*)(kdst + 16 * grp);
      dq = mfma_i8(a_q[t][KS - 1], operand(code_bytes(kw.z), code_bytes(kw.w)), mfma_i8(a_q[t][0], operand(code_bytes(kw.x), code_bytes(kw.y)), none));
    } else {
      const u32x2 kw = *(const u32x2*)(kdst + 32 * t + 8 * grp);
      dq = mfma_i8(a_q[t][0], operand(code_bytes(kw.x), code_bytes(kw.y)), none);
    }
    const int kv = HP ? (NC == 4 ? t : min(grp, G - 1) / GK) : 0;
    const f32x2 km = *(const f32x2*)(mdst + 128 * kv), vm = *(const f32x2*)(mdst + kMetaBytesOf(HP) / 2 + 128 * kv);
    float code[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) code[c] = (float)((vdst[8 * (NC == 4 ? 4 * t + c : c) + (row16 >> 1)] >> (4 * (row16 & 1))) & 15) - 8.f;
    st.open(t, (km.x * qunit[t]) * fmaf(-km.y, qsum[t], digits_value(dq)), vm, code, row16 == 0);
  }
  wave_sync();                                               // (the second batch's transfers take the place)
}

// one batch's (scale, zero) pairs: K 4 pages x 128 B, then V (twice that for a pair of 64-channel heads)
template <bool HP> constexpr int kMetaBytes = HP ? 2048 : 1024;
// The P buffer is never a transfer target.  Up to G = 4 it also serves, at the start of a range, as the
// query preparation's scratch (the rotated query rows, at most 2 KB), so that this work touches no
// memory a transfer may be writing.
template <int G, bool HP> constexpr int kWaveLdsG = 12 * kTileBytes + kPbufBytes<G> + 2 * kMetaBytes<HP>;   // per wavefront: K buffer, two V buffers, P buffer, two metadata buffers

// The start of a range that NW wavefronts of a block share, where they prepare it together (kBlockPrep): every wavefront rotates its
// share of the G query rows and of the new token's K and V vectors, a learned rotation's product is the block's, and the A operands are
// converted once (four wavefronts a k-step each) and handed out.  When each wavefront of a block of eight prepared all of it for itself that
// was 1.6 us of instructions, two wavefronts a SIMD, in front of the first batch.  With a learned rotation the new token costs its
// rows in a product that runs anyway, instead of one wavefront's product at the end of the longest range.
// Blocks of two only do this with a learned rotation: theirs is hidden by the first transfers (16 x 4096 tokens).
// (fused steps, each wavefront for itself and then together: 4 x 256 tokens 8.9 -> 8.6 us, 64 ragged with a learned rotation 47.8 -> 46.3,
// of which the fixed order of the new token's sums took 0.6 back: block_columns_ordered.)
template <int NW, bool PAIR, bool HP, bool DN>
constexpr bool kBlockPrep = !PAIR && (NW == 8 || (NW == 4 && !HP) || (DN && NW > 1));
// LDS for it beside the wavefronts' buffers, which transfers may target: the query's rotated rows, whose place its digits take, the new
// token's from row kNewRow on, and the units
template <int G> constexpr int kNewRow = (G > 4) ? G : 4;
template <int G, int NW, bool PAIR, bool HP, bool DN>
constexpr int kPrepBytes = kBlockPrep<NW, PAIR, HP, DN> ? (kNewRow<G> + 2) * 512 + (NW >= 4 ? 16 * kTiles<G> : 0) : 0;

// This wavefront's vectors (wave, wave + NW, ...: below G a query row, then K, then V): elements `lane` and `lane + 64`, as loaded.
template <int G, int NW, bool HP>
__device__ __forceinline__ void block_vectors_load(const DecodeParams& p, int b, int kvh, bool with_new, int wave, int lane,
                                                   uint32_t (&bits)[(G + 1 + NW) / NW][2]) {
  constexpr int DH = HP ? 64 : 128;
#pragma unroll
  for (int u = 0; u < (G + 1 + NW) / NW; ++u) {
    const int v = wave + NW * u;                             // (wavefront-uniform)
    bits[u][0] = bits[u][1] = 0u;
    if (v < G) {
      const int64_t at = ((int64_t)b * p.n_q_heads + kvh * G + v) * DH + lane;
      if (p.q_dtype == SAW_F32) {
        bits[u][0] = ((const uint32_t*)p.q)[at];
        if (!HP) bits[u][1] = ((const uint32_t*)p.q)[at + 64];
      } else {
        bits[u][0] = ((const uint16_t*)p.q)[at];
        if (!HP) bits[u][1] = ((const uint16_t*)p.q)[at + 64];
      }
    } else if (v < G + 2 && with_new) {
      // (the block's new K|V values are 128 contiguous elements: one head, or a pair of 64-channel heads)
      const uint16_t* const src = (const uint16_t*)(v == G ? p.k_new : p.v_new) + (int64_t)b * p.n_kv_heads * DH + (int64_t)kvh * 128 + lane;
      bits[u][0] = src[0];
      bits[u][1] = src[64];
    }
  }
}
//   x, y  rows of 128 floats; x is where the vectors are rotated (without a learned rotation it is y), y holds the result; no
//         transfer in flight may target either, and y stays until the range ends
//   dig   in a block of two: one tile of digits of this wavefront's own
template <int G, int NW, bool HP, bool DN>
__device__ __forceinline__ void block_prepare(const DecodeParams& p, const uint32_t (&bits)[(G + 1 + NW) / NW][2], bool with_new, int wave,
                                              int lane, float* __restrict__ x, float* __restrict__ y, uint8_t* __restrict__ dig,
                                              const BlockColumns<DN ? NW : 8>& cols, i32x4 (&a_q)[kTiles<G>][kSteps<G, HP>],
                                              float (&qsum)[kTiles<G>], float (&qunit)[kTiles<G>]) {
  float* const in = DN ? x : y;
#pragma unroll
  for (int u = 0; u < (G + 1 + NW) / NW; ++u) {
    const int v = wave + NW * u;
    if (v < G || (v < G + 2 && with_new)) {
      const int dt = v < G ? p.q_dtype : p.kv_new_dtype;
      const bool rot = v == G + 1 ? p.rot_v : p.rot_k;
      float e[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        e[k] = dt == SAW_F32 ? __uint_as_float(bits[u][k]) : dt == SAW_BF16 ? __uint_as_float(bits[u][k] << 16)
                                                                             : f16_to_f32(bits[u][k] & 0xffffu);
        if (rot && p.has_signs) e[k] = apply_sign(p.signs, HP ? lane : lane + 64 * k, e[k]);      // x diag(sigma) first
      }
      // (head pair: a query row has its 64 values in the half of its own kv head and zeros in the other)
      const bool second = HP && v < G && v >= G / 2;
      float* const row = in + 128 * (v < G ? v : v - G + kNewRow<G>);
      row[lane] = second ? 0.f : e[0];
      row[64 + lane] = second ? e[0] : e[1];
      wave_sync();
      if (rot) wave_lds_fwht128<1>(row, p.had_block, lane);
    }
  }
  lds_barrier();
  if constexpr (DN) {                                        // learned rotation after the Hadamard (App. A.3)
    if (p.dense_k) {
      block_columns_product<G, NW>(in, y, cols, lane);
    } else {
      for (int i = 64 * wave + lane; i < 128 * G; i += 64 * NW) y[i] = in[i];
    }
    if (with_new) {
      constexpr int R = 128 * kNewRow<G>;
      if (p.dense_k && p.dense_v) {
        block_columns_ordered<2, NW>(in + R, y + R, cols, lane);
      } else {
        if (p.dense_k) block_columns_ordered<1, NW>(in + R, y + R, cols, lane);
        else if (wave < 2) y[R + 64 * wave + lane] = in[R + 64 * wave + lane];
        if (p.dense_v) block_columns_ordered<1, NW>(in + R + 128, y + R + 128, cols, lane);
        else if (wave < 2) y[R + 128 + 64 * wave + lane] = in[R + 128 + 64 * wave + lane];
      }
    }
    lds_barrier();
  }
  constexpr int NT = kTiles<G>;
  const float qmul = p.rot_k ? p.q_scale * had_norm(p.had_block) : p.q_scale;
  if constexpr (NW >= 4) {
    uint8_t* const d = (uint8_t*)y;
    float* const units = y + 128 * (kNewRow<G> + 2);
    if (wave < NT) {
      const QueryPart part = q_part<G>(y, wave, qmul, lane);
      wave_sync();
      float unit;
      q_digits(part, lane, d + wave * kQueryTile, unit);
      if ((lane & 15) == 0) units[4 * wave + (lane >> 4)] = unit;
    }
    lds_barrier();
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      q_operands(d + t * kQueryTile, t, lane, a_q[t], qsum[t]);
      qunit[t] = units[4 * t + (lane >> 4)];
    }
  } else {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      q_digits(q_part<G>(y, t, qmul, lane), lane, dig, qunit[t]);
      wave_sync();
      q_operands(dig, t, lane, a_q[t], qsum[t]);
      wave_sync();
    }
  }
  wave_sync();
}

// The end of a range that NW wavefronts of a block shared: their running (max, sum, accumulator) states become the partition's
// record, or the sequence's output.  Every wavefront leaves its state in its own buffers; after one barrier a wavefront takes G / NW
// heads (some wavefronts none, if there are more of them) and works them out from all states with two channels per lane: weights,
// sums, normalising, the way back through the rotation and the store.  What this costs is instructions of the last
// wavefront to arrive, one every 4-5 cycles: as a fold of accumulator tiles by all, then the rest by wavefront 0, it took 2.5 us from
// the last batch to the end of the kernel for a record (16 sequences of 4096 tokens) and 3.2 us for an output (4 of 256); now 1.7 and
// 2.1.  Whole calls: 4 x 256 tokens 10.8 -> 9.3 us, 16 x 4096 23.7 -> 22.6, 48 ragged 34.2 -> 33.1, 1 x 131072 37.3 -> 35.3, 64 ragged
// with a learned rotation 50.1 -> 47.9.
template <int G, int NW, bool HP, bool DN, bool CUT>
__device__ __forceinline__ void block_epilogue(const DecodeParams& p, uint8_t* const lds_all, int wave, int lane, int b, int kvh,
                                               int split, RangeState<G, HP> st) {
  constexpr int DH = HP ? 64 : 128;
  constexpr int GK = HP ? G / 2 : G;
  constexpr int NT = kTiles<G>, NC = kColumns<G, HP>;
  constexpr int kWaveLds = kWaveLdsG<G, HP>;
  constexpr int SP = 128 + 16;                                // pitch of a head's channels: the four heads of a write differ in their banks
  constexpr int kM = G * SP;                                  // then (maximum, sum) of each head
  constexpr int HPW = (G + NW - 1) / NW;                      // heads of a wavefront
  constexpr int kScr = 12 * kTileBytes;                       // (the P and metadata buffers: no state reaches them)
  static_assert((kM + 2 * G) * 4 <= kScr, "a state fits in front of the P buffer");
  static_assert(HPW * 512 <= kPbufBytes<G> + 2 * kMetaBytesOf(HP) && G * 512 <= kPbufBytes<G> + 2 * kMetaBytesOf(HP), "the heads' rows fit behind it");
  const int row16 = lane & 15, grp = lane >> 4;
  const bool alone = !CUT && p.num_splits == 1;
  BlockColumns<DN ? NW : 8> cols;                             // (requested now: the exchange of the states hides the trip to L2)
  if constexpr (DN) {
    if (alone && p.dense_v) block_columns_load<NW>(p.dense + kDenseD * kDenseD, wave, lane, cols);
  }
  st.sum_lanes();
  {
    float* const own = (float*)(lds_all + wave * kWaveLds);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int head = 4 * t + grp;
      if (G % 4 == 0 || head < G) {
#pragma unroll
        for (int c = 0; c < NC; ++c) own[head * SP + 16 * (NC == 8 ? c : 4 * t + c) + row16] = st.value(t, c);
        if (row16 == 0) *(f32x2*)(own + kM + 2 * head) = f32x2{st.m_ref[t], st.lsum[t]};
      }
    }
  }
  __syncthreads();
  const int h0 = wave * HPW;
  if (h0 >= G && !(DN && alone)) return;                      // (wavefronts without a head help with the learned rotation)
  float* const scr = (float*)(lds_all + wave * kWaveLds + kScr);
  float o0[HPW], o1[HPW];
#pragma unroll
  for (int j = 0; j < HPW; ++j) {
    const int h = min(h0 + j, G - 1);
    float a[NW], ls[NW], mm = -INFINITY;                      // (some wavefront has a batch or the new token: the maximum is finite)
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const f32x2 ml = *(const f32x2*)((const float*)(lds_all + w * kWaveLds) + kM + 2 * h);
      a[w] = ml.x;
      ls[w] = ml.y;
      mm = fmaxf(mm, a[w]);
    }
    float l = 0.f, v0 = 0.f, v1 = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float* const so = (const float*)(lds_all + w * kWaveLds) + h * SP + lane;
      const float aw = fast_exp2(a[w] - mm);                  // 0 for a wavefront that had no batch
      l = fmaf(aw, ls[w], l);
      v0 = fmaf(aw, so[0], v0);
      v1 = fmaf(aw, so[64], v1);
    }
    if (!alone) {
      // one of several partitions: (max, sum, un-normalised accumulator) for the merge kernel
      if (h0 + j < G) {
        const int head = kvh * G + h;
        float* const dst = p.ws + (CUT ? (int64_t)head * p.cut + split : ((int64_t)b * p.n_q_heads + head) * p.num_splits + split) * (DH + 2);
        if (HP) {
          dst[2 + lane] = (h / GK) ? v1 : v0;                 // the half of the row that is this head's
        } else {
          dst[2 + lane] = v0;
          dst[2 + 64 + lane] = v1;
        }
        if (lane == 0) { dst[0] = mm; dst[1] = l; }
      }
    } else {
      const float inv = __builtin_amdgcn_rcpf(l);
      o0[j] = v0 * inv;
      o1[j] = v1 * inv;
    }
  }
  if (!alone) return;
  // rotate back once for V (App. A.4; a learned rotation's transpose first, App. A.3), write the output
  float* rows = scr;
  if constexpr (DN) {
    if (p.dense_v) {
      float* const x = (float*)(lds_all + kScr);
      float* const y = (float*)(lds_all + kWaveLds + kScr);
#pragma unroll
      for (int j = 0; j < HPW; ++j)
        if (h0 + j < G) {
          x[128 * (h0 + j) + lane] = o0[j];
          x[128 * (h0 + j) + 64 + lane] = o1[j];
        }
      __syncthreads();
      block_columns_product<G, NW>(x, y, cols, lane);
      __syncthreads();
      rows = y + 128 * h0;
    }
  }
  if (h0 >= G) return;
  if (!DN || !p.dense_v) {
#pragma unroll
    for (int j = 0; j < HPW; ++j) {
      rows[128 * j + lane] = o0[j];
      rows[128 * j + 64 + lane] = o1[j];
    }
  }
  wave_sync();
  float onorm = 1.0f;
  if (p.rot_v) {
    wave_lds_fwht128<HPW>(rows, p.had_block, lane);
    onorm = had_norm(p.had_block);
  }
#pragma unroll
  for (int j = 0; j < HPW; ++j) {
    const int h = h0 + j;
    if (h >= G) break;                                        // (wavefront-uniform)
    // two consecutive channels per lane: a whole row per store (head pair: the 32 lanes of the head's own half)
    if (HP && (lane >> 5) != h / GK) continue;
    const f32x2 o2 = *(const f32x2*)(rows + 128 * j + 2 * lane);
    const int c = (2 * lane) & (DH - 1);
    float o[2] = {o2.x * onorm, o2.y * onorm};
    if (p.rot_v && p.has_signs) {                             // (o~ H_blk) diag(sigma) = o~ R^T
      o[0] = apply_sign(p.signs, c, o[0]);
      o[1] = apply_sign(p.signs, c + 1, o[1]);
    }
    const int64_t at = ((int64_t)b * p.n_q_heads + kvh * G + h) * DH + c;
    if (p.out_dtype == SAW_F32)
      *(f32x2*)((float*)p.out + at) = f32x2{o[0], o[1]};
    else
      *(uint32_t*)((uint16_t*)p.out + at) = p.out_dtype == SAW_BF16 ? f32_to_bf16(o[0]) | ((uint32_t)f32_to_bf16(o[1]) << 16)
                                                                   : f32_to_f16(o[0]) | ((uint32_t)f32_to_f16(o[1]) << 16);
  }
}

// Two ways of giving wavefronts their work.
//
// PAIR = false: NW wavefronts share one (sequence, kv head, partition): wavefront w takes batches
// w, w + NW, ... and the block folds their running (max, sum, accumulator) states together in LDS
// at the end (block_epilogue); with several partitions the result goes to the workspace for the merge kernel.
//
// PAIR = true (one partition per sequence, batch too large for every wavefront to need help):
// a block of NW = 2 or 4 wavefronts owns the sequences at ranks r and B-1-r of the longest-first
// order and splits their batches, laid end to end (long, then short), into NW equal shares: a
// wavefront gets a stretch of the long sequence, of the short one, or - one wavefront per block
// at most - the end of the long one and the start of the short one.  A sequence that one
// wavefront covers alone is finished by it; otherwise each wavefront leaves its share as a
// (max, sum, accumulator) record in LDS and counts itself in with an LDS atomic, and whichever
// comes last combines the records (always in wavefront order) and writes the output, so nobody
// waits for anybody.  The wavefront with two stretches takes the short sequence's first, so the
// record it leaves in its own buffers is its last act; the short sequence's record, if that one
// is shared too (NW = 4 only), goes to a spare slot of the block.  Every wavefront of the launch
// then streams the same number of tokens (give or take a batch) however ragged the batch is,
// with no partial results in global memory.  NW = 4 keeps the chip's 2048 wavefront slots busy
// when there are only 512 to 1024 (sequence, kv head) items.
enum SegMode : int { kSegSplitKV = 0, kSegAlone = 1, kSegShare = 2 };

//
// HP = true ("head pair") serves head_dim 64 with an even number of kv heads: the block's kv "head" is
// a pair of neighbouring 64-channel heads, whose code tiles ([head][token][32 B]) and metadata are
// contiguous in a page.  The transfers re-order a pair's tiles into rows of 128 channels (head 2j's
// 64, then head 2j+1's), the G query rows (G/2 per kv head) carry zeros in the other head's half,
// and everything between the transfers and the epilogue runs exactly as for head_dim 128; only the
// (scale, zero) pairs are per (token, kv head), and a row's own 64 output channels are kept.
// PK (pair mode): sequences per block, 2 (ranks r and B-1-r) or 3 (ranks r, 2n-1-r and 2n+r with
// n = ceil(B/3): the first two add up alike, the third makes the totals differ by up to a third of
// the spread of the lengths).  Four wavefronts over three sequences put 4/3 wavefronts on a (sequence,
// kv head) item, which fills the chip when there are 1025 to 1536 items - too many for four
// wavefronts per pair, and with two per pair a quarter to a half of the slots would stay empty.
// CUT: the batch is cut by its own lengths (saw_cut.h), a block of NW wavefronts per slot; a kernel of its own because the code
// in front of the first page-id load costs the other modes 2 % even where it is not taken.
template <int G, int NW, bool PAIR, bool HP = false, int PK = 2, bool DN = false, bool CUT = false>
// (a launch of this kernel puts at most 8 wavefronts on a compute unit, 2 per SIMD: let the
// register allocator use the 256 registers that leaves each of them)
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 2)))
void decode_int4_mfma_kernel(DecodeParams p) {
  static_assert(!PAIR || NW == 2 || NW == 4, "a pair block has two or four wavefronts");
  static_assert(!HP || G >= 2, "a head pair has at least one query head per kv head");
  static_assert(!(PAIR && CUT), "pair blocks deal out whole sequences");
  static_assert(!(HP && DN), "the learned rotation is built for head_dim 128");
  constexpr int D = 128;                       // channels of a row (a head, or a pair of 64-channel heads)
  constexpr int DH = HP ? 64 : 128;            // channels of one head
  constexpr int GK = HP ? G / 2 : G;           // query heads per kv head
  constexpr int NT = kTiles<G>;                // row tiles: lane group grp has head 4 t + grp of tile t
  constexpr int NC = kColumns<G, HP>, KS = kSteps<G, HP>;
  constexpr int NM = (HP && NT == 2) ? 2 : 1;  // kv heads whose pairs a lane needs: its tiles' (head pair), else one
  constexpr int STEP = PAIR ? 1 : NW;          // batch stride of a wavefront inside its range
  // (which partition a block takes is rotated by its kv head and sequence: blocks go to the XCDs round
  // robin in launch order, and with the partition index as the fastest grid index and a partition count
  // that shares a factor with 8 every XCD would serve a fixed set of partition indices - of a ragged
  // batch the later partitions are mostly empty, so some XCDs got most of the work: 33 sequences x 8
  // partitions 41 us against 28-32 us with 7 or 9 partitions)
  // (a batch cut by its own lengths has one block per slot: see saw_cut.h)
  const int split = CUT ? (int)blockIdx.x : (int)((blockIdx.x + blockIdx.y + blockIdx.z) % gridDim.x);
  const int kvh = blockIdx.y;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int first_batch = PAIR ? 0 : wave;     // first batch of this wavefront inside its range

  constexpr int kWaveLds = kWaveLdsG<G, HP>;
  // One shared array for everything, the pair counter included: with a single LDS object the
  // compiler keeps the restrict scopes of the helpers' pointer arguments, which is what lets their LDS
  // accesses proceed while transfers are in flight (with two objects it replaces those scopes by
  // per-object ones and then orders every LDS access behind every transfer).
  constexpr int kRecFloats = G * 128 + 2 * G;                   // a record: accumulator rows, then (max, sum) per row
  constexpr int K = PAIR ? PK : 1;                              // sequences of a pair-mode block
  static_assert(PK == 2 || PK == 3, "a block takes two or three sequences");
  // (a wavefront can hold the head of a shared sequence and, after it, an earlier sequence of the block
  // only when the block has more than two wavefronts or more than two sequences: then that record
  // needs a slot outside the wavefront's own buffers)
  constexpr bool kSpare = PAIR && (NW > 2 || K > 2);
  constexpr int kSpareBytes = kSpare ? (K - 1) * kRecFloats * 4 : 0;
  constexpr bool kBP = kBlockPrep<NW, PAIR, HP, DN>;
  __shared__ __attribute__((aligned(16))) uint8_t lds_all[NW * kWaveLds + 16 + kSpareBytes + kPrepBytes<G, NW, PAIR, HP, DN>];
  uint8_t* const kbuf = lds_all + wave * kWaveLds;
  uint8_t* const vbuf_a = kbuf + 4 * kTileBytes;
  uint8_t* const vbuf_b = kbuf + 8 * kTileBytes;
  uint8_t* const pbuf = kbuf + 12 * kTileBytes;
  uint8_t* const mbuf_a = pbuf + kPbufBytes<G>;   // metadata of the batch in vbuf_a / vbuf_b
  uint8_t* const mbuf_b = mbuf_a + kMetaBytes<HP>;
  int* const done_cnt = (int*)(lds_all + NW * kWaveLds);        // PAIR: records left so far of the block's sequences [k]
  float* const spare_rec = (float*)(lds_all + NW * kWaveLds + 16);   // PAIR, NW = 4: spare record of sequence k >= 1 at (k - 1) * kRecFloats

  // ---- the ranges this wavefront streams: (sequence, first token, end token, what to do with the result) ----
  int nseg = 1;
  // (a wavefront has at most one range per sequence of its block; the arrays are read with
  // select chains, never indexed at run time)
  constexpr int MS = (K > 2) ? K : 2;
  int sg_t0[MS], sg_t1[MS], sg_mode[MS], sg_seq[MS];   // per range: tokens, mode, which of the block's sequences
  int bk[MS], lk[MS];                                   // per sequence of the block: index in the batch, cached tokens
#pragma unroll
  for (int i = 0; i < MS; ++i) { sg_t0[i] = 0; sg_t1[i] = 0; sg_mode[i] = kSegAlone; sg_seq[i] = 0; bk[i] = 0; lk[i] = 0; }
  bk[0] = (int)blockIdx.z; sg_t0[0] = split * p.chunk_tokens; sg_mode[0] = kSegSplitKV;
  uint32_t part_mask[MS];                      // PAIR: wavefronts with a share of sequence k of the block
#pragma unroll
  for (int i = 0; i < MS; ++i) part_mask[i] = 0u;
  bool cut_new = false;                        // a batch cut by its lengths: this block takes the sequence's new token
  if (PAIR) {
    const int B = p.batch;
    if (threadIdx.x < 4) done_cnt[threadIdx.x] = 0;
    __syncthreads();                                    // nothing in flight yet: a plain barrier is fine here
    // the block's sequences by length rank, longest first; rank >= B: no such sequence
    int rk[K], nbk[K], stk[K];
    bool present[K];
    if (K == 2) {
      rk[0] = blockIdx.z; rk[1] = B - 1 - rk[0];
      present[0] = true; present[1] = rk[1] != rk[0];   // odd batch: the middle sequence is alone
    } else {
      const int n3 = (B + 2) / 3;
      rk[0] = blockIdx.z; rk[1] = 2 * n3 - 1 - rk[0]; rk[K - 1] = 2 * n3 + rk[0];
      present[0] = true; present[1] = rk[1] < B; present[K - 1] = rk[K - 1] < B;
    }
    if (p.order) {
      // the caller supplied the longest-first order: two dependent loads per sequence instead of the ranking
      int oi[K], raw[K];
#pragma unroll
      for (int k = 0; k < K; ++k) oi[k] = present[k] ? p.order[rk[k]] : 0;
#pragma unroll
      for (int k = 0; k < K; ++k) bk[k] = min(max(oi[k], 0), B - 1);
#pragma unroll
      for (int k = 0; k < K; ++k) raw[k] = present[k] ? p.seq_lens[bk[k]] : 0;
#pragma unroll
      for (int k = 0; k < K; ++k) lk[k] = present[k] ? max(min(raw[k], p.bound), 0) : 0;
    } else {
      const LenClasses lc = build_len_classes(p, B, lane, (int*)kbuf);
#pragma unroll
      for (int k = 0; k < K; ++k) {
        bk[k] = present[k] ? seq_of_rank(lane, lc, rk[k]) : 0;
        lk[k] = present[k] ? lc.lens[bk[k]] : 0;
      }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) nbk[k] = (lk[k] + 63) >> 6;
    // Shares of the sequences' batches laid end to end: wavefront w takes [T w / NW, T (w+1) / NW).
    // A wavefront that gets the end of one sequence and the start of the next pays another
    // prologue, about the time of two or three batches: that cost sits in front of every sequence
    // but the first as kGap batches nobody streams (stk[k] is where sequence k starts; 2 and 3
    // measured 1-2 % better than their neighbours for blocks of two and of four).
    constexpr int kGap = (NW > 2) ? 3 : 2;
    int T = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      stk[k] = T + ((k > 0 && nbk[k] > 0) ? kGap : 0);
      T = stk[k] + nbk[k];
    }
#pragma unroll
    for (int w = 0; w < NW; ++w) {       // (T < 2^27 batches: the products fit 32 bits)
      const int lo_w = (int)(((uint32_t)T * (uint32_t)w) / NW), hi_w = (int)(((uint32_t)T * (uint32_t)(w + 1)) / NW);
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (max(lo_w, stk[k]) < min(hi_w, stk[k] + nbk[k])) part_mask[k] |= 1u << w;
    }
    const int lo = (int)(((uint32_t)T * (uint32_t)wave) / NW), hi = (int)(((uint32_t)T * (uint32_t)(wave + 1)) / NW);
    nseg = 0;
    // Last sequence first: what a wavefront streams last is then the sequence it shares with the
    // wavefronts before it, whose record can stay in its own buffers.  A sequence without cached
    // tokens has no share: its zero row - or, with a fused append, an empty range that still
    // attends to the new token - goes to the last wavefront (the first, for the block's longest).
#pragma unroll
    for (int k = K - 1; k >= 0; --k) {
      const int p0 = max(lo, stk[k]), p1 = min(hi, stk[k] + nbk[k]);
      bool add = false;
      int t0 = 0, t1 = 0, mode_k = kSegAlone;
      if (p0 < p1) {
        add = true;
        t0 = 64 * (p0 - stk[k]); t1 = min(lk[k], 64 * (p1 - stk[k]));
        mode_k = __popc(part_mask[k]) > 1 ? kSegShare : kSegAlone;
      } else if (present[k] && nbk[k] == 0 && wave == (k == 0 ? 0 : NW - 1)) {
        if (p.append) {
          add = true;
        } else {
          for (int i = lane; i < G * DH; i += 64)
            store_elem(p.out, p.out_dtype, ((int64_t)bk[k] * p.n_q_heads + kvh * G) * DH + i, 0.f);
        }
      }
      if (add) {
#pragma unroll
        for (int i = 0; i < MS; ++i)
          if (i == nseg) { sg_t0[i] = t0; sg_t1[i] = t1; sg_mode[i] = mode_k; sg_seq[i] = k; }
        ++nseg;
      }
    }
    wave_sync();                                        // the ranking's scratch lived in kbuf (and on into vbuf_a)
  } else if (CUT) {
    const BatchCut cut = cut_batch(p, lane);
    int b, len, part, parts, first, end;
    cut_slot(cut, split, b, len, part, parts);
    if (b < 0) return;                                  // block-uniform
    if (part == 0 && kvh == 0 && threadIdx.x == 0) p.cut_of[b] = make_int2(split, parts);
    cut_range((len + 63) >> 6, part, parts, first, end);
    bk[0] = b; lk[0] = len;
    sg_t0[0] = 64 * first; sg_t1[0] = min(len, 64 * end);
    cut_new = part == parts - 1;                        // (the last partition is one with the fewest batches)
  } else if (p.sorted) {
    // one block per (sequence, kv head), more blocks than fit the chip at once: blocks are dispatched
    // in index order as earlier ones finish, so taking the sequences longest first leaves the
    // shortest for the end of the launch
    if (p.order) {
      bk[0] = min(max(p.order[blockIdx.z], 0), p.batch - 1);
    } else {
      const LenClasses lc = build_len_classes(p, p.batch, lane, (int*)kbuf);
      bk[0] = seq_of_rank(lane, lc, blockIdx.z);
    }
    wave_sync();
  }

  // The bookkeeping above is wavefront-uniform, but it is read once per range only: parked in vector
  // registers on purpose (the set-up code is short of scalar ones) and brought back when needed.
#pragma unroll
  for (int i = 0; i < MS; ++i) {
    asm volatile("" : "+v"(sg_t0[i]), "+v"(sg_t1[i]), "+v"(sg_mode[i]), "+v"(sg_seq[i]));
    asm volatile("" : "+v"(bk[i]), "+v"(lk[i]), "+v"(part_mask[i]));
  }
  const int row16 = lane & 15, grp = lane >> 4;
  const int64_t head_tile = (int64_t)kvh * kTileBytes;
  const int64_t page_stride = (int64_t)p.n_kv_heads * (HP ? kTileBytes / 2 : kTileBytes);
  const int64_t head_meta = (int64_t)kvh * (HP ? 64 : 32);        // floats
  const int64_t page_meta = (int64_t)p.n_kv_heads * 32;
  // lane l fills LDS chunk l of a tile = token t = l/4, stored quarter (l & 3) = (Q + t/4) & 3;
  // quarter Q of a row is 16 source bytes: of the token's 64 (head_dim 128), or half Q & 1 of the
  // token's 32 in head Q >> 1 of the pair, whose tiles follow each other
  const int q_src = ((lane & 3) - (lane >> 4)) & 3;
  const auto source = [&](int quarter) { return HP ? 512 * (quarter >> 1) + 32 * (lane >> 2) + 16 * (quarter & 1) : 64 * (lane >> 2) + 16 * quarter; };
  const int g_swz = source(q_src);
  // V tiles are turned further by their page of the batch: stored quarter s of a row is quarter (s - t/4 - page) & 3, so that the
  // transpose reads, which take the same tokens of all four pages at once, touch every bank once
  int g_swz_v[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) g_swz_v[q] = source((q_src - q) & 3);
  // ---- per-lane constants ----
  const int kr_off = 16 * (4 * row16 + ((grp + (row16 >> 2)) & 3));                 // K read: t = row16, Q = grp
  // (one k-step a head: quarter 2 head + grp / 2 of token row16, half grp % 2 of its 16 bytes)
  const int kr_pair[2] = {16 * (4 * row16 + (((grp >> 1) + (row16 >> 2)) & 3)) + 8 * (grp & 1),
                          16 * (4 * row16 + ((2 + (grp >> 1) + (row16 >> 2)) & 3)) + 8 * (grp & 1)};
  // V transpose reads: a lane group takes tokens 4 grp .. + 3 of all four pages, page innermost: lane 8 i + 2 page + j supplies
  // token 4 grp + 2 i + j, so that contraction step 16 grp + 4 r + page is token 4 grp + r, and the four weights of a lane of the
  // softmax (token row16 of the four pages) are four steps in a row
  const int v_page = (row16 >> 1) & 3, v_tok = 4 * grp + 2 * (row16 >> 3) + (row16 & 1);
  int vr_off[4];                                                                     // channels 32 i .. + 15; the next 16 are 8 bytes on
#pragma unroll
  for (int i = 0; i < 4; ++i) vr_off[i] = v_page * kTileBytes + 16 * (4 * v_tok + ((i + grp + v_page) & 3));
  const int kv_of = HP ? min(grp, G - 1) / GK : 0;                                   // head pair, one tile: which of the two heads' pairs
  const int pw_off = 4 * grp * kDigitRow + 4 * row16;                                // digit l of this lane's head: row 4 grp + l
  const uint32_t pa_addr = (uint32_t)(uintptr_t)(LDS_AS uint8_t*)pbuf + row16 * kDigitRow + 16 * grp;   // LDS byte address

#pragma unroll 1
  for (int seg = 0; seg < nseg; ++seg) {
#define SAW_SEG(a) (seg == 0 ? a[0] : (seg == 1 || MS == 2) ? a[1] : a[MS - 1])
#define SAW_SEQ(a) (sq == 0 ? a[0] : (sq == 1 || MS == 2) ? a[1] : a[MS - 1])
  const int sq = __builtin_amdgcn_readfirstlane(SAW_SEG(sg_seq));
  const int b = __builtin_amdgcn_readfirstlane(SAW_SEQ(bk));
  const int t_begin = __builtin_amdgcn_readfirstlane(SAW_SEG(sg_t0));
  const int mode = __builtin_amdgcn_readfirstlane(SAW_SEG(sg_mode));
  const int64_t pt_row = (int64_t)b * p.max_pages;
  // Page ids: lane l of `pidv` holds the (clamped) physical page of logical page
  // pg_first + 64*window + l, i.e. one vector load covers a window of 16 batches; `pidv_nx` is
  // the following window, loaded a window ahead.  A batch takes its four ids with v_readlane, so
  // no page-table latency sits between consecutive batches.  The first load does not wait for
  // the sequence length: entries past the sequence's last page are read (inside the row) and
  // clamped to a valid page, and the tokens they stand for are masked out below.
  const int pg_first = t_begin >> 4;
#define SAW_LOAD_PIDS(dst, first) dst = p.page_table[pt_row + min((first) + lane, p.max_pages - 1)];
#define SAW_CLAMP_PID(id) (((id) < 0 || (id) >= p.num_pages) ? 0 : (id))
  int pidv, pidv_nx;                 // pidv_nx stays unclamped until it becomes pidv
  int window = 0;                    // 16-batch window pidv covers
  SAW_LOAD_PIDS(pidv, pg_first)
  int t_end, seq_len_b;                // seq_len_b: cached tokens of the sequence (= position of an appended token)
  if (PAIR || CUT) {
    t_end = __builtin_amdgcn_readfirstlane(SAW_SEG(sg_t1));
    seq_len_b = __builtin_amdgcn_readfirstlane(SAW_SEQ(lk));
  } else {
    seq_len_b = max(min(p.seq_lens[b], p.bound), 0);
    t_end = min(seq_len_b, t_begin + p.chunk_tokens);
    if (t_begin >= t_end && !(p.append && t_begin == 0)) {            // block-uniform
      if (p.num_splits == 1)           // empty sequence and no merge pass: the output row is zero
        for (int i = threadIdx.x; i < G * DH; i += 64 * NW)
          store_elem(p.out, p.out_dtype, ((int64_t)b * p.n_q_heads + kvh * G) * DH + i, 0.f);
      return;
    }
  }
  SAW_LOAD_PIDS(pidv_nx, pg_first + 64)
  // this lane's share of the G query vectors (element lane + 64 j), issued ahead of the code transfers; a block that prepares
  // its range together: of this wavefront's share of them and of the new token's vectors
  uint32_t qbits[kBP ? 1 : 2 * G];
  uint32_t vbits[kBP ? (G + 1 + NW) / NW : 1][2];
  const bool block_new = p.append && (CUT ? cut_new : t_begin == 0);     // some wavefront of the block takes the new token
  if constexpr (kBP) {
    block_vectors_load<G, NW, HP>(p, b, kvh, block_new, wave, lane, vbits);
  } else {
    // (the block's G query heads are contiguous: G x 128 values, or G x 64 for a head pair)
    constexpr int NQ = HP ? G : 2 * G;
    const int64_t qoff = ((int64_t)b * p.n_q_heads + kvh * G) * DH + lane;
    if (p.q_dtype == SAW_F32) {
#pragma unroll
      for (int j = 0; j < 2 * G; ++j) qbits[j] = (j < NQ) ? ((const uint32_t*)p.q)[qoff + 64 * j] : 0u;
    } else {
#pragma unroll
      for (int j = 0; j < 2 * G; ++j) qbits[j] = (j < NQ) ? ((const uint16_t*)p.q)[qoff + 64 * j] : 0u;
    }
  }

  // fused append: the range that starts the sequence also takes the step's new token (of a batch cut by its lengths the one that ends
  // it, which has the fewest batches), in a block that shares it the last wavefront, for the same reason; its inputs are requested
  // here, with the query
  constexpr bool kOpen = !PAIR && NW > 1;
  const bool takes_new = block_new && (PAIR || wave == NW - 1);
  u32x2 new_w = u32x2{0u, 0u};
  int new_pid = -1;
  if (takes_new) {
    // (the block's new K|V values are 128 contiguous elements: one head, or a pair of 64-channel heads)
    if (!kBP)
      new_w = *(const u32x2*)((const uint16_t*)(lane < 32 ? p.k_new : p.v_new) + (int64_t)b * p.n_kv_heads * DH + (int64_t)kvh * D + 4 * (lane & 31));
    // (a length beyond the caller's bound was clamped for the attention; storing at the clamped
    // position would overwrite a cached token, so such a token is attended to but not stored)
    if ((seq_len_b >> 4) < p.max_pages && p.seq_lens[b] <= p.bound) new_pid = p.page_table[pt_row + (seq_len_b >> 4)];
  }

  // (first use of the page ids: only here, so that the query and new-token loads above are in
  // flight while this waits for them)
  pidv = SAW_CLAMP_PID(pidv);
  const int nb = max(t_end - t_begin + 63, 0) >> 6;               // batches of the range (0: only an appended token)
  // last batch of this wavefront (below first_batch if it has none)
  const int my_last = nb - 1 - ((nb - 1 - first_batch) % STEP + STEP) % STEP;

  // ---- fetch: LDS-DMA for the code tiles, registers for this lane's token metadata ----
#define SAW_ROTATE_PIDS(batch)                                                                  \
  if (((batch) >> 4) != window) {                                                               \
    window = (batch) >> 4;                                                                      \
    pidv = SAW_CLAMP_PID(pidv_nx);                                                              \
    SAW_LOAD_PIDS(pidv_nx, pg_first + 64 * window + 64)                                         \
  }
#define SAW_PID(batch, q) __builtin_amdgcn_readlane(pidv, 4 * ((batch) & 15) + (q))
  // (cache policy 2 = "nt": the cache is read once per launch, and marking the transfers as
  // streaming is worth 8-10 % of the whole launch: 150 -> 138 us on the ragged 256-sequence batch)
#define SAW_DMA(gptr, ldsptr)                                                                   \
  __builtin_amdgcn_global_load_lds((const GLOBAL_AS void*)(gptr), (LDS_AS void*)(ldsptr), 16, 0, 2)
  // V tiles of `batch` into VDST and the batch's metadata into MDST: lanes 0-31 bring the K
  // (scale, zero) pairs, lanes 32-63 the V pairs, 16 bytes (two tokens) each, so the metadata
  // also goes HBM -> LDS and no register is the target of a load that is still in flight
#define SAW_FETCH_V(batch, VDST, MDST)                                                          \
  {                                                                                             \
    SAW_ROTATE_PIDS(batch)                                                                      \
    _Pragma("unroll") for (int q = 0; q < 4; ++q) {                                             \
      const uint8_t* vp = p.v_codes + (int64_t)SAW_PID(batch, q) * page_stride + head_tile;     \
      SAW_DMA(vp + g_swz_v[q], VDST + q * kTileBytes);                                               \
    }                                                                                           \
    const int mq = HP ? (lane >> 4) : (lane >> 3) & 3;                                          \
    const int id = mq == 0 ? SAW_PID(batch, 0) : mq == 1 ? SAW_PID(batch, 1)                    \
                 : mq == 2 ? SAW_PID(batch, 2) : SAW_PID(batch, 3);                             \
    if (HP) { /* a page's pairs for both heads are 256 contiguous bytes: one transfer for K, one for V */ \
      const int64_t mo = (int64_t)id * page_meta + head_meta + 4 * (lane & 15);                 \
      SAW_DMA(p.k_meta + mo, MDST);                                                             \
      SAW_DMA(p.v_meta + mo, MDST + 1024);                                                      \
    } else {                                                                                    \
      const float* mp = (lane < 32 ? p.k_meta : p.v_meta) + (int64_t)id * page_meta + head_meta + 4 * (lane & 7); \
      SAW_DMA(mp, MDST);                                                                        \
    }                                                                                           \
  }
  // K tiles of `batch` into KDST (the ids were rotated by the V fetch of the same batch)
#define SAW_FETCH_K(batch, KDST)                                                                \
  {                                                                                             \
    _Pragma("unroll") for (int q = 0; q < 4; ++q) {                                             \
      const uint8_t* kp = p.k_codes + (int64_t)SAW_PID(batch, q) * page_stride + head_tile;     \
      SAW_DMA(kp + g_swz, KDST + q * kTileBytes);                                               \
    }                                                                                           \
  }

  // ---- the first transfers, then the q~ operands ----
  // The first batch's tiles leave as soon as the page ids are here, and the q~ preparation runs while
  // they travel.  For that, two things must hold.  Every load issued so far (page ids, query, new
  // token) is waited for before the transfers go out: the ids are needed now anyway, and with nothing
  // else outstanding no later wait for one of these loads can fall on the transfers.  And the
  // preparation's LDS scratch is memory no transfer of the first batch targets, reached through
  // restrict-qualified pointers: the compiler then orders none of its LDS accesses behind them.
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0x0F70);                      // vmcnt(0)
  BlockColumns<DN && kBP ? NW : 8> cols;
  if constexpr (DN && kBP) {
    // (in front of the transfers: loads return in order, and behind them R_l's 64 KiB from L2 would wait for HBM)
    if (p.dense_k || p.dense_v) block_columns_load<NW>(p.dense, wave, lane, cols);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (first_batch < nb) {
    SAW_FETCH_V(first_batch, vbuf_a, mbuf_a)
    SAW_FETCH_K(first_batch, kbuf)
  }
  // query scratch: up to G = 4 in the P buffer (no transfer ever targets it), else the second V
  // buffer for the rows (first written by the second batch's transfers, which leave after this)
  float* const qrows = (G <= 4) ? (float*)pbuf : (float*)vbuf_b;
  i32x4 a_q[NT][KS];
  float qsum[NT], qunit[NT];
  float new_x[4] = {0.f, 0.f, 0.f, 0.f};                      // the new token's channels of this lane, rotated
  if constexpr (kBP) {
    float* const rows = (float*)(lds_all + NW * kWaveLds + 16 + kSpareBytes);
    // (rows to be multiplied: wavefront 0's second V buffer and what follows, which nobody writes to before the barrier behind the product)
    block_prepare<G, NW, HP, DN>(p, vbits, block_new, wave, lane, (float*)(lds_all + 8 * kTileBytes), rows,
                                 pbuf, cols, a_q, qsum, qunit);
    if (takes_new) {
      const f32x4 v = *(const f32x4*)(rows + 128 * kNewRow<G> + 4 * lane);                 // K, then V
      new_x[0] = v.x; new_x[1] = v.y; new_x[2] = v.z; new_x[3] = v.w;
    }
  } else {
    float qraw[2 * G];
    const bool q_is_f32 = p.q_dtype == SAW_F32, q_is_bf16 = p.q_dtype == SAW_BF16;
#pragma unroll
    for (int j = 0; j < 2 * G; ++j) {                       // all three widenings, then selects
      const float as_f32 = __uint_as_float(qbits[j]);
      const float as_bf16 = __uint_as_float(qbits[j] << 16);
      const float as_f16 = f16_to_f32(qbits[j] & 0xffffu);
      qraw[j] = q_is_f32 ? as_f32 : (q_is_bf16 ? as_bf16 : as_f16);
      // randomised Hadamard: q diag(sigma) first (element lane + 64 j is channel lane + 64 (j & 1))
      if (p.rot_k && p.has_signs) qraw[j] = apply_sign(p.signs, HP ? lane : lane + 64 * (j & 1), qraw[j]);
    }
    prepare_q<G, HP, DN, kLoads<G, PAIR>>(p, qraw, lane, qrows, pbuf, a_q, qsum, qunit);
  }

  using State = RangeState<G, HP>;
  i32x4 digits[NT][NC];
  float m_ref[NT], lsum[NT], zs[NT];
  int unit[NT], room;
  State st{digits, m_ref, unit, lsum, zs, room};
  st.clear();
  NewToken nt;
  if constexpr (kOpen) {
    if (takes_new) {
      if (!kBP) rotate_token<HP, DN, kLoads<G, PAIR>>(p, lane, new_w, (float*)vbuf_b, new_x);
      open_with_token<G, HP>(p, kvh, lane, seq_len_b, new_pid, new_x, vbuf_b, a_q, qsum, qunit, st, nt);
    }
  }

  // One batch, whose first token is position tok0 of the sequence.  On entry the transfers of batch bi
  // (V into vcur, K into kb, metadata) are the only ones this wavefront has in flight.
  // The buffers come in as __restrict__ parameters: after inlining that gives the LDS accesses
  // and the LDS-DMA transfers distinct alias scopes, so the compiler's own wait-count insertion
  // does not drain the prefetch before reading a buffer no transfer is writing.  Correctness
  // does not rest on that analysis: the explicit vmcnt(0) below covers everything batch bi needs.
  auto body = [&](const int bi, const int tok0, uint8_t* __restrict__ const kb, uint8_t* __restrict__ const vcur,
                  uint8_t* __restrict__ const vnext, uint8_t* __restrict__ const pb,
                  uint8_t* __restrict__ const mcur, uint8_t* __restrict__ const mnext) __attribute__((always_inline)) {
    // (issued through the builtin, not inline asm, so that the compiler's wait-count pass sees it
    // and stops guarding earlier loads, e.g. the q~ operands, with waits of its own further down)
    __builtin_amdgcn_s_waitcnt(0x0F70);                    // vmcnt(0): batch bi has landed (codes in LDS, metadata)
    // (this lane's tokens are row16 of the four pages, its heads 4 t + grp)
    f32x2 km[NM][4];
#pragma unroll
    for (int n = 0; n < NM; ++n)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        // head pair: [page][kv head][token]
        km[n][q] = *(const f32x2*)(mcur + (HP ? 256 * q + 128 * (NM == 2 ? n : kv_of) : 128 * q) + 8 * row16);
      }
    // K operand reads first, before the next transfers are issued.
    u32x4 kw[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (KS == 2) {
        kw[q] = *(const u32x4*)(kb + q * kTileBytes + kr_off);
      } else {                                             // 16 channels of either head
        const u32x2 a = *(const u32x2*)(kb + q * kTileBytes + kr_pair[0]), b2 = *(const u32x2*)(kb + q * kTileBytes + kr_pair[1]);
        kw[q] = u32x4{a.x, a.y, b2.x, b2.y};
      }
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);                    // lgkmcnt(0): ... and they have returned: kb is free
    // The next batch of this wavefront, if it has one (the branch is wavefront-uniform and the
    // wait at the top of a batch is a full vmcnt(0), so the number of transfers in flight may
    // depend on the path).  vnext was last read two batches ago.
    const int nxt = min(bi + STEP, my_last);
    if (bi + STEP <= my_last) {
      SAW_FETCH_V(nxt, vnext, mnext)
      SAW_FETCH_K(nxt, kb)
    }

    // ---- logits of this lane's tokens and heads ----
    float lg[NT][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const i32x4 k0 = operand(code_bytes(kw[q].x), code_bytes(kw[q].y)), k1 = operand(code_bytes(kw[q].z), code_bytes(kw[q].w));
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const i32x4 none = i32x4{0, 0, 0, 0};
        const i32x4 dq = KS == 2 ? mfma_i8(a_q[t][KS - 1], k1, mfma_i8(a_q[t][0], k0, none)) : mfma_i8(a_q[t][0], t == 0 ? k0 : k1, none);
        const f32x2 m = km[t * (NM - 1)][q];
        lg[t][q] = (m.x * qunit[t]) * fmaf(-m.y, qsum[t], digits_value(dq));
      }
    }
    f32x2 vm[NM][4];
#pragma unroll
    for (int n = 0; n < NM; ++n)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        vm[n][q] = *(const f32x2*)(mcur + kMetaBytes<HP> / 2 + (HP ? 256 * q + 128 * (NM == 2 ? n : kv_of) : 128 * q) + 8 * row16);
    if (tok0 + 64 > t_end) {                                  // wavefront-uniform
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool valid = tok0 + 16 * q + row16 < t_end;
#pragma unroll
        for (int n = 0; n < NM; ++n) vm[n][q] = valid ? vm[n][q] : f32x2{0.f, 0.f};
#pragma unroll
        for (int t = 0; t < NT; ++t) lg[t][q] = valid ? lg[t][q] : -INFINITY;
      }
    }
    st.weigh(lg, vm, pb + pw_off);
    wave_sync();
    // ---- O[row][channel] += P (rows x 64 tokens) . V codes ----
    // The P operand reads are issued by hand: written as ordinary LDS loads, the compiler's
    // wait insertion cannot tell them from the buffers the LDS-DMA prefetch is filling and would
    // drain every transfer in flight (s_waitcnt vmcnt(0)) right here.
    i32x4 pa[NT];
    if constexpr (NT == 2)
      asm volatile("ds_read_b128 %0, %2\n\tds_read_b128 %1, %2 offset:%c3\n\ts_waitcnt lgkmcnt(0)"
                   : "=&v"(pa[0]), "=&v"(pa[1])
                   : "v"(pa_addr), "i"(kDigitTile)
                   : "memory");
    else
      asm volatile("ds_read_b128 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(pa[0]) : "v"(pa_addr) : "memory");
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const i32x2 tv = __builtin_amdgcn_ds_read_tr4_b64_v2i32((LDS_AS i32x2*)(vcur + vr_off[c >> 1] + 8 * (c & 1)));
      const i32x4 vb = operand(centred_bytes((uint32_t)tv.x), centred_bytes((uint32_t)tv.y));
#pragma unroll
      for (int t = 0; t < NT; ++t)
        if (NC == 8 || (c >> 2) == t) st.digits[t][c & (NC - 1)] = mfma_i8(pa[t], vb, st.digits[t][c & (NC - 1)]);
    }
  };
  for (int bi = first_batch; bi < nb; bi += 2 * STEP) {
    body(bi, t_begin + 64 * bi, kbuf, vbuf_a, vbuf_b, pbuf, mbuf_a, mbuf_b);
    if (bi + STEP < nb) body(bi + STEP, t_begin + 64 * (bi + STEP), kbuf, vbuf_b, vbuf_a, pbuf, mbuf_b, mbuf_a);
  }

  // Everything below reuses the buffers as scratch, so no transfer may be in flight (every batch's were waited for
  // when it began, and a wavefront without a batch has requested none: this waits for nothing, it states the rule).
  __builtin_amdgcn_s_waitcnt(0x0F70);                      // vmcnt(0)

  // Fused append, if the range did not open with it: the step's new token is quantised now, placed in the (idle) buffers as
  // token 0 of a batch, and attended to by one more pass of the batch code in which only that token is
  // valid (tok0 = t_end - 1: only position tok0 + 0 lies below t_end; the batch index is past the range,
  // so nothing is requested).
  if (takes_new) {
    if constexpr (!kOpen) {
      rotate_token<HP, DN, kLoads<G, PAIR>>(p, lane, new_w, (float*)vbuf_b, new_x);
      append_token<HP>(p, kvh, lane, seq_len_b, new_pid, new_x, kbuf, vbuf_a, mbuf_a, nt);
      body(0x3fffffff, t_end - 1, kbuf, vbuf_a, vbuf_b, pbuf, mbuf_a, mbuf_b);
    }
    append_store<HP>(p, lane, nt);                         // (nobody waits for these: see append_store)
  }

  // ---- fold the wavefronts of the block together: heads are dealt out to the wavefronts ----
  if constexpr (!PAIR && NW > 1) {
    block_epilogue<G, NW, HP, DN, CUT>(p, lds_all, wave, lane, b, kvh, split, st);
    return;
  }

  // ---- epilogue: reduce the per-lane sums ----
  st.sum_lanes();
  const int emode = PAIR ? mode : (p.num_splits == 1 ? (int)kSegAlone : (int)kSegSplitKV);
  if (emode == kSegSplitKV) {
    // one of several partitions: (max, sum, un-normalised accumulator) for the merge kernel
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int head = 4 * t + grp;
      if (G % 4 != 0 && head >= G) continue;
      float* const dst = p.ws + (((int64_t)b * p.n_q_heads + kvh * G + head) * p.num_splits + split) * (DH + 2);
      const int own = head / GK;                  // head pair: the half of the row that is this head's
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const float o = st.value(t, c);
        if (!HP || NC == 4 || (c >> 2) == own) dst[2 + 16 * (HP ? (c & 3) : c) + row16] = o;
      }
      if (row16 == 0) { dst[0] = st.m_ref[t]; dst[1] = st.lsum[t]; }
    }
    return;
  }
  // The range's result as a record (every read of this wavefront's V buffers is done):
  // acc[G][128] (un-normalised, zero-point term removed), then (max, sum) per head.  It lives at the
  // start of the V buffers (with G = 8 the pairs land at the start of the second one), or in the
  // block's spare slot when this wavefront still has its share of the long sequence to stream.
  float* const fb = (float*)vbuf_a;
  // (a shared range that is not this wavefront's last is the start of sequence sq >= 1)
  const bool to_spare = kSpare && emode == kSegShare && seg != nseg - 1;
  float* const rec = to_spare ? spare_rec + (sq - 1) * kRecFloats : fb;
  float* const ml = rec + G * D;
  wave_sync();
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int head = 4 * t + grp;
    if (G % 4 != 0 && head >= G) continue;
#pragma unroll
    for (int c = 0; c < NC; ++c) rec[head * D + 16 * (NC == 8 ? c : 4 * t + c) + row16] = st.value(t, c);
    if (row16 == 0) {
      ml[2 * head] = st.m_ref[t];
      ml[2 * head + 1] = st.lsum[t];
    }
  }
  // the records that make up the sequence's result: this one, or with a shared sequence those of
  // every wavefront that has a share, in wavefront order (so the sum does not depend on who
  // happens to come last)
  const float* recs[NW];
#pragma unroll
  for (int k = 0; k < NW; ++k) recs[k] = rec;
  int nrec = 1;
  if (PAIR && emode == kSegShare) {
    // LDS operations of a wavefront complete in order, so the record is in place before the
    // count; the wavefront that finds all others counted does the rest for everybody.
    // the sequence's wavefronts, and those of them that also hold a share of an earlier sequence of
    // the block (at most one: its record is the one in the spare slot)
    uint32_t mask = part_mask[0], lower = 0u;
#pragma unroll
    for (int k = 1; k < K; ++k)
      if (k == sq) { mask = part_mask[k]; } else if (k < sq) { lower |= part_mask[k]; }
    if (sq > 0) lower |= part_mask[0];
    mask = (uint32_t)__builtin_amdgcn_readfirstlane((int)mask);
    lower = (uint32_t)__builtin_amdgcn_readfirstlane((int)lower);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    int before = 0;
    if (lane == 0) before = __hip_atomic_fetch_add(done_cnt + sq, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    before = __builtin_amdgcn_readfirstlane(before);
    if (before != __popc(mask) - 1) {
      // (a record in this wavefront's own buffers is its last act; after one in the spare slot
      // the next range's prologue reuses the buffers)
      wave_sync();
      continue;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    nrec = 0;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
      if ((mask >> k) & 1u) {
        const float* rk = ((lower >> k) & 1u) ? spare_rec + (sq - 1) * kRecFloats
                                              : (const float*)(lds_all + k * kWaveLds + 4 * kTileBytes);
#pragma unroll
        for (int r = 0; r < NW; ++r)
          if (r == nrec) recs[r] = rk;
        ++nrec;
      }
    }
  }
  wave_sync();
  // combine and normalise into this wavefront's buffer.  The weight of record r for head h, the
  // denominator already divided in, is the same in every lane and is worked out first (the (max, sum)
  // pairs sit behind the rows of a record and are read before anything is overwritten); then element by
  // element, in place where the record lives in this buffer.
  float wgt[NW][G];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    float mr[NW], lr[NW];
#pragma unroll
    for (int r = 0; r < NW; ++r) {
      mr[r] = (r < nrec) ? recs[r][G * D + 2 * h] : -INFINITY;
      lr[r] = (r < nrec) ? recs[r][G * D + 2 * h + 1] : 0.f;
    }
    float mm = mr[0];
#pragma unroll
    for (int r = 1; r < NW; ++r) mm = fmaxf(mm, mr[r]);
    float den = 0.f;
#pragma unroll
    for (int r = 0; r < NW; ++r) {
      wgt[r][h] = (PAIR && nrec > 1) ? ((r < nrec) ? fast_exp2(mr[r] - mm) : 0.f) : (r == 0 ? 1.f : 0.f);
      den = fmaf(wgt[r][h], lr[r], den);
    }
    const float inv = __builtin_amdgcn_rcpf(den);
#pragma unroll
    for (int r = 0; r < NW; ++r) wgt[r][h] *= inv;
  }
  wave_sync();
#pragma unroll
  for (int it = 0; it < G * D / 64; ++it) {
    const int idx = lane + 64 * it;
    constexpr int kPerHead = D / 64;                          // iterations per head
    const int h = it / kPerHead;                              // compile-time after unrolling
    float v = wgt[0][h] * recs[0][idx];
    if (PAIR) {
#pragma unroll
      for (int r = 1; r < NW; ++r)
        if (r < nrec) v = fmaf(wgt[r][h], recs[r][idx], v);
    }
    fb[idx] = v;
  }
  wave_sync();
  // rotate back once for V (App. A.4; a learned rotation's transpose first, App. A.3), write the output
  float onorm = 1.0f;
  if constexpr (DN) {
    if (p.dense_v) wave_lds_matvec128<G, kLoadsOut<G, PAIR>>(fb, p.dense + kDenseD * kDenseD, lane);
  }
  if (p.rot_v) {
    wave_lds_fwht128<G>(fb, p.had_block, lane);
    onorm = had_norm(p.had_block);
  }
  const int64_t obase = ((int64_t)b * p.n_q_heads + kvh * G) * DH;
  if (HP) {
    for (int i = lane; i < G * D; i += 64) {
      float o = fb[i] * onorm;
      if (p.rot_v && p.has_signs) o = apply_sign(p.signs, i & (DH - 1), o);    // (o~ H_blk) diag(sigma) = o~ R^T
      const int h = i >> 7, c = i & 127;           // a row's own 64 channels; the other half is cross terms
      if ((c >> 6) == h / GK) store_elem(p.out, p.out_dtype, obase + h * 64 + (c & 63), o);
    }
  } else {
    // four consecutive channels per lane: 16-byte (fp32) or 8-byte (16-bit) stores, whole rows per instruction
#pragma unroll
    for (int it = 0; it < (G * D + 255) / 256; ++it) {
      const int i = 4 * (lane + 64 * it);
      if (G * D % 256 != 0 && i >= G * D) break;             // (one query head: 32 lanes hold its row)
      const f32x4 o4 = *(const f32x4*)(fb + i);
      float o[4] = {o4.x * onorm, o4.y * onorm, o4.z * onorm, o4.w * onorm};
      if (p.rot_v && p.has_signs) {                                            // (o~ H_blk) diag(sigma) = o~ R^T
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = apply_sign(p.signs, (i + e) & (DH - 1), o[e]);
      }
      if (p.out_dtype == SAW_F32) {
        *(f32x4*)((float*)p.out + obase + i) = f32x4{o[0], o[1], o[2], o[3]};
      } else {
        uint32_t w0, w1;
        if (p.out_dtype == SAW_BF16) {
          w0 = f32_to_bf16(o[0]) | ((uint32_t)f32_to_bf16(o[1]) << 16);
          w1 = f32_to_bf16(o[2]) | ((uint32_t)f32_to_bf16(o[3]) << 16);
        } else {
          w0 = f32_to_f16(o[0]) | ((uint32_t)f32_to_f16(o[1]) << 16);
          w1 = f32_to_f16(o[2]) | ((uint32_t)f32_to_f16(o[3]) << 16);
        }
        typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
        *(u32x2_t*)((uint16_t*)p.out + obase + i) = u32x2_t{w0, w1};
      }
    }
  }
  wave_sync();                                   // the next range's prologue reuses these buffers
  }  // ranges of this wavefront
}

#undef SAW_FETCH_V
#undef SAW_FETCH_K
#undef SAW_DMA
#undef SAW_PID
#undef SAW_ROTATE_PIDS
#undef SAW_LOAD_PIDS
#undef SAW_CLAMP_PID
#undef SAW_SEG
#undef SAW_SEQ

template <int G, bool HP, bool DN>
static void launch_g(const DecodeParams& p, int B, int nw, dim3 grid, hipStream_t st) {
  if constexpr (!(HP && G == 8)) {       // (two such blocks of head pairs with eight query rows would not fit LDS)
    if (p.pair == 4 && p.pair_seqs == 3) {
      decode_int4_mfma_kernel<G, 4, true, HP, 3, DN><<<dim3(1, grid.y, (B + 2) / 3), dim3(256), 0, st>>>(p);
      return;
    }
    if (p.pair == 2 && p.pair_seqs == 3) {
      decode_int4_mfma_kernel<G, 2, true, HP, 3, DN><<<dim3(1, grid.y, (B + 2) / 3), dim3(128), 0, st>>>(p);
      return;
    }
  }
  if (p.pair == 4) {
    decode_int4_mfma_kernel<G, 4, true, HP, 2, DN><<<dim3(1, grid.y, (B + 1) / 2), dim3(256), 0, st>>>(p);
    return;
  }
  if (p.pair) {
    decode_int4_mfma_kernel<G, 2, true, HP, 2, DN><<<dim3(1, grid.y, (B + 1) / 2), dim3(128), 0, st>>>(p);
    return;
  }
  if (p.cut) {
    if (nw >= 4) decode_int4_mfma_kernel<G, 4, false, HP, 2, DN, true><<<grid, dim3(256), 0, st>>>(p);
    else decode_int4_mfma_kernel<G, 2, false, HP, 2, DN, true><<<grid, dim3(128), 0, st>>>(p);
    return;
  }
  if (nw >= 8) decode_int4_mfma_kernel<G, 8, false, HP, 2, DN><<<grid, dim3(512), 0, st>>>(p);
  else if (nw >= 4) decode_int4_mfma_kernel<G, 4, false, HP, 2, DN><<<grid, dim3(256), 0, st>>>(p);
  else if (nw == 2) decode_int4_mfma_kernel<G, 2, false, HP, 2, DN><<<grid, dim3(128), 0, st>>>(p);
  else decode_int4_mfma_kernel<G, 1, false, HP, 2, DN><<<grid, dim3(64), 0, st>>>(p);
}

// `G`: query heads per kv head.  `nw`: wavefronts per (sequence, kv head, partition) block: 1, 2, 4
// or 8 (ignored in pair mode).  `head_pairs`: head_dim 64, grid.y = n_kv_heads / 2 blocks of two kv
// heads each (2 G rows), G <= 4; otherwise head_dim 128 and grid.y = n_kv_heads.
int launch_decode_int4_mfma(const DecodeParams& p, int G, int B, int nw, bool head_pairs, dim3 grid, hipStream_t st) {
  if (head_pairs) {
    switch (G) {
      case 1: launch_g<2, true, false>(p, B, nw, grid, st); break;
      case 2: launch_g<4, true, false>(p, B, nw, grid, st); break;
      case 4: launch_g<8, true, false>(p, B, nw, grid, st); break;
      default: return SAW_EINVAL;
    }
    return SAW_OK;
  }
  if (p.dense) {                        // a learned rotation after the Hadamard: the kernels that carry its code
    switch (G) {
      case 1: launch_g<1, false, true>(p, B, nw, grid, st); break;
      case 2: launch_g<2, false, true>(p, B, nw, grid, st); break;
      case 4: launch_g<4, false, true>(p, B, nw, grid, st); break;
      case 8: launch_g<8, false, true>(p, B, nw, grid, st); break;
      default: return SAW_EINVAL;
    }
    return SAW_OK;
  }
  switch (G) {
    case 1: launch_g<1, false, false>(p, B, nw, grid, st); break;
    case 2: launch_g<2, false, false>(p, B, nw, grid, st); break;
    case 4: launch_g<4, false, false>(p, B, nw, grid, st); break;
    case 8: launch_g<8, false, false>(p, B, nw, grid, st); break;
    default: return SAW_EINVAL;
  }
  return SAW_OK;
}

}  // namespace saw
