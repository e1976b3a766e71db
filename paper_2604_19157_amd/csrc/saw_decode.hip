// Split-KV merge (log-sum-exp) of the decode kernels' partial results, and the dispatch of the decode calls.
// Paper: Sec. 2 (decode step), Sec. 4.1 and App. A.4 (the output is rotated back once for V).
#include "saw_decode.h"
#include "saw_wave_util.h"
#include "saw_cut.h"

namespace saw {

// The partial results of one (sequence, query head): how many, and where the first one is.
// (CUT at compile time: a test of the argument block puts one more scalar-memory latency in front of everything; the decode of 1 x
// 131072 tokens took 1.016 times as long as with the merge kernel before there were cut batches, and takes 0.987 times.)
template <int D, bool CUT>
__device__ __forceinline__ int row_records(const DecodeParams& p, int b, int j, const float*& base) {
  if (CUT) {
    const int2 own = p.cut_of[b];             // (requested with the length; not written, and not used, if nothing ran)
    const int L = min(p.seq_lens[b], p.bound);
    base = p.ws + ((int64_t)j * p.cut + own.x) * (D + 2);
    return (L > 0 || p.append) ? own.y : 0;
  }
  // partitions that ran: those that start inside the cached tokens, and with a fused append the first one
  // in any case (it carries the step's own token)
  const int L = min(p.seq_lens[b], p.bound);
  base = p.ws + ((int64_t)b * p.n_q_heads + j) * p.num_splits * (D + 2);
  return max((max(L, 0) + p.chunk_tokens - 1) / p.chunk_tokens, p.append ? 1 : 0);
}

// y[r][j] = sum_i x[r][i] M[i][j] for four rows of 128 floats in LDS, run by a block of four wavefronts: wavefront w takes
// columns 32 w .. + 31, lane l four of them and 16 of the 128 terms.  M (64 KiB, from L2) is read once per four rows.
__device__ __forceinline__ void block_lds_matvec4(const float* x, float* y, const float* __restrict__ M, int wave, int lane) {
  const int col = 32 * wave + 4 * (lane & 7), k0 = 16 * (lane >> 3);
  f32x4 m[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) m[u] = *(const f32x4*)(M + (k0 + u) * 128 + col);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u4 = 0; u4 < 4; ++u4) {
      const f32x4 xv = *(const f32x4*)(x + 128 * r + k0 + 4 * u4);
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] = fmaf(xv[k], m[4 * u4 + k][c], acc[c]);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      acc[c] += dpp_f<0x128>(acc[c]);           // row_ror:8: the other eight lanes of the row
      acc[c] = add_xor32(add_xor16(acc[c]));
    }
    if (lane < 8) *(f32x4*)(y + 128 * r + col) = f32x4{acc[0], acc[1], acc[2], acc[3]};
  }
}

// ---------------------------------------------------------------------------------------
// Merge of the partitions of a (sequence, query head) by one wavefront, four rows per block: up to 16 records are requested
// at once, so a row of few partitions costs one trip to memory and no block barrier (64 x 64 rows of 64 channels, 6 partitions
// each: 5.1 us, 7.0 with a block of 256 threads per row; 48 x 32 rows of 128 channels: 4.0 and 4.6 us; 16 x 32: 3.9 and 4.0).
// (what a trip reads in the place of records past the last one: 0 times an infinite sum would be NaN)
__device__ const __attribute__((aligned(16))) float no_record[128 + 2] = {0.f};
template <int D, bool CUT>
__global__ __launch_bounds__(256) void decode_merge_rows_kernel(DecodeParams p) {
  constexpr int E = D / 64;                   // channels per lane
  constexpr int CH = 16;                      // records per trip
  const int b = blockIdx.y, lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool live = (int)blockIdx.x * 4 + wave < p.n_q_heads;                 // (an idle wavefront shadows the last row)
  const int j = min((int)blockIdx.x * 4 + wave, p.n_q_heads - 1);
  __shared__ __attribute__((aligned(16))) float rows[2][4][128];
  const float* base;
  const int ns = row_records<D, CUT>(p, b, j, base);
  float mm = -INFINITY, den = 0.f, num[E];
#pragma unroll
  for (int e = 0; e < E; ++e) num[e] = 0.f;
  for (int s0 = 0; s0 < ns; s0 += CH) {
    const int n = min(CH, ns - s0);
    const float* const at = base + (int64_t)s0 * (D + 2);
    float2 ml = make_float2(-INFINITY, 0.f);
    if (lane < n) ml = *(const float2*)(at + lane * (D + 2));
    float v[CH][E];
#pragma unroll
    for (int k = 0; k < CH; ++k) {
      if (k % 4 == 0 && k >= n) {             // (wavefront-uniform)
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int e = 0; e < E; ++e) v[k + u][e] = 0.f;
      } else if (k % 4 == 0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float* const src = (k + u < n ? at + (k + u) * (D + 2) : no_record) + 2 + E * lane;
          if (E == 2) {
            const f32x2 w = *(const f32x2*)src;
            v[k + u][0] = w.x; v[k + u][E - 1] = w.y;
          } else {
            v[k + u][0] = src[0];
          }
        }
      }
    }
    const float mnew = fmaxf(mm, __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(row_allmax(ml.x)))));
    const float alpha = fast_exp2(mm - mnew);
    const float a = fast_exp2(ml.x - mnew);   // 0 from lane n on
    den = fmaf(den, alpha, __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(row_allsum(a * ml.y)))));
#pragma unroll
    for (int e = 0; e < E; ++e) num[e] *= alpha;
#pragma unroll
    for (int k = 0; k < CH; ++k) {
      const float w = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(a), k));
#pragma unroll
      for (int e = 0; e < E; ++e) num[e] = fmaf(w, v[k][e], num[e]);
    }
    mm = mnew;
  }
  float o[E];
#pragma unroll
  for (int e = 0; e < E; ++e) o[e] = ns ? num[e] / den : 0.f;
  const bool dense = D == 128 && p.dense_v;   // the learned rotation's transpose first (App. A.3)
  if (dense || p.rot_v) {
    float* x = rows[0][wave];
#pragma unroll
    for (int e = 0; e < E; ++e) x[E * lane + e] = o[e];
    if (dense) {                              // block-uniform
      __syncthreads();
      block_lds_matvec4(rows[0][0], rows[1][0], p.dense + kDenseD * kDenseD, wave, lane);
      __syncthreads();
      x = rows[1][wave];
    }
    wave_sync();
    float onorm = 1.f;
    if (p.rot_v) {                            // (64 channels: half of a vector, the other half is nobody's)
      wave_lds_fwht128<1>(x, p.had_block, lane);
      onorm = had_norm(p.had_block);
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
      o[e] = x[E * lane + e] * onorm;
      if (p.rot_v && p.has_signs) o[e] = apply_sign(p.signs, E * lane + e, o[e]);         // (o~ H_blk) diag(sigma) = o~ R^T
    }
  }
  if (!live) return;
  const int64_t at = ((int64_t)b * p.n_q_heads + j) * D + E * lane;
  if (E == 2 && p.out_dtype == SAW_F32) {
    *(f32x2*)((float*)p.out + at) = f32x2{o[0], o[E - 1]};
  } else if (E == 2) {
    const uint32_t w = p.out_dtype == SAW_BF16 ? f32_to_bf16(o[0]) | ((uint32_t)f32_to_bf16(o[E - 1]) << 16)
                                               : f32_to_f16(o[0]) | ((uint32_t)f32_to_f16(o[E - 1]) << 16);
    *(uint32_t*)((uint16_t*)p.out + at) = w;
  } else {
    store_elem(p.out, p.out_dtype, at, o[0]);
  }
}

// Merge by a block of NT threads per row: rows of very many partitions (long contexts, small batches).
template <int D, int NT, bool CUT>
__global__ __launch_bounds__(NT) void decode_merge_kernel(DecodeParams p) {
  constexpr int NG = NT / D;                  // channel groups working on different splits
  constexpr int NW = NT / 64;
  const int j = blockIdx.x, b = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = tid % D, g = tid / D;
  const int64_t o_idx = ((int64_t)b * p.n_q_heads + j) * D + c;
  const float* base;
  const int ns = row_records<D, CUT>(p, b, j, base);
  if (ns == 0) {
    if (g == 0) store_elem(p.out, p.out_dtype, o_idx, 0.f);
    return;
  }
  __shared__ float wgt[kMaxSplits];
  __shared__ __attribute__((aligned(16))) float red[NG][D];
  __shared__ float wred[2][NW];
  // Every split's (max, sum) pair is read once, by thread s (at most 1024 splits): reference
  // maximum, then weights and the denominator.
  static_assert(NT == kMaxSplits, "a thread per split");
  float2 ml = make_float2(-INFINITY, 0.f);
  if (tid < ns) ml = *(const float2*)(base + (int64_t)tid * (D + 2));
  float mm = max_xor32(max_xor16(row_allmax(ml.x)));
  if (lane == 0) wred[0][wave] = mm;
  __syncthreads();
  mm = wred[0][0];
#pragma unroll
  for (int k = 1; k < NW; ++k) mm = fmaxf(mm, wred[0][k]);
  const float a_mine = (tid < ns) ? fast_exp2(ml.x - mm) : 0.f;
  if (tid < ns) wgt[tid] = a_mine;
  float den = add_xor32(add_xor16(row_allsum(a_mine * ml.y)));
  if (lane == 0) wred[1][wave] = den;
  __syncthreads();
  den = wred[1][0];
#pragma unroll
  for (int k = 1; k < NW; ++k) den += wred[1][k];
  // numerator: group g takes splits g, g + NG, ...
  float num = 0.f;
#pragma unroll 4
  for (int s = g; s < ns; s += NG) num = fmaf(wgt[s], base[s * (D + 2) + 2 + c], num);
  red[g][c] = num;
  __syncthreads();
  float o = 0.f;
  if (g == 0) {
#pragma unroll
    for (int k = 1; k < NG; ++k) num += red[k][c];
    o = num / den;
  }
  if (D == 128 && p.dense_v) {        // block-uniform: the learned rotation's transpose first (App. A.3)
    float* x = red[0];
    __syncthreads();                  // every read of red[][] above is done
    if (g == 0) x[c] = o;
    __syncthreads();
    if (wave == 0) wave_lds_matvec128<1>(x, p.dense + kDenseD * kDenseD, lane);
    __syncthreads();
    o = x[c];
  }
  if (p.rot_v) {                      // block-uniform
    float* x = red[0];
    __syncthreads();                  // every read of red[][] above is done
    if (g == 0) x[c] = o;
    __syncthreads();
    if (D == 128) {                   // one wavefront, three register passes, no block barriers in between
      if (wave == 0) wave_lds_fwht128<1>(x, p.had_block, lane);
      __syncthreads();
    } else {
      for (int st = 1; st < p.had_block; st <<= 1) {
        if (tid < D / 2) {            // each butterfly pair is owned by one thread
          const int i = ((tid & ~(st - 1)) << 1) | (tid & (st - 1));
          const float a = x[i], bb = x[i + st];
          x[i] = a + bb;
          x[i + st] = a - bb;
        }
        __syncthreads();
      }
    }
    o = x[c] * had_norm(p.had_block);
    if (p.has_signs) o = apply_sign(p.signs, c, o);             // (o~ H_blk) diag(sigma) = o~ R^T
  }
  if (g != 0) return;
  store_elem(p.out, p.out_dtype, o_idx, o);
}

// ---------------------------------------------------------------------------------------
template <bool CUT>
static void launch_merge(const DecodeParams& p, int B, int D, bool many, hipStream_t st) {
  if (many) {
    const dim3 grid(p.n_q_heads, B);
    if (D == 128) decode_merge_kernel<128, 1024, CUT><<<grid, dim3(1024), 0, st>>>(p);
    else decode_merge_kernel<64, 1024, CUT><<<grid, dim3(1024), 0, st>>>(p);
  } else {
    const dim3 grid((p.n_q_heads + 3) / 4, B);
    if (D == 128) decode_merge_rows_kernel<128, CUT><<<grid, dim3(256), 0, st>>>(p);
    else decode_merge_rows_kernel<64, CUT><<<grid, dim3(256), 0, st>>>(p);
  }
}

int launch_decode(const DecodeParams& p, int B, int D, int G, bool kv16, bool valu16, int kv_dtype, hipStream_t st) {
  // (the device's cut divides by p.cut - B and keeps kMaxCut lengths, the merge pass kMaxSplits weights: a plan that breaks this
  // would turn into reads out of range)
  if (p.cut && (p.cut < 2 * B || B > kMaxCut || p.cut > kMaxSplits)) return SAW_EINVAL;
  const dim3 grid = p.cut ? dim3(p.cut, p.n_kv_heads) : dim3(p.num_splits, p.n_kv_heads, B);
  const bool head_pairs = !kv16 && decode_head_pairs(D, p.n_kv_heads, G);
  if (!kv16 && (D == 128 || head_pairs)) {
    const int ny = head_pairs ? p.n_kv_heads / 2 : p.n_kv_heads;
    const dim3 mgrid = p.cut ? dim3(p.cut, ny) : dim3(p.num_splits, ny, B);
    if (launch_decode_int4_mfma(p, G, B, p.waves_per_item, head_pairs, mgrid, st) != SAW_OK) return SAW_EINVAL;
  } else if (kv16 && valu16) {
    if (launch_decode_kv16_valu(p, G, kv_dtype, grid, st) != SAW_OK) return SAW_EINVAL;
  } else if (kv16) {
    if (launch_decode_kv16_mfma(p, D, G, kv_dtype, grid, st) != SAW_OK) return SAW_EINVAL;
  } else {
    if (launch_decode_int4_split64(p, G, p.waves_per_item, grid, st) != SAW_OK) return SAW_EINVAL;
  }
  if (hipGetLastError() != hipSuccess) return SAW_ELAUNCH;
  if (!p.cut && p.num_splits == 1 && !valu16) return SAW_OK;  // the kernel wrote the output itself
  // (a sequence has more than 16 partitions - if the lengths cut the batch, on average -: a block of 1024 threads per row; otherwise
  // a wavefront per row.  In between a cut batch has rows of more than 16, which take the wavefront a second trip: few rows and a
  // bound that allows it get the blocks as well - 4 ragged up to 9000 tokens, 32 query / 8 kv heads, fused step: 18.2 us, 19.4 with a
  // wavefront per row; 80 ragged up to 2600, 8 / 1 heads, 640 rows of 12 slots: 1.08 times as long with a block per row)
  if (p.cut) launch_merge<true>(p, B, D, p.cut > 16 * B || (D == 128 && p.cut > 14 * B && p.bound > 4096 && (int64_t)B * p.n_q_heads <= 512), st);
  else launch_merge<false>(p, B, D, p.num_splits > 16, st);
  return hipGetLastError() == hipSuccess ? SAW_OK : SAW_ELAUNCH;
}

// (Times as the lines were drawn by, with products of bf16 limbs.)
// How the matrix-core INT4 kernel hands out work when one partition covers each sequence and the
// batch provides more (sequence, kv head) items than compute units (and at most 16 lengths per
// lane for the in-kernel ranking).  A compute unit holds 8 wavefronts of this kernel, 2048 on
// the chip:
//   * up to 2048 items everything is resident at once and nothing rebalances later, so the
//     work is evened out up front: pair mode, blocks over (long, short) pairs of sequences, of
//     four wavefronts while that still fits the 2048 slots and of two beyond.  Four-wavefront
//     blocks pay off on ragged batches from 576 items on (256 sequences x 4 heads: 82 -> 70 us,
//     90 x 8: 70 -> 61 us, 72 x 8: 63 -> 57 us against 2 or 4 wavefronts interleaving each
//     item's batches; equal lengths lose 2-8 us to the ranking and the records; at 528 items
//     four interleaving wavefronts per item are ahead: 51 against 64 us).  Between 1025 and 1151
//     items two interleaving wavefronts per item still fit the slots well enough (136 x 8: 79
//     against 94 us in pair mode); from 1152 on they spill into a second round.  Up to 1536
//     items blocks of four wavefronts over THREE sequences then fill the chip where blocks of two
//     over pairs leave a quarter to a half of the slots empty (144 x 8: 93 -> 83 us, 160 x 8:
//     93 -> 85 us, 176 x 8: 94 -> 89 us, level at 192 x 8), beyond that blocks of two;
//   * beyond that blocks queue for slots in index order, which is list scheduling: one
//     wavefront per item, sequences taken longest first, so the launch ends on the shortest.
//     (Measured at 288..512 sequences x 8 heads: 173-270 us against 224-332 us in pair mode,
//     whose equal blocks make the last round as long as the others; 2 or 4 wavefronts per item
//     were never better.);
//   * short bounds leave nothing worth evening out: the plan's wavefronts take each sequence as it comes, without the ranking
//     and the records (two of them up to 1151 items, one above).  96 x 8 of 250 tokens 20 -> 14 us, ragged up to 500 23 -> 17, 128 x 8
//     x 500 25 -> 19; 144 x 8 x 250 25 -> 19, 256 x 8 ragged up to 250 25 -> 20, 512 x 8 x 63 37 -> 25.  Above these bounds the batches
//     with a few long sequences lose (128 x 8 up to 750 tokens by 6 %, 192 x 8 up to 500 by 7 %).  The caller's order saves the
//     ranking: with it up to 256 tokens and 1024 items only (128 x 8 x 250 18 -> 14 us, up to 500 tokens 16 -> 17; 130 x 8 x 63
//     14 -> 17, 400 x 8 ragged up to 250 30 -> 33).
BlockPlan plan_blocks(const saw_cache_t* c, bool kv16, int B, int G, const SplitPlan& plan, bool order) {
  BlockPlan r = {0, 2, 0};
  if (plan.cut || plan.num_splits != 1 || B > 1024 || plan.valu16) return r;
  const int64_t n_kv = (int64_t)B * c->n_kv_heads;
  if (kv16) {
    // the 16-bit matrix-core kernel has the two-wavefront pair mode as well (same conditions), so that
    // the comparison on a ragged batch is between formats and not between schedules; only above bounds of 256 tokens (48 x 8 ragged
    // up to 250 tokens 26 us with pair blocks, 22 without, 256 x 8 x 250 59 and 53, 96 x 8 x 63 18 and 13; from 500 tokens on level, and
    // 256 x 8 ragged up to 1000 ahead by 8 %), and for the shapes with eight query heads per kv head or head_dim 64 only above 1024: of
    // shorter sequences the ranking takes longer than it saves (257 x 1 kv heads of 128, eight query heads each, up to 150 tokens
    // 27.6 us with pair blocks, 15.7 without; 256 x 8 of 600 equal tokens level, ragged up to 1200 with them ahead by 6 %)
    if (plan.bound > (c->head_dim == 128 && G <= 4 ? 256 : 1024) && n_kv > 256 && (int64_t)((B + 1) / 2) * c->n_kv_heads <= 1024) r.pair = 2;
    return r;
  }
  if (c->head_dim == 64 && !decode_head_pairs(64, c->n_kv_heads, G)) {
    r.sorted = order && n_kv > 256;             // one 64-channel head at a time: the caller's order, if there is one
    return r;
  }
  const int per_seq = decode_items_per_seq(c->head_dim, c->n_kv_heads);   // head_dim 64: pairs of kv heads
  const int64_t items = (int64_t)B * per_seq;
  const int64_t blocks = (int64_t)((B + 1) / 2) * per_seq, blocks3 = (int64_t)((B + 2) / 3) * per_seq;
  // (blocks over three sequences: not for head pairs with eight query rows, two such blocks of four with their two spare records do
  // not fit a compute unit's LDS)
  const bool threes = !(c->head_dim == 64 && G == 4);
  const int short_bound = items <= 1024 ? (order ? 256 : 512) : (order ? 0 : 256);
  if (items < 576 || plan.chunk_tokens <= short_bound) return r;
  if (blocks <= 512) {
    r.pair = 4;
  } else if (items >= 1152 && blocks3 <= 512 && threes) {
    r.pair = 4;
    r.pair_seqs = 3;
  } else if (items >= 1152 && blocks <= 1024) {
    r.pair = 2;                                 // (whatever the plan's wavefronts per item)
  } else if (items > 1024 && (plan.waves_per_item == 1 || plan.chunk_tokens <= 256)) {
    // (1025 to 1151 items get here only with the caller's order, which makes pairs cheap; without it they keep the plan's two wavefronts)
    if (blocks <= 1024) {
      r.pair = 2;
    } else if (items <= 2304 && blocks3 <= 1024 && threes) {
      // just above 2048 items: blocks of two wavefronts over THREE sequences keep everything resident
      // (equal lengths, where the longest-first order has nothing to reorder and the last 32 items ran
      // alone: 260 x 8 sequences of 2304 tokens 165 -> 135 us; ragged batches 137-148 us either way up
      // to 288 x 8; from 320 x 8 on the longest-first order is ahead: 155 against 166 us)
      r.pair = 2;
      r.pair_seqs = 3;
    } else {
      r.sorted = 1;
    }
  }
  return r;
}

int run_decode(const saw_cache_t* c, bool kv16, const void* k_pages, const void* v_pages, int kv_dtype,
               const void* q, int q_dtype, int B, int Hq, const int32_t* pt, int max_pages,
               const int32_t* seq_lens, float sm_scale, void* out, int out_dtype, void* ws,
               const SplitPlan& plan, const void* k_new, const void* v_new, int kv_new_dtype,
               const int32_t* order, hipStream_t st) {
  DecodeParams p;
  p.order = kv16 ? nullptr : order;
  p.k_codes = (const uint8_t*)k_pages;
  p.v_codes = (const uint8_t*)v_pages;
  p.k_meta = c->k_meta;
  p.v_meta = c->v_meta;
  p.q = q;
  p.page_table = pt;
  p.seq_lens = seq_lens;
  p.ws = (float*)ws;
  p.out = out;
  const float scale = (sm_scale > 0.f) ? sm_scale : 1.0f / sqrtf((float)c->head_dim);
  p.q_scale = scale * 1.4426950408889634f;
  p.q_dtype = q_dtype;
  p.out_dtype = out_dtype;
  p.n_q_heads = Hq;
  p.n_kv_heads = c->n_kv_heads;
  p.max_pages = max_pages;
  p.num_pages = c->num_pages;
  p.had_block = c->had_block;
  p.rot_k = !kv16 && c->had_block > 1 && (c->rotate_mask & SAW_ROT_K);
  p.rot_v = !kv16 && c->had_block > 1 && (c->rotate_mask & SAW_ROT_V);
  for (int i = 0; i < 4; ++i) p.signs.w[i] = kv16 ? 0u : c->sign_bits[i];
  p.has_signs = (p.signs.w[0] | p.signs.w[1] | p.signs.w[2] | p.signs.w[3]) != 0;
  p.dense = kv16 ? nullptr : (const float*)c->dense_rot;
  p.dense_k = p.dense && (c->rotate_mask & SAW_ROT_K);
  p.dense_v = p.dense && (c->rotate_mask & SAW_ROT_V);
  p.num_splits = plan.num_splits;
  p.chunk_tokens = plan.chunk_tokens;
  p.bound = plan.bound;
  p.waves_per_item = plan.cut ? plan.cut_waves : plan.waves_per_item;
  p.cut = plan.cut;
  p.cut_min = plan.cut_min;
  p.cut_of = plan.cut ? (int2*)((uint8_t*)ws + partial_bytes(1, Hq, plan.cut, c->head_dim)) : nullptr;
  p.k_new = k_new;
  p.v_new = v_new;
  p.kv_new_dtype = kv_new_dtype;
  p.append = k_new != nullptr;
  p.batch = B;
  const int G = Hq / c->n_kv_heads;
  const BlockPlan blocks = plan_blocks(c, kv16, B, G, plan, p.order != nullptr);
  p.pair = blocks.pair;
  p.pair_seqs = blocks.pair_seqs;
  p.sorted = blocks.sorted;
  return launch_decode(p, B, c->head_dim, G, kv16, plan.valu16 != 0, kv_dtype, st);
}

}  // namespace saw
