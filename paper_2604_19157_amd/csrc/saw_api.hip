// C ABI entry points: argument validation on the host, then kernel launches on the
// caller's stream.  No allocation, no synchronisation, no global state.
#include <math.h>

#include <mutex>

#include "saw_decode.h"

// Split-KV scratch of saw_paged_decode_attn_static, the entry point for callers that cannot
// allocate: one array per GPU the library runs on, held until the process ends.  In host code the
// array's name is only a handle for hipGetSymbolAddress; kernels get the address that call returns.
static __device__ __align__(256) unsigned char scratch[SAW_STATIC_SCRATCH_BYTES];

namespace saw {


int launch_prepare_dense(const float*, void*, hipStream_t);
int launch_decode_order(const int32_t*, int, int, int32_t*, hipStream_t);
int launch_read_probe(const saw_cache_t*, const int32_t*, int64_t, void*, int32_t, hipStream_t);
int launch_plain_store_valu(const saw_cache_t*, const void*, const void*, int, int64_t, int64_t, const int32_t*, int32_t,
                            int32_t, const int32_t*, hipStream_t);
int launch_store_layers(const saw_cache_t*, const void* const*, const void* const*, int, int, int64_t, int64_t,
                        const int32_t*, int32_t, int32_t, const int32_t*, hipStream_t);
int launch_flatten(const saw_cache_t*, const int32_t*, int32_t, int32_t, int32_t, int32_t, void*, void*, int64_t,
                   hipStream_t);
int launch_dequant(const saw_cache_t*, const int32_t*, int32_t, int32_t, int32_t, int32_t, int32_t,
                   float*, float*, hipStream_t);
int launch_kv16_store(const saw_cache_t*, void*, void*, const void*, const void*, int64_t, int64_t,
                      const int32_t*, int32_t, int32_t, const int32_t*, hipStream_t);
int run_decode(const saw_cache_t* c, bool kv16, const void* k_pages, const void* v_pages, int kv_dtype,
               const void* q, int q_dtype, int B, int Hq, const int32_t* pt, int max_pages,
               const int32_t* seq_lens, float sm_scale, void* out, int out_dtype, void* ws,
               const SplitPlan& plan, const void* k_new, const void* v_new, int kv_new_dtype,
               const int32_t* order, hipStream_t st);

static bool aligned16(const void* p) { return (((uintptr_t)p) & 15u) == 0; }

static bool shape_ok(const saw_cache_t* c) {
  if (c->page_size != 16) return false;
  if (c->head_dim != 64 && c->head_dim != 128) return false;
  if (c->n_kv_heads < 1 || c->num_pages < 1) return false;
  return true;
}

// (The times beside the INT4 lines from here on are those the lines were drawn by, with products of bf16 limbs, when a batch took 2.6 times
// the vector instructions.  Calls take 0.86 of them now in the mean; the lines were not drawn again.)
//
// A batch cut by its own lengths (saw_cut.h) into at most `slots` partitions per kv head, of `waves` wavefronts and at least
// four 64-token batches each: a shorter one costs more in prologue and merge pass than it brings.  False if a sequence
// would not get two partitions on average (the rounding of a sequence's share to whole partitions then costs too much), and
// for a single sequence, whose fixed partitions can request their page ids before the length is there (1 x 131072 tokens,
// 64 query heads: 36.5 against 38.6 us).
static bool cut_plan(int B, int units, int slots, int waves, SplitPlan* plan) {
  constexpr int kMin = 4;
  if (B == 1 || B > kMaxCut || (int64_t)B * units >= (1 << 23)) return false;   // (counts are divided in fp32)
  const int64_t most = (int64_t)B * ((units + kMin - 1) / kMin);
  int w = slots < most ? slots : (int)most;
  if (w > kMaxSplits) w = kMaxSplits;
  if (w < 2 * B) return false;
  plan->cut = w;
  plan->cut_min = kMin;
  plan->cut_waves = waves;
  return true;
}

static bool block_ok(const saw_cache_t* c) {
  const int h = c->had_block;
  if (!(h == 1 || h == 16 || h == 32 || h == 64 || h == 128)) return false;
  if (h > c->head_dim) return false;
  if (c->rotate_mask & ~(SAW_ROT_K | SAW_ROT_V)) return false;
  // sign bits exist for the head's channels only
  if (c->head_dim == 64 && (c->sign_bits[2] | c->sign_bits[3])) return false;
  // the learned rotation is built for head_dim 128, its prepared buffer read with 16-byte loads
  if (c->dense_rot && (c->head_dim != kDenseD || !aligned16(c->dense_rot))) return false;
  return true;
}


// Wavefronts of the INT4 block that takes a whole sequence (one partition), by the number of (kv head, or pair of heads, sequence)
// items; `rows`: query heads of a block; `nw`: what the bound alone asks for.  Up to 256 items the block of eight above; from 1152
// on pair blocks and one wavefront (plan_blocks).  In between the chip holds four wavefronts for every item up to 512 and two up to
// 1024, and a wavefront that has only a batch or two is still better than a slot left empty, however short the sequences.  Fused
// step, 32 query / 8 kv heads, us, one wavefront an item (pair blocks) before: 64 x 250 tokens 17.6, now 10.8; 64 x 750 30 and 16.4; 64
// ragged up to 1500 30 and 21; learned 64 x 750 40 and 22.  513 to 575 items: 68 x 250 22 and 13, four wavefronts only from 1024
// tokens on, where their second round is paid for (68 x 250 17, x 750 level, 68 ragged up to 1000 20.4 against 24 with two), with one or
// two query rows a block from 2048 on (one: 140 x 4 heads x 1400 28.8, 31.5 with four, two: x 1500 30.7 and 33.4; from 2000 on level);
// 1040 ragged up to 750 33 and 24.  More than 1024 sequences were never in pair blocks, and two wavefronts are no gain over one
// (1030 x 1 kv head x 100 tokens, four query heads 14.3 and 16.9, eight 17.2 and 21.1; x 600 level).
static int whole_waves(int64_t items, int rows, int units, int nw) {
  if (items <= 256 || items >= 1152) return nw;
  if (items <= 512 || (items < 576 && units >= (rows <= 2 ? 32 : 16))) return 4;
  return 2;
}

// The matrix-core INT4 kernel for rows of 128 channels holds 2048 wavefronts.  `per_seq`: (kv head, or pair of heads) items of a
// sequence.  What was measured, decode or fused step, 32 query / 8 kv heads, against the fixed partitions (in brackets):
//   * partitions of four wavefronts, which fold in LDS, leave the merge pass a quarter of the records, where that still gives
//     a sequence eight partitions on average, so that rounding its share to whole ones costs little: 4 x 131072 tokens
//     108.7 us (111.5; two wavefronts 109.7), 8 ragged up to 3000 under a loose bound 17.0 (22.8; 18.7), 8 x 8192 24.3 (26.0);
//   * two wavefronts otherwise: 16 x 4096 24.2 (25.8), 48 ragged up to 4096 34.3 (37.5, with a loose bound 54; four wavefronts
//     39.7), 32 ragged 26.7 (27.8, loose 47), 200 ragged x 2 heads 35.2 (37.0).  Equal lengths under a tight bound, which fixed partitions
//     serve best, at 43 to 63 sequences: 43 x 4096 52.0 (54.2), 48 x 4096 52.9 (62.9), 63 x 2304 39.3 (51.0), the least 43 x 1100
//     24.4 (23.8) and 43 x 3000 under a loose bound 38.3 (37.5); 10 x 7000 27.6 (26.7), 60 x 7000 x 3 heads 43.0 (41.7);
//   * from 512 items on one partition per sequence stays ahead or level (64 ragged 43.0 against 43.2, equal lengths 35.0
//     against 39.8, 96 ragged 57.3 against 59.6);
//   * the block of eight, which has no merge pass and follows the lengths too, stays ahead where its wavefronts have at most four
//     batches (4 x 256 12.7 against 16.4, 16 ragged up to 1000 under a bound of 2000 14.7 against 16.7), five from 129 items on
//     (20 x 2304 19.0 against 21.4, 16 x 2304 18.9 against 19.3 but ragged 18.3 against 17.4), eight from 192 on (24 x 2560 20.7 against
//     23.9, 28 x 3584 26.2 against 30.3, 28 of up to 1750 under a bound of 3500 16.6 against 18.6; 28 ragged up to 3500 24.4 against
//     23.1, 24 ragged up to 4000 26.1 against 23.0).  Pairs of 64-channel heads: five from 192 items on (56 x 3584 31.2
//     against 33.4, but ragged 29.8 against 25.5);
//   * from 257 items on four wavefronts over the whole sequence (whole_waves) take its place where each has at most four batches
//     (40 x 200 tokens 17.6 us, 10.6 with them, 62 x 800 21.1 and 17.7), three for pairs of 64-channel heads, five with the learned rotation,
//     whose preparation every partition would repeat, but with eight query heads three.  The line is where a batch with one sequence in
//     sixteen at the bound and the others an eighth of it does not lose (over the time of the cut: 50 x 1000 0.92, x 1150 1.08, x 1400 1.19;
//     pairs 100 x 700 0.96, x 850 1.08, x 1150 1.18; learned 50 x 1150 0.99, x 1400 1.05, x 2000 1.18, eight query heads 132 x 2 heads x 700
//     0.99, x 850 1.10, x 1150 1.15); equal and ragged lengths would gain up to 1500 tokens (48 x 1500 0.85).
static void plan_cut(int B, int units, int per_seq, int G, bool pairs, bool learned, SplitPlan* plan) {
  const int64_t items = (int64_t)B * per_seq;
  const int per_wave = (units + 7) / 8;
  const int most = pairs ? (items >= 192 ? 5 : 4) : items >= 192 ? 8 : items > 128 ? 5 : 4;
  if (plan->waves_per_item == 8 && per_wave <= most) return;
  if (items >= 512) return;
  if (items > 256 && (units + 3) / 4 <= (pairs || (learned && G == 8) ? 3 : learned ? 5 : 4)) {
    plan->num_splits = 1;
    plan->chunk_tokens = units * 64;
    plan->waves_per_item = whole_waves(items, pairs ? 2 * G : G, units, 1);
    return;
  }
  if (cut_plan(B, units, 512 / per_seq, 4, plan) && plan->cut >= 8 * B) return;
  plan->cut = 0;
  cut_plan(B, units, 1024 / per_seq, 2, plan);
}

// The kernel that takes 64-channel heads one at a time (saw_decode_split.hip).  Its registers allow 12 wavefronts on a
// compute unit and a batch is only 5 KiB, so it wants 3072 of them.  Small batches of short contexts: one block of eight
// wavefronts per (sequence, kv head), a single launch.  Otherwise the batch is cut by its own lengths, as long as that
// gives a sequence two slots on average; beyond that one partition per sequence, of four wavefronts while they fit.  Four
// wavefronts a slot, 2048 in all, where a sequence gets four slots of those (16 ragged x 8 heads of 300-3000 tokens 17.5 us, 19.1
// with 3072, 22.4 and 25.3 with one wavefront a slot; 64 ragged 40.0, with one wavefront 32.1, which is why it needs the four).
// Short bounds of more items are not cut: four wavefronts over the whole sequence, no merge pass, while they fit and have at most
// six batches each (eight query heads, fused step: 33 x 400 tokens 17 us, 13 so, 64 x 700 22 and 16, 96 ragged up to 1000 26 and 22), four
// with eight query heads in batches that can be cut (with one sequence in sixteen at the bound, the others an eighth of it: 95 x 1000 level,
// x 1150 27 % longer than cut, x 1400 40 %; four query heads 0.72 to 0.96 up to 1530), and up to 1024 items, where they no longer fit, at most three (110 x 400 24 and
// 21, 128 x 767 33 and 29; x 1000 level); one or two batches in all still go to one wavefront there (200 tokens 15 and 20).
static void plan_split64(const saw_cache_t* c, int B, int G, int units, SplitPlan* plan) {
  const int64_t items = (int64_t)B * c->n_kv_heads;
  constexpr int kWaves = 3072;
  const int per_wave = (units + 7) / 8;
  plan->waves_per_item = 1;
  if (items <= 256 && (per_wave <= 5 || (items >= 192 && per_wave <= 8))) {
    plan->num_splits = 1;
    plan->chunk_tokens = units * 64;
    plan->waves_per_item = 8;
    return;
  }
  if (items > 256 && (items <= 768 ? units <= (G == 8 && B <= kMaxCut ? 16 : 24) : items <= 1024 && B <= kMaxCut && units > 4 && units <= 12)) {
    plan->num_splits = 1;
    plan->chunk_tokens = units * 64;
    plan->waves_per_item = 4;
    return;
  }
  if (cut_plan(B, units, 2048 / 4 / c->n_kv_heads, 4, plan) && plan->cut >= 4 * B) return;
  plan->cut = 0;
  if (B == 1) {
    const int s = 512 / c->n_kv_heads < (units + 3) / 4 ? 512 / c->n_kv_heads : (units + 3) / 4;
    const int chunk = (units + (s > 1 ? s : 1) - 1) / (s > 1 ? s : 1);
    plan->num_splits = (units + chunk - 1) / chunk;
    plan->chunk_tokens = chunk * 64;
    plan->waves_per_item = 4;
    return;
  }
  if (cut_plan(B, units, kWaves / c->n_kv_heads, 1, plan)) return;
  // (fixed partitions, as planned, where a batch of long contexts or bounds is beyond what can be cut)
  if ((B > kMaxCut || (int64_t)B * units >= (1 << 23)) && items < kWaves / 2) return;
  plan->num_splits = 1;
  plan->chunk_tokens = units * 64;
  plan->waves_per_item = items * 4 <= kWaves ? 4 : 1;
}

// Does the vector-ALU kernel take a 16-bit call?  One query head per kv head: always.  Two: unless the batch fills the chip with
// items several times over (above 2048 items the matrix-core kernel takes 0.60 to 1.01 of its time), or has long contexts for enough
// items and can be cut by its own lengths (bounds above 1280 tokens, 33 to 1023 items: 0.64 to 1.04).  Elsewhere the matrix-core kernel's
// start-up decides (2 x 2304 tokens x 8 kv heads 11.2 and 12.0 us) or the ranking of the pair blocks (257 x 1 of up to 250
// tokens 10.9 and 16.7), and between 1024 and 2048 items the partitions that a bound of the caller's leaves empty (200 ragged x 8 up
// to 600 tokens under a bound of 1200: 40 and 58).
static bool takes_valu16(const saw_cache_t* c, int B, int G, int units) {
  if (c->head_dim != 64 || G < 1 || G > 2) return false;
  const int64_t items = (int64_t)B * c->n_kv_heads;
  const bool many = items > 2048;
  const bool long_ones = units > 20 && items > 32 && items < 1024 && B <= kMaxCut;
  return G == 1 || !(many || long_ones);
}

// Partitions of 64 or 128 tokens (make_plan): wavefronts in all; of the 16-bit call items and partitions a sequence; of the INT4 call of
// one sequence items and 64-token units
constexpr int64_t kFineWaves = 1792, kFineItems16 = 320, kFine16 = 448, kFineItems4 = 16, kFineUnits4 = 128;

// Split-KV plan.  Partitions are whole multiples of 64 tokens so every wavefront pass
// starts on a page boundary.  The automatic choice aims at about 2048 wavefronts (8 per compute
// unit): one partition per sequence once the batch alone provides them, otherwise partitions of
// at least 256 tokens, and 2 or 4 wavefronts per partition when even those are too few.
// The INT4 kernels (`kv16` false) stay with one partition from 512 (sequence, kv head) items on:
// their pair mode evens out ragged lengths inside the launch at any occupancy, and the merge
// pass costs more than the extra wavefronts bring (256 sequences x 4 kv heads, 2304 tokens each:
// 61 us against 66 us with two partitions; ragged 80 against 84; at 320 items partitions win).
// `G`: query heads per kv head.  `fixed`: the plan in fixed partitions that saw_decode_plan reports is wanted.
static bool make_plan(const saw_cache_t* c, int B, int G, bool fixed, int max_pages, int max_seq_len, int num_splits,
                      bool kv16, SplitPlan* plan) {
  const int64_t cap = (int64_t)max_pages * c->page_size;
  if (cap <= 0 || cap > 0x7fffffffLL) return false;
  int bound = (max_seq_len <= 0) ? (int)cap : max_seq_len;
  if (bound > cap) return false;
  if (num_splits < 0 || num_splits > kMaxSplits) return false;
  const int units = (bound + 63) / 64;                    // 64-token units
  const bool valu16 = kv16 && takes_valu16(c, B, G, units);
  int S = num_splits;
  bool block_of_eight = false;
  if (S == 0) {
    const int64_t items = (int64_t)B * (kv16 && !fixed && !valu16 ? c->n_kv_heads : decode_items_per_seq(c->head_dim, c->n_kv_heads));
    // one wavefront per (item, partition), about 8 per compute unit; a quarter more for 257 to 511 items,
    // the zone of mid-size ragged batches, where many partitions of the shorter sequences are empty
    // (48 ragged sequences x 8 kv heads: 6 partitions 37.1 us, 7: 34.4 us, 8: 34.2 us; 33 x 8: 8 partitions
    // 30.3 us, 10: 27.7 us)
    const int64_t slots = (items > 256 && items < 512) ? 2560 : 2048;
    int64_t s = (slots + items - 1) / items;
    const int64_t max_by_min_chunk = (units + 3) / 4;      // partitions of >= 256 tokens
    if (s > max_by_min_chunk) s = max_by_min_chunk;
    // ... of the 16-bit call 64 or 128 where all of those are resident at once with room to spare (1792 of 2048 wavefronts): its
    // batches are 32 tokens, eight of them in a row take longer than the merge pass takes for more records (32 query / 8 kv heads, us:
    // 1 x 400 tokens 17.3 with 256 a partition, 12.1 with 64; 4 x 1000 19.7 and 13.8; 8 x 2000 25.6 and 23.0 with 128; 16 ragged up to 800
    // 23.0 and 17.7; 32 x 512 25.8 and 22.7 with 128; with 192 level, under loose bounds 5 % slower).  Bounds of up to five units
    // stay as they are (28 ragged up to 128 under a bound of 256, one query head: 10.1, cut 13.4, the second launch; 32 up to 130 under
    // 272: 16.8 and 17.5), and so do more than 320 items (48 ragged up to 600 25.9 and 28.2).  At most 448 partitions, more cost
    // the merge too much: 2 x 32768 tokens, one kv head 22.4 with 256 a partition, 23.1 with 64 (512 of them), 20.9 with 128; 1 x 65536
    // 24.0, with 64 29.1.  Not in the fixed plan, whose scratch every call has to bring.
    if (kv16 && !fixed && !valu16 && units > 5 && items <= kFineItems16) {
      int64_t finer = kFineWaves / items < units ? kFineWaves / items : units;
      if (finer > kFine16) finer = kFine16;
      if (2 * finer >= units && s < finer) s = finer;
    }
    if (!kv16 && items >= 512 && B <= 1024) s = 1;
    // Very many partitions (a single long sequence): a quarter of them, each shared by four wavefronts
    // that fold their states in LDS, leaves the merge pass a quarter of the partial records to write
    // and read - as long as every wavefront keeps its 512 tokens (131072 tokens x 8 kv heads: 256
    // partitions 40.0 us, 64 partitions of four wavefronts 37.8 us).
    if (!kv16 && s > 64 && units / (s / 4) >= 32) s /= 4;
    // Small batches of short contexts: ONE block of eight wavefronts per (sequence, kv head) - a compute
    // unit's worth, the wavefronts taking every eighth 64-token batch and folding their states in LDS -
    // covers the whole sequence, so the call is a single launch without partial results in memory and
    // without a merge pass (with a fused append: the whole decode step in one launch).  It pays while
    // every wavefront has at most five batches, or eight when the blocks fill most of the chip
    // (32 sequences x 8 kv heads x 2304 tokens: 26.0 -> 21.8 us, x 4096 tokens: 35.0 -> 31.7 us;
    // 16 x 1024: 20.7 -> 18.0 us; 4 x 2304: 20.5 -> 18.8 us; with longer contexts or fewer blocks the
    // partitions win: 16 x 4096: 23.6 against 27.2 us, 1 x 8192: 20.3 against 42.4 us).
    const int64_t per_wave = (units + 7) / 8;
    const bool matrix_core_shape = c->head_dim == 128 || c->n_kv_heads % 2 == 0;
    if (!kv16 && matrix_core_shape && items <= 256 && (per_wave <= 5 || (items >= 192 && per_wave <= 8))) {
      s = 1;
      block_of_eight = true;
    }
    // A single sequence, which is not cut by its length, takes partitions of 64 or 128 tokens as well (fixed plan as above) up to 8192
    // tokens and 16 items (8 kv heads, decode, four query heads each, us: 2600 tokens 14.2 with 256 a partition, 11.6 with 64, 8000
    // 14.5 and 13.3; 12000 15.6 and 16.0, 28000 17.2 and 19.3, the merge of so many records; 32 items x 3300, eight query heads,
    // 16.7 and 18.0).  With the learned rotation up to 896 wavefronts of them, because each multiplies the query by all of R_l (eight
    // query heads: 8 kv heads x 6000 tokens, 752 wavefronts, 25.1 and 24.0; x 8100, 1016, 24.8 and 26.6; 16 x 6000, 1504, 26.5 and 28.5).
    if (!kv16 && !fixed && B == 1 && !block_of_eight && units <= kFineUnits4 && items <= kFineItems4) {
      const int64_t most = (c->dense_rot ? kFineWaves / 2 : kFineWaves) / items;
      const int64_t finer = most < units ? most : units;
      if (2 * finer >= units && s < finer) s = finer;
    }
    if (s < 1) s = 1;
    if (s > kMaxSplits) s = kMaxSplits;
    S = (int)s;
  }
  if (S > units) S = units;
  if (S < 1) S = 1;
  const int chunk_units = (units + S - 1) / S;
  plan->chunk_tokens = chunk_units * 64;
  plan->num_splits = (units + chunk_units - 1) / chunk_units;
  plan->bound = bound;
  // wavefronts per partition: only when the partitions alone cannot fill the chip (about 2560
  // wavefront slots), and while every wavefront keeps at least 8 batches (512 tokens) of its own
  const int64_t blocks = (int64_t)B * decode_items_per_seq(c->head_dim, c->n_kv_heads) * plan->num_splits;
  int nw = 1;
  while (nw < 4 && blocks * nw * 2 <= 2560 && plan->chunk_tokens / (nw * 2) >= 512) nw *= 2;
  // (INT4, a whole sequence in one partition: whole_waves; single 64-channel heads, where the chip holds 3072 wavefronts: four while all of
  // those fit - 66 x 8, eight query heads x 700 tokens 21.9 and 18.7 us, but 250 x 8 x 200 18 and 27, x 700 34 and 44)
  const bool single64 = !kv16 && c->head_dim == 64 && !decode_head_pairs(64, c->n_kv_heads, G);
  if (!kv16 && plan->num_splits == 1) {
    const int64_t heads = (int64_t)B * c->n_kv_heads;
    if (block_of_eight) nw = 8;
    else if (!single64) nw = B <= 1024 ? whole_waves(blocks, c->head_dim == 64 ? 2 * G : G, units, nw) : nw;
    else if (heads > 256 && heads <= 768) nw = 4;
  }
  plan->waves_per_item = nw;
  plan->cut = plan->cut_min = plan->cut_waves = 0;
  plan->valu16 = valu16;
  if (num_splits != 0 || fixed || valu16) return true;
  const int per_seq = kv16 ? c->n_kv_heads : decode_items_per_seq(c->head_dim, c->n_kv_heads);
  if (single64) plan_split64(c, B, G, units, plan);
  // (partitions of 256 tokens are the shortest a cut makes: fixed ones that are no longer have the shorter start - 8 ragged up to 8000
  // tokens, 32 query / 8 kv heads, 42 us, 49 cut; above that 40 ragged up to 8000 161 and 131)
  else if (kv16) { if (plan->num_splits > 1 && chunk_units > 4) cut_plan(B, units, 2048 / per_seq, 1, plan); }
  else plan_cut(B, units, per_seq, G, c->head_dim == 64, c->dense_rot != nullptr, plan);
  return true;
}

}  // namespace saw

using namespace saw;

extern "C" {

int saw_version(void) { return SAW_VERSION; }

const char* saw_strerror(int code) {
  switch (code) {
    case SAW_OK: return "ok";
    case SAW_EINVAL: return "invalid argument (shape, Hadamard block, dtype, stride or alignment)";
    case SAW_ENULL: return "null pointer";
    case SAW_EWORKSPACE: return "workspace too small";
    case SAW_ELAUNCH: return "kernel launch failed";
    case SAW_ESCRATCH: return "the split-KV partial results of this call exceed the static scratch of the no-allocation entry point";
    default: return "unknown error";
  }
}

size_t saw_dense_rotation_bytes(int32_t head_dim) { return head_dim == kDenseD ? kDenseBytes : 0; }

int saw_prepare_dense_rotation(const float* R, int32_t head_dim, void* prepared, size_t prepared_bytes,
                               saw_stream_t stream) {
  if (!R || !prepared) return SAW_ENULL;
  if (head_dim != kDenseD || prepared_bytes < kDenseBytes || !aligned16(R) || !aligned16(prepared)) return SAW_EINVAL;
  return launch_prepare_dense(R, prepared, (hipStream_t)stream);
}

int saw_rotate_quant_store(const saw_cache_t* c, const void* K, const void* V, int32_t in_dtype,
                           int64_t T, int64_t token_stride_elems, const int32_t* page_table,
                           int32_t n_seqs, int32_t max_pages_per_seq, const int32_t* slots,
                           saw_stream_t stream) {
  if (!c) return SAW_ENULL;
  if (!shape_ok(c) || !block_ok(c)) return SAW_EINVAL;
  if (in_dtype != SAW_F16 && in_dtype != SAW_BF16) return SAW_EINVAL;
  if (T < 0 || n_seqs < 1 || max_pages_per_seq < 1) return SAW_EINVAL;
  if (T == 0) return SAW_OK;
  if (!c->k_codes || !c->v_codes || !c->k_meta || !c->v_meta || !K || !V || !page_table || !slots)
    return SAW_ENULL;
  if (token_stride_elems < (int64_t)c->n_kv_heads * c->head_dim || (token_stride_elems & 7)) return SAW_EINVAL;
  if (!aligned16(K) || !aligned16(V) || !aligned16(c->k_codes) || !aligned16(c->v_codes) ||
      (((uintptr_t)c->k_meta) & 7u) || (((uintptr_t)c->v_meta) & 7u) || (((uintptr_t)slots) & 7u))
    return SAW_EINVAL;
  return launch_store_layers(c, &K, &V, 1, in_dtype, T, token_stride_elems, page_table, n_seqs, max_pages_per_seq,
                             slots, (hipStream_t)stream);
}

int saw_rotate_quant_store_layers(const saw_cache_t* caches, const void* const* K, const void* const* V,
                                  int32_t n_layers, int32_t in_dtype, int64_t T, int64_t token_stride_elems,
                                  const int32_t* page_table, int32_t n_seqs, int32_t max_pages_per_seq,
                                  const int32_t* slots, saw_stream_t stream) {
  if (!caches || !K || !V) return SAW_ENULL;
  if (n_layers < 1) return SAW_EINVAL;
  if (in_dtype != SAW_F16 && in_dtype != SAW_BF16) return SAW_EINVAL;
  if (T < 0 || n_seqs < 1 || max_pages_per_seq < 1) return SAW_EINVAL;
  const saw_cache_t* c0 = caches;
  if (!shape_ok(c0) || !block_ok(c0)) return SAW_EINVAL;
  if (token_stride_elems < (int64_t)c0->n_kv_heads * c0->head_dim || (token_stride_elems & 7)) return SAW_EINVAL;
  if (!page_table || !slots) return T == 0 ? SAW_OK : SAW_ENULL;
  if (((uintptr_t)slots) & 7u) return SAW_EINVAL;
  for (int l = 0; l < n_layers; ++l) {
    const saw_cache_t* c = caches + l;
    // one launch, one shape: the layers of a model agree in everything but their pools, inputs and learned rotation
    if (c->num_pages != c0->num_pages || c->n_kv_heads != c0->n_kv_heads || c->page_size != c0->page_size ||
        c->head_dim != c0->head_dim || c->had_block != c0->had_block || c->rotate_mask != c0->rotate_mask ||
        c->sign_bits[0] != c0->sign_bits[0] || c->sign_bits[1] != c0->sign_bits[1] ||
        c->sign_bits[2] != c0->sign_bits[2] || c->sign_bits[3] != c0->sign_bits[3] ||
        (c->dense_rot != nullptr) != (c0->dense_rot != nullptr))
      return SAW_EINVAL;
    if (!block_ok(c)) return SAW_EINVAL;
    if (T == 0) continue;
    if (!c->k_codes || !c->v_codes || !c->k_meta || !c->v_meta || !K[l] || !V[l]) return SAW_ENULL;
    if (!aligned16(K[l]) || !aligned16(V[l]) || !aligned16(c->k_codes) || !aligned16(c->v_codes) ||
        (((uintptr_t)c->k_meta) & 7u) || (((uintptr_t)c->v_meta) & 7u))
      return SAW_EINVAL;
  }
  if (T == 0) return SAW_OK;
  for (int l0 = 0; l0 < n_layers; l0 += SAW_MAX_STORE_LAYERS) {       // 32 layers per launch
    const int n = n_layers - l0 < SAW_MAX_STORE_LAYERS ? n_layers - l0 : SAW_MAX_STORE_LAYERS;
    const int rc = launch_store_layers(caches + l0, K + l0, V + l0, n, in_dtype, T, token_stride_elems, page_table,
                                       n_seqs, max_pages_per_seq, slots, (hipStream_t)stream);
    if (rc != SAW_OK) return rc;
  }
  return SAW_OK;
}

int saw_read_probe(const saw_cache_t* c, const int32_t* page_ids, int64_t n_pages, void* sink, size_t sink_bytes,
                   saw_stream_t stream) {
  if (!c) return SAW_ENULL;
  if (!shape_ok(c) || c->head_dim != 128 || n_pages < 1) return SAW_EINVAL;
  if (!c->k_codes || !c->v_codes || !c->k_meta || !c->v_meta || !page_ids || !sink) return SAW_ENULL;
  if (!aligned16(c->k_codes) || !aligned16(c->v_codes) || !aligned16(c->k_meta) || !aligned16(c->v_meta)) return SAW_EINVAL;
  const int32_t n_waves = (2048 / c->n_kv_heads) * c->n_kv_heads;       // as many as the chip holds of the decode kernel
  if (n_waves < c->n_kv_heads || sink_bytes < (size_t)n_waves * 4) return SAW_EINVAL;
  return launch_read_probe(c, page_ids, n_pages, sink, n_waves, (hipStream_t)stream);
}

int saw_plain_quant_store_valu(const saw_cache_t* c, const void* K, const void* V, int32_t in_dtype, int64_t T,
                               int64_t token_stride_elems, const int32_t* page_table, int32_t n_seqs,
                               int32_t max_pages_per_seq, const int32_t* slots, saw_stream_t stream) {
  if (!c) return SAW_ENULL;
  if (!shape_ok(c) || c->head_dim != 128) return SAW_EINVAL;
  if (in_dtype != SAW_F16 && in_dtype != SAW_BF16) return SAW_EINVAL;
  if (T < 0 || n_seqs < 1 || max_pages_per_seq < 1) return SAW_EINVAL;
  if (T == 0) return SAW_OK;
  if (!c->k_codes || !c->v_codes || !c->k_meta || !c->v_meta || !K || !V || !page_table || !slots) return SAW_ENULL;
  if (token_stride_elems < (int64_t)c->n_kv_heads * c->head_dim || (token_stride_elems & 7)) return SAW_EINVAL;
  if (!aligned16(K) || !aligned16(V) || !aligned16(c->k_codes) || !aligned16(c->v_codes) ||
      (((uintptr_t)c->k_meta) & 7u) || (((uintptr_t)c->v_meta) & 7u) || (((uintptr_t)slots) & 7u))
    return SAW_EINVAL;
  return launch_plain_store_valu(c, K, V, in_dtype, T, token_stride_elems, page_table, n_seqs, max_pages_per_seq, slots,
                                 (hipStream_t)stream);
}

size_t saw_decode_workspace_bytes(const saw_cache_t* c, int32_t B, int32_t n_q_heads,
                                  int32_t max_seq_len, int32_t num_splits) {
  if (!c || !shape_ok(c) || B < 1 || n_q_heads < 1 || max_seq_len < 1) return 0;
  SplitPlan plan;
  const int max_pages = (max_seq_len + c->page_size - 1) / c->page_size;
  // (the INT4 and the 16-bit calls may choose different partition counts, and either may take its fixed partitions: enough for all)
  const int G = n_q_heads % c->n_kv_heads ? 0 : n_q_heads / c->n_kv_heads;
  size_t most = 0;
  for (int k = 0; k < 4; ++k) {
    const bool fixed = G == 0 || (k & 1);
    if (!make_plan(c, B, G, fixed, max_pages, max_seq_len, num_splits, (k & 2) != 0, &plan)) return 0;
    const size_t n = plan_bytes(plan, B, n_q_heads, c->head_dim);
    if (n > most) most = n;
  }
  if (num_splits == 0) {
    // ... and the partitions of 64 or 128 tokens of calls with fewer sequences or a shorter bound, so that a program that sizes its
    // scratch once, for the largest call, gets them there (as many as make_plan ever takes)
    const int64_t units = ((int64_t)max_seq_len + 63) / 64;
    const int per_seq = decode_items_per_seq(c->head_dim, c->n_kv_heads);
    int64_t records = 0;
    if (units > 5 && c->n_kv_heads <= kFineItems16 && !(c->head_dim == 64 && G == 1)) {
      records = B * (units < kFine16 ? units : kFine16);
      if (records > kFineWaves / c->n_kv_heads) records = kFineWaves / c->n_kv_heads;
    }
    if (per_seq <= kFineItems4) {
      const int64_t one = units < kFineUnits4 ? units : kFineUnits4;
      const int64_t r = one < kFineWaves / per_seq ? one : kFineWaves / per_seq;
      if (units > 40 && r > records) records = r;
    }
    const size_t n = partial_bytes(1, n_q_heads, (int)records, c->head_dim);
    if (n > most) most = n;
  }
  return most;
}

int saw_decode_plan(const saw_cache_t* c, int32_t B, int32_t max_seq_len, int32_t num_splits,
                    int32_t* splits_out, int32_t* chunk_tokens_out) {
  if (!c) return SAW_ENULL;
  if (!shape_ok(c) || B < 1 || max_seq_len < 1) return SAW_EINVAL;
  SplitPlan plan;
  const int max_pages = (max_seq_len + c->page_size - 1) / c->page_size;
  if (!make_plan(c, B, 0, true, max_pages, max_seq_len, num_splits, false, &plan)) return SAW_EINVAL;
  if (splits_out) *splits_out = plan.num_splits;
  if (chunk_tokens_out) *chunk_tokens_out = plan.chunk_tokens;
  return SAW_OK;
}

int saw_decode_schedule(const saw_cache_t* c, int32_t B, int32_t n_q_heads, int32_t max_seq_len, int32_t num_splits, int32_t cache16,
                        int32_t with_order, saw_decode_schedule_t* out) {
  if (!c || !out) return SAW_ENULL;
  if (!shape_ok(c) || B < 1 || B > 65535 || c->n_kv_heads > 65535 || max_seq_len < 1 || n_q_heads < 1 || n_q_heads % c->n_kv_heads)
    return SAW_EINVAL;
  const int G = n_q_heads / c->n_kv_heads;
  if (!(G == 1 || G == 2 || G == 4 || G == 8)) return SAW_EINVAL;
  const bool kv16 = cache16 != 0;
  SplitPlan plan;
  if (!make_plan(c, B, G, false, (max_seq_len + c->page_size - 1) / c->page_size, max_seq_len, num_splits, kv16, &plan)) return SAW_EINVAL;
  const BlockPlan blocks = plan_blocks(c, kv16, B, G, plan, with_order && !kv16);
  out->partitions = plan.cut ? 0 : plan.num_splits;
  out->slots = plan.cut;
  // (the 16-bit kernels' blocks are of one wavefront, or two in pair mode; the one for single 64-channel heads has no block of two)
  const int nw = plan.cut ? plan.cut_waves : plan.waves_per_item;
  const bool single64 = !kv16 && c->head_dim == 64 && !decode_head_pairs(64, c->n_kv_heads, G);
  out->waves = blocks.pair ? blocks.pair : kv16 ? 1 : single64 && nw == 2 ? 4 : nw;
  out->pair_seqs = blocks.pair ? blocks.pair_seqs : 0;
  out->longest_first = blocks.sorted;
  return SAW_OK;
}

int saw_decode_rank_order(const int32_t* seq_lens_host, int32_t B, int32_t max_seq_len, int32_t* order_out) {
  if (!seq_lens_host || !order_out) return SAW_ENULL;
  if (B < 1 || B > 1024) return SAW_EINVAL;
  const int bound = max_seq_len <= 0 ? 0x7fffffff : max_seq_len;
  int nbmax = 0;
  int cls[1024];
  for (int b = 0; b < B; ++b) {
    const int len = seq_lens_host[b] < 0 ? 0 : (seq_lens_host[b] > bound ? bound : seq_lens_host[b]);
    cls[b] = len;
    const int nb = (int)(((int64_t)len + 63) >> 6);
    if (nb > nbmax) nbmax = nb;
  }
  const float kscale = rank_scale(nbmax);
  for (int b = 0; b < B; ++b) cls[b] = rank_class(cls[b], kscale);
  int n = 0;
  for (int c = 0; c < 64; ++c)                       // class 0 first; inside a class by sequence index
    for (int b = 0; b < B; ++b)
      if (cls[b] == c) order_out[n++] = b;
  return SAW_OK;
}

int saw_decode_order(const int32_t* seq_lens, int32_t B, int32_t max_seq_len, int32_t* order_out, saw_stream_t stream) {
  if (!seq_lens || !order_out) return SAW_ENULL;
  if (B < 1 || B > 1024) return SAW_EINVAL;
  return launch_decode_order(seq_lens, B, max_seq_len <= 0 ? 0x7fffffff : max_seq_len, order_out, (hipStream_t)stream);
}

// The plan of one call.  What the fixed partitions need is what a call has to bring; what the plan for these shapes needs
// beyond that it gets from a workspace sized by saw_decode_workspace_bytes, and a smaller one gets the fixed partitions.
static int plan_call(const saw_cache_t* c, int B, int Hq, int max_pages, int max_seq_len, int num_splits, bool kv16,
                     size_t ws_bytes, SplitPlan* plan) {
  const int G = Hq % c->n_kv_heads ? 0 : Hq / c->n_kv_heads;
  SplitPlan fixed;
  if (!make_plan(c, B, G, true, max_pages, max_seq_len, num_splits, kv16, &fixed) ||
      !make_plan(c, B, G, G == 0, max_pages, max_seq_len, num_splits, kv16, plan))
    return SAW_EINVAL;
  if (ws_bytes < plan_bytes(fixed, B, Hq, c->head_dim)) return SAW_EWORKSPACE;
  if (ws_bytes < plan_bytes(*plan, B, Hq, c->head_dim)) *plan = fixed;
  return SAW_OK;
}

static int decode_common(const saw_cache_t* c, bool kv16, const void* kp, const void* vp, int kv_dtype,
                         const void* q, int32_t q_dtype, int32_t B, int32_t Hq, const int32_t* pt,
                         int32_t max_pages, const int32_t* seq_lens, int32_t max_seq_len, float sm_scale,
                         void* out, int32_t out_dtype, void* ws, size_t ws_bytes, int32_t num_splits,
                         const saw_decode_hints_t* hints, saw_stream_t stream) {
  if (!c) return SAW_ENULL;
  if (!shape_ok(c)) return SAW_EINVAL;
  if (!kv16 && !block_ok(c)) return SAW_EINVAL;
  if (kv16 && kv_dtype != SAW_F16 && kv_dtype != SAW_BF16) return SAW_EINVAL;
  if (q_dtype != SAW_F16 && q_dtype != SAW_BF16 && q_dtype != SAW_F32) return SAW_EINVAL;
  if (out_dtype != SAW_F16 && out_dtype != SAW_BF16 && out_dtype != SAW_F32) return SAW_EINVAL;
  if (B < 1 || Hq < 1 || max_pages < 1) return SAW_EINVAL;
  if (B > 65535 || c->n_kv_heads > 65535) return SAW_EINVAL;
  if (Hq % c->n_kv_heads) return SAW_EINVAL;
  const int G = Hq / c->n_kv_heads;
  if (!(G == 1 || G == 2 || G == 4 || G == 8)) return SAW_EINVAL;
  if (!kp || !vp || !q || !pt || !seq_lens || !out || !ws) return SAW_ENULL;
  if (!kv16 && (!c->k_meta || !c->v_meta)) return SAW_ENULL;
  if (!aligned16(kp) || !aligned16(vp) || !aligned16(ws) || !aligned16(out)) return SAW_EINVAL;
  // (the INT4 kernels fetch the (scale, zero) pairs with 16-byte transfers)
  if (!kv16 && (!aligned16(c->k_meta) || !aligned16(c->v_meta))) return SAW_EINVAL;
  if (!isfinite(sm_scale)) return SAW_EINVAL;
  SplitPlan plan;
  const int rc = plan_call(c, B, Hq, max_pages, max_seq_len, num_splits, kv16, ws_bytes, &plan);
  if (rc != SAW_OK) return rc;
  return run_decode(c, kv16, kp, vp, kv_dtype, q, q_dtype, B, Hq, pt, max_pages, seq_lens, sm_scale, out,
                    out_dtype, ws, plan, nullptr, nullptr, 0, hints ? hints->order : nullptr, (hipStream_t)stream);
}

int saw_paged_decode_attn(const saw_cache_t* c, const void* q, int32_t q_dtype, int32_t B,
                          int32_t n_q_heads, const int32_t* page_table, int32_t max_pages_per_seq,
                          const int32_t* seq_lens, int32_t max_seq_len, float sm_scale, void* out,
                          int32_t out_dtype, void* workspace, size_t workspace_bytes,
                          int32_t num_splits, saw_stream_t stream) {
  if (!c) return SAW_ENULL;
  return decode_common(c, false, c->k_codes, c->v_codes, 0, q, q_dtype, B, n_q_heads, page_table,
                       max_pages_per_seq, seq_lens, max_seq_len, sm_scale, out, out_dtype, workspace,
                       workspace_bytes, num_splits, nullptr, stream);
}

int saw_paged_decode_attn_hinted(const saw_cache_t* c, const void* q, int32_t q_dtype, int32_t B,
                                 int32_t n_q_heads, const int32_t* page_table, int32_t max_pages_per_seq,
                                 const int32_t* seq_lens, int32_t max_seq_len, float sm_scale, void* out,
                                 int32_t out_dtype, void* workspace, size_t workspace_bytes,
                                 int32_t num_splits, const saw_decode_hints_t* hints, saw_stream_t stream) {
  if (!c) return SAW_ENULL;
  return decode_common(c, false, c->k_codes, c->v_codes, 0, q, q_dtype, B, n_q_heads, page_table,
                       max_pages_per_seq, seq_lens, max_seq_len, sm_scale, out, out_dtype, workspace,
                       workspace_bytes, num_splits, hints, stream);
}

// The device address of `scratch` on the current device, resolved once per device with that device
// current (every GPU holds its own copy of the array at its own address).
static int static_scratch_ptr(void** out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* ptrs[kMaxDevices] = {nullptr};
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SAW_ELAUNCH;
  std::lock_guard<std::mutex> lock(mu);
  if (!ptrs[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return SAW_ELAUNCH;
    ptrs[dev] = p;
  }
  *out = ptrs[dev];
  return SAW_OK;
}

int saw_paged_decode_attn_static(const saw_cache_t* c, const void* q, int32_t q_dtype, int32_t B,
                                 int32_t n_q_heads, const int32_t* page_table, int32_t max_pages_per_seq,
                                 const int32_t* seq_lens, int32_t max_seq_len, float sm_scale, void* out,
                                 int32_t out_dtype, int32_t num_splits, saw_stream_t stream) {
  if (!c) return SAW_ENULL;
  if (!shape_ok(c) || B < 1 || n_q_heads < 1 || max_pages_per_seq < 1) return SAW_EINVAL;
  // the scratch the plan needs, before anything else: too large is an error of its own
  SplitPlan plan;
  int rc = plan_call(c, B, n_q_heads, max_pages_per_seq, max_seq_len, num_splits, false, (size_t)SAW_STATIC_SCRATCH_BYTES, &plan);
  if (rc != SAW_OK) return rc == SAW_EWORKSPACE ? SAW_ESCRATCH : rc;
  void* ws = nullptr;
  rc = static_scratch_ptr(&ws);
  if (rc != SAW_OK) return rc;
  // (nothing in the scratch has to start at zero: every partial record the merge pass reads was
  // written by the decode pass of the same call)
  return decode_common(c, false, c->k_codes, c->v_codes, 0, q, q_dtype, B, n_q_heads, page_table,
                       max_pages_per_seq, seq_lens, max_seq_len, sm_scale, out, out_dtype, ws,
                       (size_t)SAW_STATIC_SCRATCH_BYTES, num_splits, nullptr, stream);
}

static int append_common(const saw_cache_t* c, const void* K_new, const void* V_new, int32_t kv_dtype,
                         const void* q, int32_t q_dtype, int32_t B, int32_t Hq,
                         const int32_t* page_table, int32_t max_pages, const int32_t* seq_lens,
                         int32_t max_seq_len, float sm_scale, void* out, int32_t out_dtype,
                         void* ws, size_t ws_bytes, const saw_decode_hints_t* hints, saw_stream_t stream) {
  if (!c) return SAW_ENULL;
  if (!shape_ok(c) || !block_ok(c)) return SAW_EINVAL;
  if (kv_dtype != SAW_F16 && kv_dtype != SAW_BF16) return SAW_EINVAL;
  if (q_dtype != SAW_F16 && q_dtype != SAW_BF16 && q_dtype != SAW_F32) return SAW_EINVAL;
  if (out_dtype != SAW_F16 && out_dtype != SAW_BF16 && out_dtype != SAW_F32) return SAW_EINVAL;
  if (B < 1 || Hq < 1 || max_pages < 1 || B > 65535 || c->n_kv_heads > 65535) return SAW_EINVAL;
  if (Hq % c->n_kv_heads) return SAW_EINVAL;
  const int G = Hq / c->n_kv_heads;
  if (!(G == 1 || G == 2 || G == 4 || G == 8)) return SAW_EINVAL;
  if (!c->k_codes || !c->v_codes || !c->k_meta || !c->v_meta || !K_new || !V_new || !q || !page_table ||
      !seq_lens || !out || !ws)
    return SAW_ENULL;
  if (!aligned16(K_new) || !aligned16(V_new) || !aligned16(c->k_codes) || !aligned16(c->v_codes) ||
      !aligned16(ws) || !aligned16(out) || !aligned16(c->k_meta) || !aligned16(c->v_meta))
    return SAW_EINVAL;
  if (!isfinite(sm_scale) || max_seq_len < 0) return SAW_EINVAL;
  // the plan covers the lengths after the append (max_seq_len + 1 tokens)
  const int64_t cap = (int64_t)max_pages * c->page_size;
  const int64_t after = (max_seq_len <= 0 ? cap - 1 : (int64_t)max_seq_len) + 1;
  if (after > cap) return SAW_EINVAL;
  SplitPlan plan;
  const int rc = plan_call(c, B, Hq, max_pages, (int)after, 0, false, ws_bytes, &plan);
  if (rc != SAW_OK) return rc;
  // the decode kernel stores the new token itself and attends to it from on-chip memory (with several
  // partitions per sequence one of them does, and the merge kernel follows);
  // the cached range is [0, seq_lens[b]), bounded by max_seq_len as given
  plan.bound = (int)(after - 1);
  return run_decode(c, false, c->k_codes, c->v_codes, 0, q, q_dtype, B, Hq, page_table, max_pages, seq_lens,
                    sm_scale, out, out_dtype, ws, plan, K_new, V_new, kv_dtype, hints ? hints->order : nullptr,
                    (hipStream_t)stream);
}

int saw_append_decode_attn(const saw_cache_t* c, const void* K_new, const void* V_new, int32_t kv_dtype,
                           const void* q, int32_t q_dtype, int32_t B, int32_t Hq,
                           const int32_t* page_table, int32_t max_pages, const int32_t* seq_lens,
                           int32_t max_seq_len, float sm_scale, void* out, int32_t out_dtype,
                           void* ws, size_t ws_bytes, saw_stream_t stream) {
  return append_common(c, K_new, V_new, kv_dtype, q, q_dtype, B, Hq, page_table, max_pages, seq_lens, max_seq_len,
                       sm_scale, out, out_dtype, ws, ws_bytes, nullptr, stream);
}

int saw_append_decode_attn_hinted(const saw_cache_t* c, const void* K_new, const void* V_new, int32_t kv_dtype,
                                  const void* q, int32_t q_dtype, int32_t B, int32_t Hq,
                                  const int32_t* page_table, int32_t max_pages, const int32_t* seq_lens,
                                  int32_t max_seq_len, float sm_scale, void* out, int32_t out_dtype,
                                  void* ws, size_t ws_bytes, const saw_decode_hints_t* hints, saw_stream_t stream) {
  return append_common(c, K_new, V_new, kv_dtype, q, q_dtype, B, Hq, page_table, max_pages, seq_lens, max_seq_len,
                       sm_scale, out, out_dtype, ws, ws_bytes, hints, stream);
}

int saw_dequant_pages(const saw_cache_t* c, const int32_t* page_table, int32_t max_pages_per_seq,
                      int32_t seq, int32_t pos_begin, int32_t pos_end, int32_t unrotate, float* k_out,
                      float* v_out, saw_stream_t stream) {
  if (!c) return SAW_ENULL;
  if (!shape_ok(c) || !block_ok(c)) return SAW_EINVAL;
  if (seq < 0 || pos_begin < 0 || pos_end < pos_begin || max_pages_per_seq < 1) return SAW_EINVAL;
  if ((int64_t)pos_end > (int64_t)max_pages_per_seq * c->page_size) return SAW_EINVAL;
  if (pos_end == pos_begin) return SAW_OK;
  if (!c->k_codes || !c->v_codes || !c->k_meta || !c->v_meta || !page_table) return SAW_ENULL;
  if (!k_out && !v_out) return SAW_OK;
  if ((k_out && !aligned16(k_out)) || (v_out && !aligned16(v_out))) return SAW_EINVAL;
  return launch_dequant(c, page_table, max_pages_per_seq, seq, pos_begin, pos_end, unrotate, k_out, v_out,
                        (hipStream_t)stream);
}

int saw_flatten_dequant(const saw_cache_t* c, const int32_t* page_table, int32_t max_pages_per_seq,
                        int32_t seq, int32_t pos_begin, int32_t pos_end, int32_t unrotate,
                        int32_t out_dtype, void* k_out, void* v_out, int64_t token_stride_elems,
                        saw_stream_t stream) {
  if (!c) return SAW_ENULL;
  if (!shape_ok(c) || !block_ok(c)) return SAW_EINVAL;
  if (out_dtype != SAW_F16 && out_dtype != SAW_BF16 && out_dtype != SAW_F32) return SAW_EINVAL;
  if (seq < 0 || pos_begin < 0 || pos_end < pos_begin || max_pages_per_seq < 1) return SAW_EINVAL;
  if ((int64_t)pos_end > (int64_t)max_pages_per_seq * c->page_size) return SAW_EINVAL;
  if (token_stride_elems < (int64_t)c->n_kv_heads * c->head_dim || (token_stride_elems % 8)) return SAW_EINVAL;
  if (unrotate && c->dense_rot && (c->rotate_mask & (SAW_ROT_K | SAW_ROT_V))) return SAW_EINVAL;   // not built here
  if (pos_end == pos_begin) return SAW_OK;
  if (!c->k_codes || !c->v_codes || !c->k_meta || !c->v_meta || !page_table) return SAW_ENULL;
  if (!k_out && !v_out) return SAW_OK;
  if ((k_out && !aligned16(k_out)) || (v_out && !aligned16(v_out))) return SAW_EINVAL;
  return launch_flatten(c, page_table + (int64_t)seq * max_pages_per_seq, pos_begin, pos_end, unrotate,
                        out_dtype, k_out, v_out, token_stride_elems, (hipStream_t)stream);
}

int saw_kv16_store(const saw_cache_t* c, void* k_pages, void* v_pages, int32_t dtype, const void* K,
                   const void* V, int64_t T, int64_t token_stride_elems, const int32_t* page_table,
                   int32_t n_seqs, int32_t max_pages_per_seq, const int32_t* slots, saw_stream_t stream) {
  if (!c) return SAW_ENULL;
  if (!shape_ok(c)) return SAW_EINVAL;
  if (dtype != SAW_F16 && dtype != SAW_BF16) return SAW_EINVAL;
  if (T < 0 || n_seqs < 1 || max_pages_per_seq < 1) return SAW_EINVAL;
  if (T == 0) return SAW_OK;
  if (!k_pages || !v_pages || !K || !V || !page_table || !slots) return SAW_ENULL;
  if (token_stride_elems < (int64_t)c->n_kv_heads * c->head_dim || (token_stride_elems & 7)) return SAW_EINVAL;
  if (!aligned16(K) || !aligned16(V) || !aligned16(k_pages) || !aligned16(v_pages)) return SAW_EINVAL;
  return launch_kv16_store(c, k_pages, v_pages, K, V, T, token_stride_elems, page_table, n_seqs,
                           max_pages_per_seq, slots, (hipStream_t)stream);
}

int saw_kv16_paged_decode_attn(const saw_cache_t* c, const void* k_pages, const void* v_pages,
                               int32_t dtype, const void* q, int32_t q_dtype, int32_t B,
                               int32_t n_q_heads, const int32_t* page_table, int32_t max_pages_per_seq,
                               const int32_t* seq_lens, int32_t max_seq_len, float sm_scale, void* out,
                               int32_t out_dtype, void* workspace, size_t workspace_bytes,
                               int32_t num_splits, saw_stream_t stream) {
  return decode_common(c, true, k_pages, v_pages, dtype, q, q_dtype, B, n_q_heads, page_table,
                       max_pages_per_seq, seq_lens, max_seq_len, sm_scale, out, out_dtype, workspace,
                       workspace_bytes, num_splits, nullptr, stream);
}

}  // extern "C"
