// 16-bit-KV paged decode attention on the gfx950 matrix cores: the unquantised comparison path (the cache the
// paper measures INT4 against, Sec. 2), written with the same machinery as the INT4 kernel so that the
// comparison is between formats, not between efforts.  head_dim 64 and 128, up to eight query heads per kv head.
//
// One wavefront owns one (sequence, kv head, partition) and walks it in batches of 16 KiB of cache: two pages
// (32 tokens) of head_dim 128, four pages (64 tokens) of head_dim 64.  Per batch:
//   * K needs no staging: lane (token = lane % 16, k-group = lane / 16) of the logit MFMA's B
//     operand wants 8 consecutive channels of its token, which is one 16-byte global load, so the
//     eight K operand registers of a batch are loaded straight from HBM one batch ahead;
//   * V is wanted with tokens along the contraction: its page tiles go HBM -> LDS
//     directly (global_load_lds_dwordx4) into a double buffer, 16-byte chunks XOR-swizzled by row so
//     that ds_read_b64_tr_b16 (a 4x16 transpose of 16-bit elements inside each 16-lane group) reads
//     them without bank conflicts and hands each lane 4 tokens of one channel;
//   * logits: D[head][token] = q~ (heads x channels) . K (channels x tokens) with
//     v_mfma_f32_16x16x32, q~ carried as 16-bit limbs in separate rows of the tile;
//   * softmax with a lazily updated reference maximum, P through LDS once as limb rows,
//     O[head][channel] in 16x16 tiles.
// The tile holds the heads' first limbs, then their second limbs (rows 0-3 and 4-7 up to four heads, 0-7 and
// 8-15 for eight).  What bounds the kernel is HBM; the matrix cores are idle most of the time (eight products per
// 16 KiB of cache), so eight heads and head_dim 64 - which ran on the vector ALU before, in fp32 - afford a
// third limb (kThree): a second product per k-step.  A bf16 limb has fp32's exponents, so the third limbs' rows are
// 0.., added into the first limbs' rows, and the three sum to the fp32 value.  An fp16 limb has not: numbers below 2^-14
// lose bits and below 2^-25 everything, while the sum of the weights still counts them in fp32 (one dominant token 25 bits
// above a long tail: a hundredth of the output).  So q~ is brought to 2^13 .. 2^14 per head and P is kept 2^7 higher, both by powers
// of two that cancel exactly, the second and third limbs are held 2^12 times as large, in rows of their own, and what is
// lost of a weight is below 2^-43 of the largest one's.
// An infinity in the cache times a limb that is zero is NaN, where fp32 gives a logit of -inf no weight and hands an infinite
// value on: a range whose sums are not finite is worked out again in fp32 (range_fp32).
// 16 ragged sequences of 4000-12000 tokens, 64 query / 8 kv heads of 128: 433 -> 109 us.
//
// PAIR = true gives this kernel the INT4 kernel's way of evening out a ragged batch when all of it
// is resident at once (one partition per sequence, 257..2048 (sequence, kv head) items): a block
// of two wavefronts owns the sequences at ranks r and B-1-r of the longest-first order and halves
// their batches: wavefront 0 streams the first part of the long sequence, wavefront 1 the
// short sequence and then the rest of the long one; the two leave their shares of the long
// sequence as (max, sum, accumulator) records in LDS, and whichever comes second combines them
// (wavefront 0's first) and writes the output.
#include "saw_decode.h"
#include "saw_wave_util.h"
#include "saw_rank.h"
#include "saw_cut.h"

namespace saw {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef short i16x4 __attribute__((ext_vector_type(4)));

namespace kv16 {

constexpr int kVbufBytes = 8192;               // V of a batch: 32 token rows of 256 bytes, or 64 of 128
constexpr float kLazyTau = 8.0f;
template <int D, int G, int DT>
struct Shape {
  static constexpr int NP = 256 / D;                       // pages per batch
  static constexpr int TB = 16 * NP;                       // tokens per batch
  static constexpr int kRowBytes = 2 * D;                  // one token's head vector
  static constexpr int kPageBytes = 16 * kRowBytes;        // one (page, head) tile
  static constexpr int LO = (G > 4) ? 8 : 4;               // first row of the second limbs
  static constexpr bool kThree = G > 4 || D == 64;
  static constexpr bool kScaled = kThree && DT == SAW_F16; // limbs scaled by powers of two; the third ones in the second ones' rows
  static constexpr int kProw = TB + 8;                     // P row stride in 16-bit elements (8 pad)
  static constexpr int kPbufBytes = (kThree ? 3 : 2) * LO * kProw * 2;
  static constexpr int kWaveLds = 2 * kVbufBytes + kPbufBytes;
};

template <int DT>
__device__ __forceinline__ f32x4 mfma16(u32x4 a, u32x4 b, f32x4 c) {
  if (DT == SAW_BF16)
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// x = hi + lo as two 16-bit values of the cache's type (hi truncated / rounded, lo the rounded rest)
template <int DT>
__device__ __forceinline__ void split16(float x, uint32_t& hi16, uint32_t& lo16) {
  if (DT == SAW_BF16) {
    float sum;
    split_bf16(x, hi16, lo16, sum);
  } else {
    hi16 = f32_to_f16(x);
    lo16 = f32_to_f16(x - f16_to_f32(hi16));
  }
}
// x as three bf16 values whose sum is x exactly (two truncations, eight bits of remainder left)
__device__ __forceinline__ void split16x3(float x, uint32_t& hi16, uint32_t& mid16, uint32_t& lo16) {
  hi16 = __float_as_uint(x) >> 16;
  const float r = x - __uint_as_float(hi16 << 16);
  mid16 = __float_as_uint(r) >> 16;
  lo16 = __float_as_uint(r - __uint_as_float(mid16 << 16)) >> 16;
}

constexpr float kLow = 1.f / 4096.f;           // what the scaled second and third fp16 limbs stand for
// x as three fp16 values: hi + (mid + lo) kLow
__device__ __forceinline__ void split16x3_scaled(float x, uint32_t& hi16, uint32_t& mid16, uint32_t& lo16) {
  hi16 = f32_to_f16(x);
  const float r = (x - f16_to_f32(hi16)) * 4096.f;
  mid16 = f32_to_f16(r);
  lo16 = f32_to_f16(r - f16_to_f32(mid16));
}

// Positions [t_begin, t_end) of one (sequence, kv head) by one wavefront in plain fp32, lane = token for the logits and lane =
// channel for the outputs: rec = un-normalised sums [G][D], then (max, sum) per head.  For caches that hold infinities or NaN.
template <int D, int G, int DT>
__device__ __forceinline__ void range_fp32(const DecodeParams& p, int b, int kvh, int t_begin, int t_end, int lane,
                                                     float* qs, float* rec) {
  constexpr int E = D / 64;
  const int64_t pt_row = (int64_t)b * p.max_pages;
#pragma unroll 1
  for (int h = 0; h < G; ++h) {
#pragma unroll
    for (int e = 0; e < E; ++e)
      qs[lane + 64 * e] = load_elem(p.q, p.q_dtype, ((int64_t)b * p.n_q_heads + kvh * G + h) * D + lane + 64 * e) * p.q_scale;
    wave_sync();
    float m = -INFINITY, l = 0.f, acc[E];
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] = 0.f;
#pragma unroll 1
    for (int t0 = t_begin; t0 < t_end; t0 += 64) {
      const int n = min(64, t_end - t0), t = t0 + min(lane, n - 1);
      int page = p.page_table[pt_row + (t >> 4)];
      page = (page < 0 || page >= p.num_pages) ? 0 : page;
      const uint32_t* const k = (const uint32_t*)(p.k_codes + (((int64_t)page * p.n_kv_heads + kvh) * 16 + (t & 15)) * (2 * D));
      float dot = 0.f;
#pragma unroll 4
      for (int i = 0; i < D / 2; ++i) {
        float lo, hi;
        widen2<DT>(k[i], lo, hi);
        dot = fmaf(qs[2 * i], lo, dot);
        dot = fmaf(qs[2 * i + 1], hi, dot);
      }
      const float lg = lane < n ? dot : -INFINITY;
      const float mnew = fmaxf(m, max_xor32(max_xor16(row_allmax(lg))));
      const float a = m == mnew ? 1.f : fast_exp2(m - mnew);
      const float w = lg == -INFINITY ? 0.f : fast_exp2(lg - mnew);
      l = fmaf(l, a, w);
#pragma unroll
      for (int e = 0; e < E; ++e) acc[e] *= a;
      m = mnew;
#pragma unroll 1
      for (int j = 0; j < n; ++j) {
        const float wj = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(w), j));
        const int64_t row = ((int64_t)__builtin_amdgcn_readlane(page, j) * p.n_kv_heads + kvh) * 16 + ((t0 + j) & 15);
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] = fmaf(wj, load_elem(p.v_codes, DT, row * D + lane + 64 * e), acc[e]);
      }
    }
    l = add_xor32(add_xor16(row_allsum(l)));
#pragma unroll
    for (int e = 0; e < E; ++e) rec[h * D + lane + 64 * e] = acc[e];
    if (lane == 0) { rec[G * D + 2 * h] = m; rec[G * D + 2 * h + 1] = l; }
    wave_sync();
  }
}

}  // namespace kv16

template <int D, int G, int DT, bool PAIR, bool CUT>
__global__ __launch_bounds__(PAIR ? 128 : 64) __attribute__((amdgpu_waves_per_eu(2)))
void decode_kv16_mfma_kernel(DecodeParams p) {
  static_assert(!(PAIR && CUT), "pair blocks deal out whole sequences");
  using namespace kv16;
  using Sh = Shape<D, G, DT>;
  constexpr int NP = Sh::NP, TB = Sh::TB, kRowBytes = Sh::kRowBytes, kPageBytes = Sh::kPageBytes;
  constexpr int LO = Sh::LO, kProw = Sh::kProw, kWaveLds = Sh::kWaveLds;
  constexpr bool kThree = Sh::kThree, kScaled = Sh::kScaled;
  constexpr float kLift = kScaled ? 7.f : 0.f;                 // P is kept 2^kLift higher: at most 2^(kLift + kLazyTau) = 32768
  constexpr int KK = D / 32, CT = D / 16;                      // k-steps of the logits, 16-channel output tiles
  // The softmax layout.  Up to four heads: a lane holds one token of the batch and every head (32-token batches
  // leave lanes 32.. idle).  Eight heads: a lane holds four of them, for one token (32-token batches) or two.
  constexpr int NH = (G > 4) ? 4 : G;
  constexpr int NS = (G > 4 && NP == 4) ? 2 : 1;
  constexpr int NWV = PAIR ? 2 : 1;
  // (the partition index is rotated by kv head and sequence, so that no XCD serves a fixed set of partitions)
  // (a batch cut by its own lengths has one block per slot: see saw_cut.h;
  // there the order is shifted from head to head: the slots that a batch does not fill are the last ones, and with every head's in the
  // same place the blocks that have work meet on a few compute units - nine sequences of 437 tokens and one of 7000, 46 of 256 slots,
  // 42.6 us, 26.5 with the shift)
  const int split = (int)((CUT ? blockIdx.x + 32 * blockIdx.y : blockIdx.x + blockIdx.y + blockIdx.z) % gridDim.x);
  const int kvh = blockIdx.y;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row16 = lane & 15, grp = lane >> 4;
  // (one shared array for everything: see the INT4 kernel on why)
  __shared__ __attribute__((aligned(16))) uint8_t lds_all[NWV * kWaveLds + 16];
  uint8_t* const lds = lds_all + wave * kWaveLds;
  uint8_t* const vbuf_a = lds;
  uint8_t* const vbuf_b = lds + kVbufBytes;
  uint8_t* const pbuf = lds + 2 * kVbufBytes;
  int* const done_cnt = (int*)(lds_all + NWV * kWaveLds);      // PAIR: records left of the long sequence

  // ---- the ranges this wavefront streams ----
  int nseg = 1;
  int sg_b[2] = {(int)blockIdx.z, 0}, sg_t0[2] = {0, 0}, sg_t1[2] = {0, 0};
  bool sg_share[2] = {false, false};
  if (PAIR) {
    const int B = p.batch;
    if (threadIdx.x == 0) done_cnt[0] = 0;
    __syncthreads();
    const LenClasses lc = build_len_classes(p, B, lane, (int*)vbuf_a);
    const int r_long = blockIdx.z, r_short = B - 1 - r_long;
    const bool self = r_long == r_short;                // odd batch: the middle sequence pairs with itself
    const int b_long = seq_of_rank(lane, lc, r_long);
    const int b_short = self ? b_long : seq_of_rank(lane, lc, r_short);
    const int l_long = lc.lens[b_long];
    const int l_short = self ? 0 : lc.lens[b_short];
    const int nb_long = (l_long + TB - 1) / TB, nb_short = (l_short + TB - 1) / TB;
    // wavefront 1 pays a second prologue when the long sequence is shared: two batches in its favour
    const int cut = min(nb_long, (nb_long + nb_short + 2) >> 1);
    const bool shared = cut < nb_long;
    nseg = 0;
    if (wave == 0) {
      if (nb_long == 0) {                               // empty sequence: zero output row
        for (int i = lane; i < G * D; i += 64)
          store_elem(p.out, p.out_dtype, ((int64_t)b_long * p.n_q_heads + kvh * G) * D + i, 0.f);
      } else {
        sg_b[0] = b_long; sg_t0[0] = 0; sg_t1[0] = min(l_long, TB * cut); sg_share[0] = shared;
        nseg = 1;
      }
    } else {
      if (nb_short > 0) {
        sg_b[0] = b_short; sg_t0[0] = 0; sg_t1[0] = l_short; sg_share[0] = false;
        nseg = 1;
      } else if (!self) {
        for (int i = lane; i < G * D; i += 64)
          store_elem(p.out, p.out_dtype, ((int64_t)b_short * p.n_q_heads + kvh * G) * D + i, 0.f);
      }
      if (shared) {                                     // last, so that its record can stay in this wavefront's buffers
        if (nseg == 0) { sg_b[0] = b_long; sg_t0[0] = TB * cut; sg_t1[0] = l_long; sg_share[0] = true; }
        else           { sg_b[1] = b_long; sg_t0[1] = TB * cut; sg_t1[1] = l_long; sg_share[1] = true; }
        ++nseg;
      }
    }
    wave_sync();                                        // the ranking's scratch lived in vbuf_a
  } else if (CUT) {
    const BatchCut cut = cut_batch(p, lane);
    int len, part, parts, first, end;
    cut_slot(cut, split, sg_b[0], len, part, parts);
    if (sg_b[0] < 0) return;
    if (part == 0 && kvh == 0 && lane == 0) p.cut_of[sg_b[0]] = make_int2(split, parts);
    cut_range((len + 63) >> 6, part, parts, first, end);
    sg_t0[0] = 64 * first;
    sg_t1[0] = min(len, 64 * end);
  } else {
    const int L = min(p.seq_lens[sg_b[0]], p.bound);
    sg_t0[0] = split * p.chunk_tokens;
    sg_t1[0] = min(L, sg_t0[0] + p.chunk_tokens);
    if (sg_t0[0] >= sg_t1[0]) {
      if (p.num_splits == 1)
        for (int i = lane; i < G * D; i += 64)
          store_elem(p.out, p.out_dtype, ((int64_t)sg_b[0] * p.n_q_heads + kvh * G) * D + i, 0.f);
      return;
    }
  }

#pragma unroll 1
  for (int seg = 0; seg < nseg; ++seg) {
  const int b = seg == 0 ? sg_b[0] : sg_b[1];
  const int t_begin = seg == 0 ? sg_t0[0] : sg_t0[1];
  const int t_end = seg == 0 ? sg_t1[0] : sg_t1[1];
  const bool share = seg == 0 ? sg_share[0] : sg_share[1];

  const uint8_t* const kpages = p.k_codes;
  const uint8_t* const vpages = p.v_codes;
  const int64_t pt_row = (int64_t)b * p.max_pages;
  const int64_t page_stride = (int64_t)p.n_kv_heads * kPageBytes;
  const int64_t head_off = (int64_t)kvh * kPageBytes;
  const int pg_first = t_begin >> 4;
  const int nb = (t_end - t_begin + TB - 1) / TB;

  // ---- q~ = q sm_scale log2(e) as the logit MFMA's A operand: rows 0.. first limbs, LO.. second limbs;
  // third limbs (kThree) in rows 0.. (kScaled: LO..) of a second operand whose other rows are zero ----
  // An fp16 limb holds at most 65504: a larger q~ is scaled by a power of two first (kScaled: every head is) and the logits
  // scaled back.
  u32x4 a_q[KK], a_q3[kThree ? KK : 1];
  float q_back[kScaled ? NH : 1] = {1.f};
  {
    const bool is_lo = (row16 & LO) != 0;
    const int qhead = row16 & (LO - 1);
    const bool live = row16 < 2 * LO && qhead < G;
    const int64_t qbase = ((int64_t)b * p.n_q_heads + kvh * G + (live ? qhead : 0)) * D;
    float x[KK][8];
    float big = 0.f;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        x[kk][j] = live ? load_elem(p.q, p.q_dtype, qbase + 32 * kk + 8 * grp + j) * p.q_scale : 0.f;
        big = fmaxf(big, fabsf(x[kk][j]));
      }
    if constexpr (kScaled) {
      const float top = max_xor32(max_xor16(big));                      // of this lane's head
      const int e = min(max(14 - __builtin_amdgcn_frexp_expf(top), -100), 100);
#pragma unroll
      for (int i = 0; i < NH; ++i) {
        int of = __builtin_amdgcn_readlane(e, i);                       // (lane i: the first limbs of head i)
        if (G > 4) of = (grp & 1) ? __builtin_amdgcn_readlane(e, 4 + i) : of;
        q_back[i] = __builtin_ldexpf(1.f, -of);
      }
#pragma unroll
      for (int kk = 0; kk < KK; ++kk)
#pragma unroll
        for (int j = 0; j < 8; ++j) x[kk][j] = __builtin_ldexpf(x[kk][j], e);
    } else if (DT == SAW_F16 && __any(big > 32768.f)) {
      const float top = max_xor32(max_xor16(row_allmax(big)));          // the same in every lane
      const int e = min(max(15 - __builtin_amdgcn_frexp_expf(top), -100), 0);
      q_back[0] = __builtin_ldexpf(1.f, -e);
#pragma unroll
      for (int kk = 0; kk < KK; ++kk)
#pragma unroll
        for (int j = 0; j < 8; ++j) x[kk][j] = __builtin_ldexpf(x[kk][j], e);
    }
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      uint32_t limb[8], third[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        uint32_t h16, l16, t16 = 0;
        if (kScaled) split16x3_scaled(x[kk][j], h16, l16, t16);
        else if (kThree) split16x3(x[kk][j], h16, l16, t16);
        else split16<DT>(x[kk][j], h16, l16);
        limb[j] = is_lo ? l16 : h16;
        third[j] = is_lo == kScaled ? t16 : 0u;
      }
      a_q[kk] = u32x4{limb[0] | (limb[1] << 16), limb[2] | (limb[3] << 16), limb[4] | (limb[5] << 16), limb[6] | (limb[7] << 16)};
      if (kThree) a_q3[kk] = u32x4{third[0] | (third[1] << 16), third[2] | (third[3] << 16), third[4] | (third[5] << 16), third[6] | (third[7] << 16)};
    }
  }

  // ---- fetch ----
  // page ids of a batch: lanes 0 .. NP - 1 of `pidv`
  auto load_pids = [&](int batch) {
    const int lp = min(pg_first + NP * batch + (lane & (NP - 1)), p.max_pages - 1);
    const int id = p.page_table[pt_row + lp];
    return (id < 0 || id >= p.num_pages) ? 0 : id;
  };
  // K operand registers of a batch: kreg[page][kk] = channels 32kk + 8grp .. +7 of token row16; V tiles into VDST:
  // a transfer covers 1 KiB of LDS, RT token rows; the lane at chunk position c of row r brings source chunk
  // c ^ v_swz(r).  (All K and V reads are marked streaming, cache policy "nt", as in the INT4 kernel.)
  u32x4 kreg[NP][KK];
  constexpr int RT = 1024 / kRowBytes, CPR = kRowBytes / 16;         // rows per transfer, chunks per row
  const int v_row = lane / CPR;                                      // row inside the transfer
  // (rows of 256 bytes start on the same bank: the swizzle spreads four of them; rows of 128 bytes alternate
  // between two halves of the banks: it spreads the pairs, and two groups of eight rows)
  auto v_swz = [](int r) { return D == 128 ? 2 * (r & 3) : (2 * ((r >> 1) & 1)) ^ (4 * ((r >> 3) & 1)); };
#define KV16_FETCH(pidv, VDST)                                                                   \
  _Pragma("unroll") for (int pg = 0; pg < NP; ++pg) {                                            \
    const int64_t tile = (int64_t)__builtin_amdgcn_readlane(pidv, pg) * page_stride + head_off;  \
    const uint8_t* const k0 = kpages + tile + row16 * kRowBytes + 16 * grp;                      \
    _Pragma("unroll") for (int kk = 0; kk < KK; ++kk)                                            \
      kreg[pg][kk] = __builtin_nontemporal_load((const u32x4*)(k0 + 64 * kk));                   \
    _Pragma("unroll") for (int j = 0; j < 16 / RT; ++j) {                                        \
      const uint8_t* const v0 = vpages + tile + (j * RT + v_row) * kRowBytes + 16 * ((lane & (CPR - 1)) ^ v_swz(j * RT + v_row)); \
      __builtin_amdgcn_global_load_lds((const GLOBAL_AS void*)v0, (LDS_AS void*)(VDST + pg * kPageBytes + j * 1024), 16, 0, 2); \
    }                                                                                            \
  }
  int pid_nx;                                                        // ids of the batch after the one in flight
  {
    const int pv = load_pids(0);
    KV16_FETCH(pv, vbuf_a)
    pid_nx = load_pids(min(1, nb - 1));
  }

  // ---- per-lane constants ----
  // V transpose reads: source lane (s = row16, g = grp), half h, addresses 4 channels (16c + 4(s&3) ..)
  // of token row r = 32 ks + 8g + 4h + s/4 of k-step ks: chunk 2c + (s&3)/2 of that row, at chunk position
  // (2c + (s&3)/2) ^ v_swz(r).  Head_dim 128: v_swz depends on s/4 only; head_dim 64: on s/4 and g.
  const int v_rho = row16 >> 2;
  const int vr_base = (8 * grp + v_rho) * kRowBytes + 16 * ((row16 & 3) >> 1) + 8 * (row16 & 1);
  const int vr_swz = v_swz(8 * grp + v_rho);
  // P: a lane writes column 16 pg + row16 of its token's page; the A operand read of lane (row, g) takes tokens
  // 32 ks + 8g .. + 7 of row % (2 LO), of the third limbs row % LO (zeroed for the rows from LO on)
  const uint32_t pa_addr = (uint32_t)(uintptr_t)(LDS_AS uint8_t*)pbuf + ((row16 & (2 * LO - 1)) * kProw + 8 * grp) * 2;
  const uint32_t pa3_addr = (uint32_t)(uintptr_t)(LDS_AS uint8_t*)pbuf + ((2 * LO + (row16 & (LO - 1))) * kProw + 8 * grp) * 2;
  const uint32_t third_rows = (kScaled ? (row16 & LO) != 0 : row16 < LO) ? 0xffffffffu : 0u;
  const int head0 = (G > 4) ? 4 * (grp & 1) : 0;                     // first head of this lane

  f32x4 oacc[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) oacc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_ref[NH], lsum[NH];
#pragma unroll
  for (int i = 0; i < NH; ++i) { m_ref[i] = -INFINITY; lsum[i] = 0.f; }

  auto two_batches = [&](const int bi0, uint8_t* __restrict__ const va, uint8_t* __restrict__ const vb,
                         uint8_t* __restrict__ const pb) {
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      if (half == 1 && bi0 + 1 >= nb) break;
      const int bi = bi0 + half;
      uint8_t* const vcur = half ? vb : va;
      uint8_t* const vnext = half ? va : vb;
      __builtin_amdgcn_s_waitcnt(0x0F70);                    // vmcnt(0): batch bi has landed (K registers, V in LDS)
      const int tok0 = t_begin + TB * bi;
      if (tok0 + TB > t_end) {
        // the slots past the range's last token may hold anything, NaN included, and 0 . NaN is NaN: clear their V rows
        for (int r = t_end - tok0 + v_row; r < TB; r += RT)
          *(u32x4*)(vcur + r * kRowBytes + 16 * (lane & (CPR - 1))) = u32x4{0u, 0u, 0u, 0u};
        wave_sync();
      }
      // ---- logits ----
      f32x4 dq[NP];
#pragma unroll
      for (int pg = 0; pg < NP; ++pg) {
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
          if (kThree) acc = mfma16<DT>(a_q3[kk], kreg[pg][kk], acc);
          acc = mfma16<DT>(a_q[kk], kreg[pg][kk], acc);
        }
        dq[pg] = acc;
      }
      // the next batch, if there is one: K into the registers just consumed, V into the other buffer
      if (bi + 1 < nb) {
        KV16_FETCH(pid_nx, vnext)
        pid_nx = load_pids(min(bi + 2, nb - 1));
      }
      // ---- gather: second limbs added to the first, lane = token, registers = heads ----
      float lg[NS][NH];
      int col[NS];                                             // this lane's token(s) of the batch
      bool need = false;
#pragma unroll
      for (int s = 0; s < NS; ++s)
        col[s] = 16 * (G > 4 ? 2 * s + (lane >> 5) : (NP == 4 ? grp : grp & 1)) + row16;
      const bool idle = G <= 4 && NP == 2 && lane >= 32;
#pragma unroll
      for (int i = 0; i < NH; ++i) {
        float v[NS];
        if constexpr (G > 4) {                                 // tile rows: first 0-3 | first 4-7 | second 0-3 | second 4-7
#pragma unroll
          for (int s = 0; s < NS; ++s) {
            float hi, lo;
            swap32(dq[2 * s][i], dq[2 * s + 1][i], hi, lo);
            v[s] = kScaled ? fmaf(lo, kLow, hi) : hi + lo;
          }
        } else if constexpr (NP == 4) {                        // first | second | idle | idle
          float h01, l01, h23, l23, hi, lo, junk;
          swap16(dq[0][i], dq[1][i], h01, l01);
          swap16(dq[2][i], dq[3][i], h23, l23);
          swap32(h01, h23, hi, junk);
          swap32(l01, l23, lo, junk);
          v[0] = kScaled ? fmaf(lo, kLow, hi) : hi + lo;
        } else {
          float hi, lo;
          swap16(dq[0][i], dq[1][i], hi, lo);                  // hi: rows (p0.hi, p1.hi, ..), lo: rows (p0.lo, p1.lo, ..)
          v[0] = hi + lo;
        }
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          if (DT == SAW_F16) v[s] *= q_back[kScaled ? i : 0];
          lg[s][i] = (!idle && tok0 + col[s] < t_end) ? v[s] : -INFINITY;
          need |= lg[s][i] > m_ref[i] + (kLazyTau + kLift);
        }
      }
      if (__any(need)) {
#pragma unroll
        for (int i = 0; i < NH; ++i) {
          float mx = lg[0][i];
          if (NS > 1) mx = fmaxf(mx, lg[NS - 1][i]);
          mx = row_allmax(mx);
          if (G <= 4) mx = max_xor16(mx);                      // eight heads: neighbouring lane groups hold other heads
          mx = max_xor32(mx);
          const float mnew = fmaxf(m_ref[i], mx - kLift);
          const float alpha = fast_exp2(m_ref[i] - mnew);
          lsum[i] *= alpha;
#pragma unroll
          for (int c = 0; c < CT; ++c) oacc[c][i] *= alpha;
          m_ref[i] = mnew;
        }
      }
#pragma unroll
      for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int i = 0; i < NH; ++i) {
          const float pr = fast_exp2(lg[s][i] - m_ref[i]);     // 0 for masked tokens and idle lanes
          lsum[i] += pr;
          uint32_t h16, l16, t16 = 0;
          if (kScaled) split16x3_scaled(pr, h16, l16, t16);
          else if (kThree) split16x3(pr, h16, l16, t16);
          else split16<DT>(pr, h16, l16);
          if (!idle) {
            ((uint16_t*)pb)[(head0 + i) * kProw + col[s]] = (uint16_t)h16;
            ((uint16_t*)pb)[(LO + head0 + i) * kProw + col[s]] = (uint16_t)l16;
            if (kThree) ((uint16_t*)pb)[(2 * LO + head0 + i) * kProw + col[s]] = (uint16_t)t16;
          }
        }
      wave_sync();
      // ---- O[row][channel] += P (rows x tokens) . V ----
      // (kThree: a batch's sums start at zero and are added to the running ones by the vector ALU, which rounds to nearest; the
      // matrix cores cut off what does not fit the accumulator, always in the same direction: 8000 tokens of like sign in one
      // partition came out 6e-6 too small)
      f32x4 tsum[kThree ? CT : 1];
#pragma unroll
      for (int c = 0; c < (kThree ? CT : 0); ++c) tsum[c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < TB / 32; ++ks) {
        u32x4 pa, pa3 = u32x4{0u, 0u, 0u, 0u};
        if constexpr (kThree) {
          asm volatile("ds_read_b128 %0, %2\n\tds_read_b128 %1, %3\n\ts_waitcnt lgkmcnt(0)"
                       : "=&v"(pa), "=&v"(pa3) : "v"(pa_addr + 64 * ks), "v"(pa3_addr + 64 * ks) : "memory");
          pa3 &= u32x4{third_rows, third_rows, third_rows, third_rows};
        } else {
          asm volatile("ds_read_b128 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(pa) : "v"(pa_addr + 64 * ks) : "memory");
        }
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          // (an even swizzle leaves the half-chunk bits of vr_base alone; rows 4 apart have the same one)
          const int voff = vr_base + 32 * ks * kRowBytes + 16 * ((2 * c) ^ vr_swz);
          const i16x4 t0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS i16x4*)(vcur + voff));
          const i16x4 t1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS i16x4*)(vcur + voff + 4 * kRowBytes));
          const u32x2 b0 = __builtin_bit_cast(u32x2, t0), b1 = __builtin_bit_cast(u32x2, t1);
          const u32x4 bv = u32x4{b0.x, b0.y, b1.x, b1.y};
          if constexpr (kThree) {
            tsum[c] = mfma16<DT>(pa3, bv, tsum[c]);
            tsum[c] = mfma16<DT>(pa, bv, tsum[c]);
          } else {
            oacc[c] = mfma16<DT>(pa, bv, oacc[c]);
          }
        }
      }
#pragma unroll
      for (int c = 0; c < (kThree ? CT : 0); ++c) oacc[c] += tsum[c];
      wave_sync();                                           // P is rewritten by the next batch
    }
  };
  for (int bi = 0; bi < nb; bi += 2) two_batches(bi, vbuf_a, vbuf_b, pbuf);
  __builtin_amdgcn_s_waitcnt(0x0F70);                        // nothing this wavefront requested is still on its way

  // ---- epilogue ----
#pragma unroll
  for (int i = 0; i < NH; ++i) {
    lsum[i] = row_allsum(lsum[i]);
    if (G <= 4) lsum[i] = add_xor16(lsum[i]);
    lsum[i] = add_xor32(lsum[i]);
  }
  // oacc[c][i] of lane (grp, row16) = O[row 4 grp + i][channel 16c + row16]: up to four heads rows 0..3 (grp 0) hold
  // the first (and third) limbs' part, rows 4..7 (grp 1) the second limbs'; eight heads: grps 0, 1 and 2, 3
  const bool writer = (G > 4) ? grp < 2 : grp == 0;
  const float limb = kScaled && ((G > 4) ? grp >= 2 : (grp & 1)) ? kLow : 1.f;
  auto both_limbs = [&](float v) { return (G > 4) ? add_xor32(v * limb) : add_xor16(v * limb); };
  if constexpr (kThree) {
    bool bad = false;
#pragma unroll
    for (int i = 0; i < NH; ++i) {
      bad |= !(lsum[i] < INFINITY);
#pragma unroll
      for (int c = 0; c < CT; ++c) bad |= !(fabsf(oacc[c][i]) < INFINITY);
    }
    if (__any(bad)) {
      static_assert(G * D * 4 + G * 8 <= kVbufBytes, "a record fits a V buffer");
      const float* const rec = (const float*)vbuf_b;
      wave_sync();                                                    // (every read of the buffers is done)
      range_fp32<D, G, DT>(p, b, kvh, t_begin, t_end, lane, (float*)vbuf_a, (float*)vbuf_b);
#pragma unroll
      for (int i = 0; i < NH; ++i) {
        m_ref[i] = rec[G * D + 2 * (head0 + i)];
        lsum[i] = rec[G * D + 2 * (head0 + i) + 1];
#pragma unroll
        for (int c = 0; c < CT; ++c) oacc[c][i] = writer ? rec[(head0 + i) * D + 16 * c + row16] : 0.f;
      }
      wave_sync();
    }
  }
  if (PAIR && share) {
    // this wavefront's share of the long sequence as a record in its own V buffer (every read of
    // it is done and nothing is in flight): acc[G][D] un-normalised, then (max, sum) per head
    static_assert(G * D * 4 + G * 8 <= kVbufBytes, "a record fits a V buffer");
    float* const rec = (float*)vbuf_a;
    wave_sync();
#pragma unroll
    for (int i = 0; i < NH; ++i) {
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        const float o = both_limbs(oacc[c][i]);
        if (writer) rec[(head0 + i) * D + 16 * c + row16] = o;
      }
      if (writer && row16 == 0) { rec[G * D + 2 * (head0 + i)] = m_ref[i]; rec[G * D + 2 * (head0 + i) + 1] = lsum[i]; }
    }
    // LDS operations of a wavefront complete in order, so the record is in place before the count;
    // the wavefront that finds the other already counted does the rest for both (a shared range
    // is always a wavefront's last).
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    int before = 0;
    if (lane == 0) before = __hip_atomic_fetch_add(done_cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    before = __builtin_amdgcn_readfirstlane(before);
    if (before == 0) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    const float* const rec0 = (const float*)lds_all;                  // wavefront 0's record is always the first operand
    const float* const rec1 = (const float*)(lds_all + kWaveLds);
    const int64_t obase = ((int64_t)b * p.n_q_heads + kvh * G) * D;
    for (int idx = lane; idx < G * D; idx += 64) {
      const int h = idx / D;
      const float m0 = rec0[G * D + 2 * h], m1 = rec1[G * D + 2 * h];
      const float mm = fmaxf(m0, m1);
      const float a0 = fast_exp2(m0 - mm), a1 = fast_exp2(m1 - mm);
      const float v = fmaf(a1, rec1[idx], a0 * rec0[idx]);
      const float l = fmaf(a1, rec1[G * D + 2 * h + 1], a0 * rec0[G * D + 2 * h + 1]);
      store_elem(p.out, p.out_dtype, obase + idx, v / l);
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < NH; ++i) {
    const int head = kvh * G + head0 + i;
    const bool alone = !CUT && p.num_splits == 1;
    float* part = p.ws + (CUT ? (int64_t)head * p.cut + split : ((int64_t)b * p.n_q_heads + head) * p.num_splits + split) * (D + 2);
    const float inv = 1.0f / lsum[i];
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      const float o = both_limbs(oacc[c][i]);
      if (writer) {
        if (alone)
          store_elem(p.out, p.out_dtype, ((int64_t)b * p.n_q_heads + head) * D + 16 * c + row16, o * inv);
        else
          part[2 + 16 * c + row16] = o;
      }
    }
    if (!alone && writer && row16 == 0) { part[0] = m_ref[i]; part[1] = lsum[i]; }
  }
  wave_sync();                                   // the next range's prologue reuses the buffers
  }  // ranges of this wavefront
}

#undef KV16_FETCH

template <int D, int G, int DT>
static void go_kv16(const DecodeParams& p, dim3 grid, hipStream_t st) {
  if (p.pair) decode_kv16_mfma_kernel<D, G, DT, true, false><<<dim3(1, grid.y, (p.batch + 1) / 2), dim3(128), 0, st>>>(p);
  else if (p.cut) decode_kv16_mfma_kernel<D, G, DT, false, true><<<grid, dim3(64), 0, st>>>(p);
  else decode_kv16_mfma_kernel<D, G, DT, false, false><<<grid, dim3(64), 0, st>>>(p);
}
template <int D, int DT>
static int go_kv16_g(const DecodeParams& p, int G, dim3 grid, hipStream_t st) {
  switch (G) {
    case 1: go_kv16<D, 1, DT>(p, grid, st); return SAW_OK;
    case 2: go_kv16<D, 2, DT>(p, grid, st); return SAW_OK;
    case 4: go_kv16<D, 4, DT>(p, grid, st); return SAW_OK;
    case 8: go_kv16<D, 8, DT>(p, grid, st); return SAW_OK;
    default: return SAW_EINVAL;
  }
}

// `D`: head_dim, 64 or 128; `G`: query heads per kv head, 1, 2, 4 or 8.
int launch_decode_kv16_mfma(const DecodeParams& p, int D, int G, int kv_dtype, dim3 grid, hipStream_t st) {
  if (D == 128) return kv_dtype == SAW_BF16 ? go_kv16_g<128, SAW_BF16>(p, G, grid, st) : go_kv16_g<128, SAW_F16>(p, G, grid, st);
  return kv_dtype == SAW_BF16 ? go_kv16_g<64, SAW_BF16>(p, G, grid, st) : go_kv16_g<64, SAW_F16>(p, G, grid, st);
}

}  // namespace saw
