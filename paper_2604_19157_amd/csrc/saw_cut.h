// Cutting a batch into partitions by its own lengths, in the kernel: shared by the decode kernels and the merge pass.
#pragma once

#include "saw_decode.h"
#include "saw_rank.h"

namespace saw {

// Split-KV with a partition length worked out on the host has to go by the caller's bound: with a loose bound (the
// usual serving call, which avoids a host read of the lengths) or a ragged batch most of its partitions are empty
// and the longest sequences decide.  Here the W = p.cut partition slots of a kv head are dealt out by the lengths
// themselves: c = the smallest number of 64-token batches (at least p.cut_min) for which sum_b ceil(nb_b / c) <= W,
// sequence b gets P_b = ceil(nb_b / c) consecutive slots and its batches are spread evenly over them.  No slot streams
// more than c batches, and c <= max(p.cut_min, ceil(sum / (W - B))): up to twice the ideal sum / W where the host gives a batch only
// twice as many slots as sequences (W = 128: 48 sequences of 64 batches get c = 32 against 24, a quarter of the slots stays empty).
// Every wavefront works this out for itself from the lengths (one load each, up to kMaxCut sequences); an empty sequence has
// no slot, with a fused append one slot (its new token).  The wavefront of a sequence's first slot leaves (first slot, slots) for
// the merge pass, which has thousands of blocks to work it out again in otherwise (64 x 64 rows: 10.4 against 5.1 us).
constexpr int kCutGroups = kMaxCut / 64;

struct BatchCut {
  int nb[kCutGroups];      // batches of sequence 64 v + lane (an empty sequence with an append: 1)
  int len[kCutGroups];     // its length, clamped
  int V;                   // ceil(B / 64)
  int c;
  float rc;                // 1 / c
};
__device__ __forceinline__ int wave_sum_i(int v) {
  v += dpp_i0<0x121, 0xf>(v);
  v += dpp_i0<0x122, 0xf>(v);
  v += dpp_i0<0x124, 0xf>(v);
  v += dpp_i0<0x128, 0xf>(v);
  return (__builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16)) +
         (__builtin_amdgcn_readlane(v, 32) + __builtin_amdgcn_readlane(v, 48));
}
// inclusive prefix sum over the 64 lanes
__device__ __forceinline__ int wave_scan_i(int v) {
  v += dpp_i0<0x111, 0xf>(v);
  v += dpp_i0<0x112, 0xf>(v);
  v += dpp_i0<0x114, 0xf>(v);
  v += dpp_i0<0x118, 0xf>(v);
  v += dpp_i0<0x142, 0xa>(v);
  v += dpp_i0<0x143, 0xc>(v);
  return v;
}
// ceil(n / c), n < 2^23 (the host keeps longer bounds away): the float quotient is off by one at most
__device__ __forceinline__ int parts_of(int n, int c, float rc) {
  const int x = n + c - 1;
  int q = (int)((float)x * rc);
  const int r = x - q * c;
  q += (r >= c) ? 1 : 0;
  q -= (r < 0) ? 1 : 0;
  return q;
}
__device__ __forceinline__ int cut_count(const BatchCut& k, int c) {
  const float rc = 1.0f / (float)c;
  int s = 0;
#pragma unroll
  for (int v = 0; v < kCutGroups; ++v)
    if (v < k.V) s += parts_of(k.nb[v], c, rc);
  return wave_sum_i(s);
}
__device__ __forceinline__ BatchCut cut_batch(const DecodeParams& p, int lane) {
  BatchCut k;
  const int B = p.batch, W = p.cut;
  k.V = (B + 63) >> 6;
#pragma unroll
  for (int v = 0; v < kCutGroups; ++v) {
    k.nb[v] = k.len[v] = 0;
    if (v < k.V && 64 * v + lane < B) k.len[v] = p.seq_lens[64 * v + lane];
  }
  int sum = 0;
#pragma unroll
  for (int v = 0; v < kCutGroups; ++v)
    if (v < k.V && 64 * v + lane < B) {
      k.len[v] = max(min(k.len[v], p.bound), 0);
      k.nb[v] = max((k.len[v] + 63) >> 6, p.append ? 1 : 0);
      sum += k.nb[v];
    }
  const int T = wave_sum_i(sum);                              // (below 2^23: the host bounds B times the bound)
  // ceil(T / W) is a lower end; an upper one is ceil(T / (W - B)), because sum_b ceil(nb_b / c) <= T / c + B
  // (the host gives a cut batch more slots than sequences)
  int lo = max(p.cut_min, parts_of(T, W, 1.0f / (float)W));
  if (cut_count(k, lo) > W) {
    int hi = max(lo, parts_of(T, W - B, 1.0f / (float)(W - B)));
    while (hi - lo > 1) {                                     // count(lo) > W >= count(hi)
      const int mid = (lo + hi) >> 1;
      if (cut_count(k, mid) > W) lo = mid; else hi = mid;
    }
    lo = hi;
  }
  k.c = lo;
  k.rc = 1.0f / (float)lo;
  return k;
}
// the sequence, its length and the partition of slot w: b < 0 if the batch does not fill that many slots
__device__ __forceinline__ void cut_slot(const BatchCut& k, int w, int& b, int& len, int& part, int& parts) {
  b = -1; part = 0; parts = 1; len = 0;
  int base = 0;
#pragma unroll
  for (int v = 0; v < kCutGroups; ++v) {
    if (v < k.V && b < 0) {                                   // wavefront-uniform
      const int P = parts_of(k.nb[v], k.c, k.rc);
      const int incl = wave_scan_i(P);
      const unsigned long long hit = __ballot(w - base >= incl - P && w - base < incl);
      if (hit) {
        const int l = __ffsll((long long)hit) - 1;
        b = 64 * v + l;
        parts = __builtin_amdgcn_readlane(P, l);
        len = __builtin_amdgcn_readlane(k.len[v], l);
        part = w - base - (__builtin_amdgcn_readlane(incl, l) - parts);
      }
      base += __builtin_amdgcn_readlane(incl, 63);
    }
  }
}
// floor(n / c), n < 2^23
__device__ __forceinline__ int floor_div(int n, int c) { return parts_of(n - c + 1, c, 1.0f / (float)c); }
// batches [first, end) of partition `part` of `parts` of a sequence of nb batches: the first nb % parts partitions
// have one more than the others
__device__ __forceinline__ void cut_range(int nb, int part, int parts, int& first, int& end) {
  const int q = floor_div(nb, parts), r = nb - q * parts;
  first = part * q + min(part, r);
  end = first + q + (part < r ? 1 : 0);
}

}  // namespace saw
