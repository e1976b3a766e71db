// 16-bit-KV paged decode attention on the vector ALU, in fp32: head_dim 64 with one query head per kv head, and with two where
// the call is small.  (The comparison path: the cache the paper measures INT4 against, Sec. 2.)
//
// One block of four wavefronts per (sequence, kv head, partition); a wavefront covers 16 tokens per pass, a token's row split over
// four lanes.  With so few query heads the products are few, and the matrix-core kernel (saw_decode_kv16_mfma.hip) spends more on
// its limbs and on the layout changes around 16-row tiles, most of whose rows are idle, than the products cost here; this kernel's
// short chain of dependent steps and its four wavefronts per partition decide the rest.  Measured, 8 kv heads, one query head per kv
// head, this kernel against that one: 2 x 2304 tokens 9.9 and 12.2 us, 200 ragged up to 600 31.7 and 57, 170 ragged up to 2304
// 95 and 122; behind it 64 x 8000 189 and 171 (equal lengths, all resident).
#include "saw_decode.h"
#include "saw_wave_util.h"

namespace saw {

template <int G, int DT>
__global__ __launch_bounds__(256) void decode_kv16_valu_kernel(DecodeParams p) {
  constexpr int D = 64, LPT = 4;       // head_dim; lanes a token's row is split over
  constexpr int TPW = 64 / LPT;        // tokens per wavefront and pass
  constexpr int CPL = D / LPT;         // elements per lane
  constexpr int WPL = CPL / 2;         // dwords per lane
  // (the partition index is rotated by kv head and sequence, so that no XCD serves a fixed set of partitions)
  const int split = (blockIdx.x + blockIdx.y + blockIdx.z) % gridDim.x, kvh = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int L = min(p.seq_lens[b], p.bound);
  const int t_begin = split * p.chunk_tokens;
  const int t_end = min(L, t_begin + p.chunk_tokens);
  if (t_begin >= t_end) return;

  __shared__ float qs[G * D];
  __shared__ float red[4][G][D + 4];
  for (int i = tid; i < G * D; i += 256)
    qs[i] = p.q_scale * load_elem(p.q, p.q_dtype, ((int64_t)b * p.n_q_heads + kvh * G) * D + i);
  __syncthreads();

  const int part = lane % LPT;
  float m[G], lsum[G], acc[G][CPL];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    m[g] = -INFINITY; lsum[g] = 0.f;
#pragma unroll
    for (int j = 0; j < CPL; ++j) acc[g][j] = 0.f;
  }
  const uint16_t* kpages = (const uint16_t*)p.k_codes;
  const uint16_t* vpages = (const uint16_t*)p.v_codes;
  const int64_t pt_row = (int64_t)b * p.max_pages;
  for (int t0 = t_begin + wave * TPW; t0 < t_end; t0 += 4 * TPW) {
    const int t = t0 + lane / LPT;
    const bool valid = t < t_end;
    const int tt = valid ? t : t_end - 1;
    int32_t page = p.page_table[pt_row + (tt >> 4)];
    page = (page < 0 || page >= p.num_pages) ? 0 : page;
    const int64_t vec = ((int64_t)page * p.n_kv_heads + kvh) * 16 + (tt & 15);
    const uint4* kp = (const uint4*)(kpages + vec * D + part * CPL);
    const uint4* vp = (const uint4*)(vpages + vec * D + part * CPL);
    float dot[G];
#pragma unroll
    for (int g = 0; g < G; ++g) dot[g] = 0.f;
#pragma unroll
    for (int i = 0; i < WPL / 4; ++i) {
      const uint4 w4 = kp[i];
      const uint32_t ww[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float lo, hi;
        widen2<DT>(ww[j], lo, hi);
#pragma unroll
        for (int g = 0; g < G; ++g) {
          dot[g] = fmaf(qs[g * D + part * CPL + i * 8 + 2 * j], lo, dot[g]);
          dot[g] = fmaf(qs[g * D + part * CPL + i * 8 + 2 * j + 1], hi, dot[g]);
        }
      }
    }
    float w[G], mnew[G];
    bool grow = false;
#pragma unroll
    for (int g = 0; g < G; ++g) {
#pragma unroll
      for (int mk = 1; mk < LPT; mk <<= 1) dot[g] += __shfl_xor(dot[g], mk, SAW_WAVE);
      const float logit = valid ? dot[g] : -INFINITY;
      float mt = logit;
#pragma unroll
      for (int mk = LPT; mk < 64; mk <<= 1) mt = fmaxf(mt, __shfl_xor(mt, mk, SAW_WAVE));
      mnew[g] = fmaxf(m[g], mt);
      grow |= mnew[g] > m[g];
      w[g] = logit;
    }
    if (grow) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const float a = fast_exp2(m[g] - mnew[g]);
        lsum[g] *= a;
#pragma unroll
        for (int j = 0; j < CPL; ++j) acc[g][j] *= a;
        m[g] = mnew[g];
      }
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      w[g] = valid ? fast_exp2(w[g] - m[g]) : 0.f;
      lsum[g] += w[g];
    }
#pragma unroll
    for (int i = 0; i < WPL / 4; ++i) {
      const uint4 w4 = vp[i];
      const uint32_t ww[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float lo, hi;
        widen2<DT>(ww[j], lo, hi);
#pragma unroll
        for (int g = 0; g < G; ++g) {
          acc[g][i * 8 + 2 * j] = fmaf(w[g], lo, acc[g][i * 8 + 2 * j]);
          acc[g][i * 8 + 2 * j + 1] = fmaf(w[g], hi, acc[g][i * 8 + 2 * j + 1]);
        }
      }
    }
  }
#pragma unroll
  for (int g = 0; g < G; ++g) {
#pragma unroll
    for (int mk = LPT; mk < 64; mk <<= 1) {
      lsum[g] += __shfl_xor(lsum[g], mk, SAW_WAVE);
#pragma unroll
      for (int j = 0; j < CPL; ++j) acc[g][j] += __shfl_xor(acc[g][j], mk, SAW_WAVE);
    }
  }
  if (lane < LPT) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
#pragma unroll
      for (int j = 0; j < CPL; ++j) red[wave][g][part * CPL + j] = acc[g][j];
      if (part == 0) { red[wave][g][D] = m[g]; red[wave][g][D + 1] = lsum[g]; }
    }
  }
  __syncthreads();
  for (int idx = tid; idx < G * (D + 2); idx += 256) {
    const int g = idx / (D + 2), c = idx % (D + 2);
    float mm = -INFINITY;
#pragma unroll
    for (int wv = 0; wv < 4; ++wv) mm = fmaxf(mm, red[wv][g][D]);
    float v;
    if (c == 0) {
      v = mm;
    } else {
      const int src = (c == 1) ? D + 1 : c - 2;
      v = 0.f;
#pragma unroll
      for (int wv = 0; wv < 4; ++wv) v += fast_exp2(red[wv][g][D] - mm) * red[wv][g][src];
    }
    p.ws[(((int64_t)b * p.n_q_heads + kvh * G + g) * p.num_splits + split) * (D + 2) + c] = v;
  }
}

template <int G>
static void go_kv16_valu(const DecodeParams& p, int kv_dtype, dim3 grid, hipStream_t st) {
  if (kv_dtype == SAW_BF16) decode_kv16_valu_kernel<G, SAW_BF16><<<grid, dim3(256), 0, st>>>(p);
  else decode_kv16_valu_kernel<G, SAW_F16><<<grid, dim3(256), 0, st>>>(p);
}

// `G`: query heads per kv head, 1 or 2.
int launch_decode_kv16_valu(const DecodeParams& p, int G, int kv_dtype, dim3 grid, hipStream_t st) {
  if (G == 1) go_kv16_valu<1>(p, kv_dtype, grid, st);
  else if (G == 2) go_kv16_valu<2>(p, kv_dtype, grid, st);
  else return SAW_EINVAL;
  return SAW_OK;
}

}  // namespace saw
