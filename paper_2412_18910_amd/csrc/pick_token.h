// What the kernel that fixes a draft token does with it: its embedding for the next chained forward, the exit rule's statistic.
#pragma once
#include "ae_internal.h"
#include "packed.h"

namespace ae {

// Embedding of token t -> row cat.row, k = d .. 2d - 1 (the second half of the draft head's input
// [feature ; embedding of the next token]); all threads of the workgroup.
__device__ __forceinline__ void write_embedding(const DraftCat &cat, int32_t t) {
  const int d = cat.d;
  if (cat.f32) {
    const float *e = (const float *)cat.emb + (size_t)t * d;
    float *o = (float *)cat.Xp + (size_t)cat.row * 2 * d + d;
    for (int k0 = threadIdx.x * 4; k0 < d; k0 += blockDim.x * 4)
      *reinterpret_cast<float4 *>(o + k0) = *reinterpret_cast<const float4 *>(e + k0);
    return;
  }
  const uint16_t *e = (const uint16_t *)cat.emb + (size_t)t * d;
  for (int k0 = threadIdx.x * 4; k0 < d; k0 += blockDim.x * 4) {
    const uint2 raw = *reinterpret_cast<const uint2 *>(e + k0);
    packed_store4((u32x4 *)cat.Xp, cat.row, d + k0, __uint_as_float(raw.x << 16), __uint_as_float(raw.x & 0xffff0000u),
                  __uint_as_float(raw.y << 16), __uint_as_float(raw.y & 0xffff0000u));
  }
}

// What a kernel knows already when it calls ddd_finish: the token's logit; held: the maximum over the row-blocks and this thread's
// share of the sum of exponentials (row-blocks threadIdx.x + 256 * j).
struct DddPartial {
  bool held = false;
  float logit = 0.f, mx = -INFINITY, se = 0.f;
};

// AdaEAGLE-DDD bookkeeping behind draft token i (Sec. 3.4, 4.2) from the LM-head epilogue's
// row-block statistics of row 0; all threads of the workgroup call, 256 of them work.  Fixed-shape reductions.
__device__ inline void ddd_finish(const DddFinish &d, int i, DevState *st, const DddPartial &part) {
  __shared__ float red_s[4];
  const int t = threadIdx.x;
  float mx = part.mx, se = part.se;
  if (!part.held) {
    for (int p = t; t < 256 && p < d.NB; p += 256) mx = fmaxf(mx, d.val[p]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    if ((t & 63) == 0 && t < 256) red_s[t >> 6] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(red_s[0], red_s[1]), fmaxf(red_s[2], red_s[3]));
    __syncthreads();
    for (int p = t; t < 256 && p < d.NB; p += 256) se += d.lse_sum[p] * expf((d.val[p] - mx) * d.inv_t);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) se += __shfl_xor(se, o, 64);
  if ((t & 63) == 0 && t < 256) red_s[t >> 6] = se;
  __syncthreads();
  if (t == 0) {
    se = (red_s[0] + red_s[1]) + (red_s[2] + red_s[3]);
    const float lp = (part.logit - mx) * d.inv_t - logf(se);
    const float cum = (i == 0 ? 0.f : st->cum_logp) + lp;
    st->draft_lp[i] = lp;
    st->cum_logp = cum;
    st->draft_len = i + 1;
    const bool stop = i + 1 >= d.k && !(cum >= d.theta);
    if (stop) st->draft_live = 0;
    if (d.flag) __hip_atomic_store(d.flag, d.seq << 1 | (stop ? 0u : 1u), __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

}  // namespace ae
