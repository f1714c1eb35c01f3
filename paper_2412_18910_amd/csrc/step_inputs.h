// Small per-step work that rides on a kernel that is launched anyway instead of a launch of its own (a dependent
// launch costs 1.5-4 us, whatever it does): the ids of the verify block, the inputs of a draft, feature rows, the greedy
// acceptance test.  Four launches of a step fall away: float32 tiny model 334 -> 323 us, 4 layers of 7B with the exit
// rule 842 -> 835; in a step of 32 layers (3.8 ms) that is less than runs differ by.
#pragma once
#include "ae_internal.h"

namespace ae {

// Token id of row r; a block that is put together here is recorded in st->block by the caller's workgroup of that row.
__device__ __forceinline__ int32_t block_id(const BlockIds &b, int r) {
  if (b.ids) return b.ids[r];
  const int32_t id = !b.hist ? b.v[r] : r == 0 ? b.hist[b.kv_len] : b.st->draft_ids[r - 1];
  if (threadIdx.x == 0) b.st->block[r] = id;
  return id;
}

// Override table, chain gate and sampling uniforms of a draft, by the first wave of one workgroup.
__device__ __forceinline__ void store_draft_inputs(const DraftInputs &in) {
  const int t = threadIdx.x;
  if (t < kMaxRows) {
    in.st->override_ids[t] = in.override_ids[t];
    if (t < in.n_u) in.st->u_draft[t] = in.u[t];
  }
  if (t == 0) {
    in.st->draft_live = 1;
    in.st->draft_len = 0;
  }
}

// out = (x / sqrt(mean(x^2) + eps)) * g for one row, 256 threads
__device__ __forceinline__ void rmsnorm_row(const float *xr, const float *g, int d, float eps, float *out) {
  __shared__ float red_n[4];
  float ss = 0.f;
  for (int i = threadIdx.x * 4; i < d; i += 1024) {   // d is a multiple of 8
    const float4 v = *reinterpret_cast<const float4 *>(xr + i);
    ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
  if ((threadIdx.x & 63) == 0) red_n[threadIdx.x >> 6] = ss;
  __syncthreads();
  const float tot = (red_n[0] + red_n[1]) + (red_n[2] + red_n[3]);
  const float r = 1.0f / sqrtf(tot / (float)d + eps);
  for (int i = threadIdx.x * 4; i < d; i += 1024) {
    const float4 v = *reinterpret_cast<const float4 *>(xr + i), gn = *reinterpret_cast<const float4 *>(g + i);
    *reinterpret_cast<float4 *>(out + i) = make_float4((v.x * r) * gn.x, (v.y * r) * gn.y, (v.z * r) * gn.z, (v.w * r) * gn.w);
  }
}

// Length of the longest draft prefix equal to the target argmax; every lane of a wave calls.
__device__ __forceinline__ int greedy_accepted(const DevState *st, int k) {
  const int lane = threadIdx.x & 63;
  const bool same = lane < k && st->block[1 + (lane < kMaxRows - 1 ? lane : 0)] == st->argmax[lane < kMaxRows ? lane : 0];
  return __builtin_ctzll(~(unsigned long long)__ballot(same));
}
// ... and the history, length and bonus token that follow from it (one thread)
__device__ __forceinline__ void greedy_record(DevState *st, int32_t *hist, int kv_len, int acc) {
  const int32_t bonus = st->argmax[acc];
  for (int i = 0; i <= acc; ++i) hist[kv_len + i] = st->block[i];
  hist[kv_len + 1 + acc] = bonus;
  st->n_acc = acc;
  st->bonus = bonus;
}

}  // namespace ae
