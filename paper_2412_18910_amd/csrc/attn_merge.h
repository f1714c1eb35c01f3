// Chunks of keys that one attention workgroup holds, a group of four waves each: what attn_merge_log2_kernel makes of their
// partials, bit for bit, without the launch between (4.5 us of a 7B layer, 4 of the smallest model's; latency bounds both, so
// the sums stay in LDS and 16 rows are merged at once).
#pragma once
#include "ae_internal.h"

namespace ae {

template <int HD, int NG>
struct ChunkMerge {
  float o[NG][16][HD], mx[NG][16], l[NG][16];   // sums against the chunk's maximum (log2 domain), that maximum, sum of weights

  // elements k0 .. k0 + 3 of row m; chunks in ascending order against the overall maximum
  __device__ __forceinline__ float4 merged(int m, int k0) const {
    float mall = mx[0][m];
#pragma unroll
    for (int i = 1; i < NG; ++i) mall = fmaxf(mall, mx[i][m]);
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    float dall = 0.f;
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      if (mx[i][m] > -INFINITY) {
        const float wgt = __builtin_amdgcn_exp2f(mx[i][m] - mall);
        const float4 v = *reinterpret_cast<const float4 *>(&o[i][m][k0]);
        acc.x = fmaf(wgt, v.x, acc.x); acc.y = fmaf(wgt, v.y, acc.y);
        acc.z = fmaf(wgt, v.z, acc.z); acc.w = fmaf(wgt, v.w, acc.w);
        dall = fmaf(wgt, l[i][m], dall);
      }
    }
    return make_float4(acc.x / dall, acc.y / dall, acc.z / dall, acc.w / dall);
  }
};

}  // namespace ae
