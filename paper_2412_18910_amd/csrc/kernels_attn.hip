// KV cache layout, import and export.
//
// Float32 cache of one layer:
//   K: [n_kv_heads][head_dim/8][n_ctx_max][8]   -- "d-group major": for a fixed group of 8
//      head-dim elements, consecutive slots are contiguous;
//   V: [n_kv_heads][n_ctx_max][head_dim]        -- row-major.
// The bf16 cache holds MFMA operand tiles (kernels_attn_mfma.hip).
// A verify block first appends its K/V rows at slots pos0.., then every row attends the
// cache causally (row i sees slots 0..pos0+i).  Split-KV chunks are fixed by absolute
// slot, masked keys contribute exact zeros, and all reductions
// have a fixed shape, so a row's result does not depend on how many rows share the block.
#include "ae_internal.h"

namespace ae {

using bf16_t = uint16_t;

__device__ __forceinline__ float bf2f_(bf16_t h) { return __uint_as_float((uint32_t)h << 16); }
// round-to-nearest-even float -> bf16 bits
__device__ __forceinline__ bf16_t f2bf_(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u) return (bf16_t)(u >> 16);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}
template <typename T> __device__ __forceinline__ float cvt_in(T v);
template <> __device__ __forceinline__ float cvt_in<float>(float v) { return v; }
template <> __device__ __forceinline__ float cvt_in<bf16_t>(bf16_t v) { return bf2f_(v); }
template <typename T> __device__ __forceinline__ T cvt_out(float v);
template <> __device__ __forceinline__ float cvt_out<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16_t cvt_out<bf16_t>(float v) { return f2bf_(v); }

static size_t esize(const ae_config &c) { return c.dtype == AE_BF16 ? 2 : 4; }
int kv_capacity(const ae_config &c) { return (c.n_ctx_max + kAttnChunk - 1) / kAttnChunk * kAttnChunk; }
size_t kv_v_offset_bytes(const ae_config &c) {
  return (size_t)c.n_kv_heads * c.head_dim * kv_capacity(c) * esize(c);
}
size_t kv_layer_bytes(const ae_config &c) { return 2 * kv_v_offset_bytes(c); }

// Element index of K[kh][slot][d] / V[kh][slot][d] in the cache of one layer.  n_ctx is
// the capacity (a multiple of kAttnChunk).  `tiled` selects the MFMA operand layout
// of kernels_attn_mfma.hip, else the layout described at the top of this file.
template <typename T>
__device__ __forceinline__ size_t k_index(int kh, int d, int slot, int hd, int n_ctx, bool tiled) {
  if (tiled)  // [kh][slot/16][d/32][lane = ((d%32)/8)*16 + slot%16][d%8]
    return ((((size_t)kh * (n_ctx / 16) + (slot >> 4)) * (hd / 32) + (d >> 5)) * 64 + ((d & 31) >> 3) * 16 + (slot & 15)) * 8 + (d & 7);
  return (((size_t)kh * (hd / 8) + (d >> 3)) * n_ctx + slot) * 8 + (d & 7);
}
__device__ __forceinline__ size_t v_index(int kh, int d, int slot, int hd, int n_ctx, bool tiled) {
  if (tiled) {  // [kh][slot/32][d/16][lane = ((slot%16)/4)*16 + d%16][e = slot%4 + 4*((slot%32)/16)]
    const int w16 = slot & 15, half = (slot & 31) >> 4;
    return ((((size_t)kh * (n_ctx / 32) + (slot >> 5)) * (hd / 16) + (d >> 4)) * 64 + (w16 >> 2) * 16 + (d & 15)) * 8 + (w16 & 3) + 4 * half;
  }
  return ((size_t)kh * n_ctx + slot) * hd + d;
}

size_t attn_part_floats(const ae_config &c) {
  const int max_chunks = kv_capacity(c) / (c.dtype == AE_BF16 ? kMfmaAttnChunk : attn_f32_chunk_keys());
  return (size_t)c.n_heads * max_chunks * kMaxRows * (c.head_dim + 2);
}

// ------------------------------------------------------------------ import / export (tests, set-up)
template <typename T>
__global__ void kv_import_kernel(T *Kc, T *Vc, const float *k, const float *v, int n, int Hkv, int hd, int n_ctx,
                                 bool tiled) {
  const size_t total = (size_t)n * Hkv * hd;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
    const int d = i % hd, kh = (i / hd) % Hkv, slot = i / ((size_t)hd * Hkv);
    Kc[k_index<T>(kh, d, slot, hd, n_ctx, tiled)] = cvt_out<T>(k[i]);
    Vc[v_index(kh, d, slot, hd, n_ctx, tiled)] = cvt_out<T>(v[i]);
  }
}

void launch_kv_import(void *kv_layer, size_t v_off, const ae_config &c, const float *k_dev, const float *v_dev, int n,
                      bool tiled, hipStream_t s) {
  void *vc = (char *)kv_layer + v_off;
  if (c.dtype == AE_BF16)
    kv_import_kernel<bf16_t><<<1024, 256, 0, s>>>((bf16_t *)kv_layer, (bf16_t *)vc, k_dev, v_dev, n, c.n_kv_heads,
                                                  c.head_dim, kv_capacity(c), tiled);
  else
    kv_import_kernel<float><<<1024, 256, 0, s>>>((float *)kv_layer, (float *)vc, k_dev, v_dev, n, c.n_kv_heads,
                                                 c.head_dim, kv_capacity(c), tiled);
}

template <typename T>
__global__ void kv_export_kernel(const T *Kc, const T *Vc, int which, int slot, int Hkv, int hd, int n_ctx, bool tiled,
                                 float *out) {
  for (int i = threadIdx.x; i < Hkv * hd; i += blockDim.x) {
    const int d = i % hd, kh = i / hd;
    out[i] = which ? cvt_in<T>(Vc[v_index(kh, d, slot, hd, n_ctx, tiled)]) : cvt_in<T>(Kc[k_index<T>(kh, d, slot, hd, n_ctx, tiled)]);
  }
}

hipError_t launch_kv_export(const void *kv_layer, size_t v_off, const ae_config &c, int which, int slot, float *out_dev,
                            bool tiled, hipStream_t s) {
  const void *vc = (const char *)kv_layer + v_off;
  if (c.dtype == AE_BF16)
    return launch_checked(kv_export_kernel<bf16_t>, dim3(1), dim3(256), s, (const bf16_t *)kv_layer, (const bf16_t *)vc, which, slot,
                          c.n_kv_heads, c.head_dim, kv_capacity(c), tiled, out_dev);
  return launch_checked(kv_export_kernel<float>, dim3(1), dim3(256), s, (const float *)kv_layer, (const float *)vc, which, slot,
                        c.n_kv_heads, c.head_dim, kv_capacity(c), tiled, out_dev);
}

}  // namespace ae
