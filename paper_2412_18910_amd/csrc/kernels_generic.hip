// Small kernels of the decode step shared by the bf16 and the float32 configuration (gfx950,
// wave64): RMSNorm, step inputs, greedy acceptance, LDLP, set-up.
#include "ae_internal.h"
#include "step_inputs.h"

namespace ae {

using bf16_t = uint16_t;

__device__ __forceinline__ float bf2f(bf16_t h) { return __uint_as_float((uint32_t)h << 16); }

template <typename T>
__device__ __forceinline__ float ld1(const T *p);
template <>
__device__ __forceinline__ float ld1<float>(const float *p) { return *p; }
template <>
__device__ __forceinline__ float ld1<bf16_t>(const bf16_t *p) { return bf2f(*p); }

// 8 consecutive weights -> float[8] with 128-bit loads
struct Raw8f { float4 a, b; };
__device__ __forceinline__ Raw8f raw8(const float *p) { return Raw8f{*reinterpret_cast<const float4 *>(p), *reinterpret_cast<const float4 *>(p + 4)}; }
__device__ __forceinline__ uint4 raw8(const bf16_t *p) { return *reinterpret_cast<const uint4 *>(p); }
__device__ __forceinline__ void unpack8(const Raw8f &r, float *w) {
  w[0] = r.a.x; w[1] = r.a.y; w[2] = r.a.z; w[3] = r.a.w; w[4] = r.b.x; w[5] = r.b.y; w[6] = r.b.z; w[7] = r.b.w;
}
__device__ __forceinline__ void unpack8(const uint4 &a, float *w) {
  w[0] = __uint_as_float(a.x << 16); w[1] = __uint_as_float(a.x & 0xffff0000u);
  w[2] = __uint_as_float(a.y << 16); w[3] = __uint_as_float(a.y & 0xffff0000u);
  w[4] = __uint_as_float(a.z << 16); w[5] = __uint_as_float(a.z & 0xffff0000u);
  w[6] = __uint_as_float(a.w << 16); w[7] = __uint_as_float(a.w & 0xffff0000u);
}
template <typename T>
__device__ __forceinline__ void ld8(const T *p, float *w) { unpack8(raw8(p), w); }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ __forceinline__ float silu_f(float x) { return x / (1.0f + expf(-x)); }

// ------------------------------------------------------------------ RMSNorm
// out = (x / sqrt(mean(x^2) + eps)) * g, one workgroup per row
__global__ __launch_bounds__(256) void rmsnorm_kernel(const float *x, const float *g, int d, float eps, float *out) {
  rmsnorm_row(x + (size_t)blockIdx.x * d, g, d, eps, out + (size_t)blockIdx.x * d);
}

void launch_rmsnorm(const float *x, const float *g, int rows, int d, float eps, float *out, hipStream_t s) {
  rmsnorm_kernel<<<rows, 256, 0, s>>>(x, g, d, eps, out);
}

// ------------------------------------------------------------------ tiny control kernels
// Greedy acceptance (longest draft prefix equal to the target argmax, then the target's
// own token) and the token-history side of the rollback, where no LDLP follows (one wave).
__global__ void accept_greedy_kernel(DevState *st, int32_t *hist, int kv_len, int rows, int k_on_device) {
  const int acc = greedy_accepted(st, k_on_device ? min(st->draft_len, rows - 1) : rows - 1);
  if (threadIdx.x == 0) greedy_record(st, hist, kv_len, acc);
}
void launch_accept_greedy(DevState *st, int32_t *hist, int kv_len, int rows, bool k_on_device, hipStream_t s) {
  accept_greedy_kernel<<<1, 64, 0, s>>>(st, hist, kv_len, rows, k_on_device ? 1 : 0);
}

// The host reads the device state through a mirror in pinned host memory that the device
// writes itself (no copy engine, no blit kernel) and polls its flag word (a stream synchronisation takes
// about 10 us longer to notice).
__device__ __forceinline__ void publish_state(const DevState *st, HostMirror *mirror, uint32_t seq) {
  const uint32_t *src = reinterpret_cast<const uint32_t *>(st);
  uint32_t *dst = reinterpret_cast<uint32_t *>(&mirror->st);
  for (int i = threadIdx.x; i < (int)(sizeof(DevState) / 4); i += blockDim.x) dst[i] = src[i];
  __threadfence_system();
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(&mirror->published, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}
__global__ void publish_state_kernel(const DevState *st, HostMirror *mirror, uint32_t seq) { publish_state(st, mirror, seq); }
void launch_publish_state(const DevState *st, HostMirror *mirror, uint32_t seq, hipStream_t s) {
  publish_state_kernel<<<1, 128, 0, s>>>(st, mirror, seq);
}

// The state a sequence goes on from, out of pinned host memory (the host does not wait for it).
__global__ __launch_bounds__(1024) void set_state_kernel(const float *feat, int d, float *F, int32_t *hist2, int32_t last_tok,
                                                         int32_t pending, HostMirror *mirror, uint32_t seq) {
  for (int i = threadIdx.x; i < d; i += 1024) F[i] = feat[i];
  __syncthreads();
  if (threadIdx.x == 0) {
    hist2[0] = last_tok;
    hist2[1] = pending;
    __hip_atomic_store(&mirror->imported, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}
hipError_t launch_set_state(const float *feat, int d, float *F, int32_t *hist2, int32_t last_tok, int32_t pending, HostMirror *mirror,
                            uint32_t seq, hipStream_t s) {
  return launch_checked(set_state_kernel, dim3(1), dim3(1024), s, feat, d, F, hist2, last_tok, pending, mirror, seq);
}

// One row to pinned host memory, a workgroup and a flag per piece: the host copies a piece on while the next ones are
// on their way.
__global__ __launch_bounds__(256) void export_row_kernel(const float *src, size_t n, float *dst, uint32_t *flags, uint32_t seq) {
  const size_t first = blockIdx.x * kExportPiece, end = first + kExportPiece < n ? first + kExportPiece : n;
  size_t i = first + threadIdx.x;
  if ((reinterpret_cast<uintptr_t>(src) & 15) == 0) {   // else: a row of an odd vocabulary
    for (size_t k = first + threadIdx.x * 4; k < first + kExportPiece; k += 1024)
      if (k + 4 <= end) *reinterpret_cast<float4 *>(dst + k) = *reinterpret_cast<const float4 *>(src + k);
    i += (end - first) / 4 * 4;
  }
  for (; i < end; i += 256) dst[i] = src[i];
  __threadfence_system();
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(flags + blockIdx.x, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}
hipError_t launch_export_row(const float *src, size_t n, float *dst, uint32_t *flags, uint32_t seq, hipStream_t s) {
  return launch_checked(export_row_kernel, dim3((n + kExportPiece - 1) / kExportPiece), dim3(256), s, src, n, dst, flags, seq);
}

// ------------------------------------------------------------------ LDLP (Eq. 3)
// Input layer z0 = W_in u + b_in with u = [e ; f] (in_mode 0) or f (in_mode 1) read in place:
// e = embedding of the last validated token (hist[slot]), f = its feature row F[f_row].  When
// use_nacc is set, slot and row are taken relative to the acceptance result that an earlier
// kernel left in *st; with ga.st set it is the greedy one, which every wave works out for itself (one load
// of block and argmax) and the first workgroup records.  One wave per output, lanes stride over the input in 8-element pieces
// (the summation order of the generic GEMM).
template <typename T>
__global__ __launch_bounds__(256) void ldlp_in_kernel(const T *W, const float *bias, const T *emb, const int32_t *hist,
                                                      const float *F, int d, int in_mode, int h, int slot, int f_row,
                                                      int use_nacc, const DevState *st, const GreedyAccept ga, float *z0) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int n = blockIdx.x * 4 + wave;
  const int K = in_mode == 0 ? 2 * d : d;
  const T *wrow = W + (size_t)min(n, h - 1) * K;
  // weights of the first pieces set out before the token and its slot are known: two trips to memory instead of three
  // (7B 9.7 -> 8.7 us)
  constexpr int PF = 8;
  const bool ahead = K >= PF * 512;
  decltype(raw8(W)) pf[PF];
#pragma unroll
  for (int i = 0; i < PF; ++i)
    if (ahead) pf[i] = raw8(wrow + lane * 8 + i * 512);
  int add = 0;
  int32_t tok;
  if (ga.st) {
    add = greedy_accepted(ga.st, ga.k_on_device ? min(ga.st->draft_len, ga.rows - 1) : ga.rows - 1);
    tok = ga.st->block[add];
    if (blockIdx.x == 0 && threadIdx.x == 0) greedy_record(ga.st, ga.hist, ga.kv_len, add);
  } else {
    if (use_nacc) add = st->n_acc;
    tok = hist[slot + add];
  }
  if (n >= h) return;
  const float *f = F + (size_t)(f_row + add) * d;
  const T *e = emb + (size_t)tok * d;
  float acc = 0.f;
  // unrolled so that several iterations' loads are in flight; the products still join acc in index order
  const auto join = [&](const auto &wr, int k0) {
    float w[8], x[8];
    unpack8(wr, w);
    if (in_mode == 0 && k0 < d) ld8(e + k0, x);
    else ld8(f + (in_mode == 0 ? k0 - d : k0), x);
#pragma unroll
    for (int j = 0; j < 8; ++j) acc = fmaf(x[j], w[j], acc);
  };
#pragma unroll
  for (int i = 0; i < PF; ++i)
    if (ahead) join(pf[i], lane * 8 + i * 512);
#pragma unroll 8
  for (int k0 = lane * 8 + (ahead ? PF * 512 : 0); k0 < K; k0 += 512) join(raw8(wrow + k0), k0);
  acc = wave_sum(acc);
  if (lane == 0) z0[n] = acc + bias[n];
}

void launch_ldlp_in(const void *W, const float *bias, const void *emb, int dtype, const int32_t *hist, const float *F, int d,
                    int in_mode, int h, int slot, int f_row, const DevState *st_nacc, const GreedyAccept &ga, float *z0,
                    hipStream_t s) {
  const int use = st_nacc != nullptr;
  const dim3 grid((h + 3) / 4);
  if (dtype == AE_BF16)
    ldlp_in_kernel<bf16_t><<<grid, 256, 0, s>>>((const bf16_t *)W, bias, (const bf16_t *)emb, hist, F, d, in_mode, h, slot,
                                                f_row, use, st_nacc, ga, z0);
  else
    ldlp_in_kernel<float><<<grid, 256, 0, s>>>((const float *)W, bias, (const float *)emb, hist, F, d, in_mode, h, slot,
                                               f_row, use, st_nacc, ga, z0);
}

// z0 = W_in u + b_in comes from the GEMM; here: residual blocks z += silu(W_r z + b_r),
// y = w_out . silu(z) + b_out, k = clamp(round_half_even(y), 0, k_max)  (Eq. 3).
// cls != 0: the classification variant (Sec. 4.3 ablation), one score per length 0..k_max,
// k = argmax (lowest length on ties), y_next = the winning score.
template <typename T>
__global__ __launch_bounds__(1024) void ldlp_tail_kernel(const float *z0, const T *w_res, const float *b_res,
                                                         const float *w_out, const float *b_out, int h, int n_res,
                                                         int k_max, int cls, DevState *st, HostMirror *mirror,
                                                         uint32_t seq) {
  __shared__ float z[kMaxLdlpHidden];
  __shared__ float t[kMaxLdlpHidden];
  static_assert(sizeof(DevState) % 4 == 0 && sizeof(DevState) / 4 <= 1024, "a word of the state a thread");
  const int i = threadIdx.x;
  // read beside z0, not behind the sums; with one barrier to the sum instead of ten 7.2 -> 6.4 us
  const uint32_t word = i < (int)(sizeof(DevState) / 4) ? reinterpret_cast<const uint32_t *>(st)[i] : 0u;
  const float wo = i < h ? w_out[i] : 0.f, bo = b_out[0];
  if (i < h) z[i] = z0[i];
  __syncthreads();
  for (int r = 0; r < n_res; ++r) {
    if (i < h) {
      const T *row = w_res + ((size_t)r * h + i) * h;
      float a = 0.f;
      for (int j = 0; j < h; ++j) a = fmaf(z[j], ld1(row + j), a);
      t[i] = silu_f(a + b_res[(size_t)r * h + i]);
    }
    __syncthreads();
    if (i < h) z[i] += t[i];
    __syncthreads();
  }
  const float a = i < h ? silu_f(z[i]) : 0.f;
  int best = 0;
  float best_y = 0.f;
  for (int c = 0; c < (cls ? k_max + 1 : 1); ++c) {
    t[i] = i < h ? a * (c == 0 ? wo : w_out[(size_t)c * h + i]) : 0.f;
    __syncthreads();
    if (i < 64) {   // fixed-shape tree over 1024 values: i and i + 512, then + 256, ... + 1
      float v[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) v[j] = t[i + 64 * j];
#pragma unroll
      for (int o = 8; o > 0; o >>= 1)
#pragma unroll
        for (int j = 0; j < o; ++j) v[j] += v[j + o];
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) v[0] += __shfl_down(v[0], o, 64);
      if (i == 0) {
        const float y = v[0] + (c == 0 ? bo : b_out[c]);
        if (c == 0 || y > best_y) { best = c; best_y = y; }
      }
    }
    __syncthreads();
  }
  if (i == 0) {
    int k = best;
    if (!cls) {
      float r = rintf(best_y);  // round half to even
      if (!(r >= 0.f)) r = 0.f;
      if (r > (float)k_max) r = (float)k_max;
      k = (int)r;
    }
    st->y_next = best_y;
    st->k_next = k;
    mirror->st.y_next = best_y;
    mirror->st.k_next = k;
  }
  // the rest of the state (acceptance result, block ids, draft bookkeeping) was written by earlier kernels
  static_assert(offsetof(DevState, y_next) == offsetof(DevState, k_next) + 4, "k_next and y_next are adjacent words");
  constexpr int kSkip = offsetof(DevState, k_next) / 4;
  if (i < (int)(sizeof(DevState) / 4) && i != kSkip && i != kSkip + 1) reinterpret_cast<uint32_t *>(&mirror->st)[i] = word;
  __threadfence_system();
  __syncthreads();
  if (i == 0) __hip_atomic_store(&mirror->published, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

void launch_ldlp_tail(const float *z0, const void *w_res, int dtype, const float *b_res, const float *w_out,
                      const float *b_out, int h, int n_res, int k_max, int cls, DevState *st, HostMirror *mirror,
                      uint32_t seq, hipStream_t s) {
  if (dtype == AE_BF16)
    ldlp_tail_kernel<bf16_t><<<1, 1024, 0, s>>>(z0, (const bf16_t *)w_res, b_res, w_out, b_out, h, n_res, k_max, cls, st,
                                                mirror, seq);
  else
    ldlp_tail_kernel<float><<<1, 1024, 0, s>>>(z0, (const float *)w_res, b_res, w_out, b_out, h, n_res, k_max, cls, st,
                                               mirror, seq);
}

// ------------------------------------------------------------------ set-up helpers
// (cos, sin) of pos * base^(-2i/hd), evaluated in double and rounded once to float
__global__ void rope_table_kernel(float2 *tab, int n_pos, int half, int head_dim, double base) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n_pos * half) return;
  const int p = idx / half, i = idx % half;
  const double inv = pow(base, -2.0 * (double)i / (double)head_dim);
  const double ang = (double)p * inv;
  tab[idx] = make_float2((float)cos(ang), (float)sin(ang));
}

void launch_rope_table(float2 *tab, int n_pos, int head_dim, float base, hipStream_t s) {
  const int half = head_dim / 2, n = n_pos * half;
  rope_table_kernel<<<(n + 255) / 256, 256, 0, s>>>(tab, n_pos, half, head_dim, (double)base);
}

__global__ void fill_zero_kernel(uint4 *p, size_t n16) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x)
    p[i] = make_uint4(0, 0, 0, 0);
}

void launch_fill_zero(void *p, size_t bytes, hipStream_t s) {  // bytes must be a multiple of 16
  fill_zero_kernel<<<2048, 256, 0, s>>>((uint4 *)p, bytes / 16);
}

}  // namespace ae
