// Float32 models (weights, activations and KV cache in float32) on the gfx950 matrix cores.
//
// Everything but the prompt GEMM multiplies with v_mfma_f32_16x16x4_f32: operands and accumulators stay float32, the
// weights are read in the caller's row-major layout.  A lane (g = lane/16, m = lane%16) feeds four
// consecutive k of one row (one 128-bit load) to four instructions, element e of every lane to
// instruction e: the order of k inside a sum is free, so the A operand (weight row m) and the B
// operand (activation row m) need no shuffles.  The accumulator holds weight rows 4g..4g+3 of
// activation row m: the tile layout of the bf16 kernels, and the same epilogues in float32.
//
//  * gemm_f32_kernel: up to 16 activation rows (decode, verify).  HBM-bound: a workgroup owns one
//    block of 16 weight rows (gate/up: one of each) and all of K, dealt to its waves in pieces of 64.
//    One kernel for every row count, so a row's result does not depend on the rows beside it.
//  * gemm_f32_dense_kernel: prompts.  Bound by the matrix cores, which there multiply float32 numbers as three bf16 parts
//    each: tiles of 128 weight rows x 16, 32, 48 or 64 activation rows through LDS.
//  * attn_f32_kernel: split-KV attention of up to 16 rows; attn_prefill_f32_kernel: causal flash
//    attention of a prompt chunk.
// Every product that joins an accumulator is rounded, so long sums are cut.  Counted in variances of one rounding at
// the result's magnitude, a chain of c products costs c / 2, a chain of n sums of c products n / 2, and what is left
// of K then K / (2 c n).  The sums that a wave of scalar code makes (64 lanes, each a chain of K / 64 products, and a
// butterfly) cost K / 128 + 6 of these, and neither GEMM may cost more: the decode GEMM cuts at 16 products (8 where K
// is below 1024) and adds wave results as a tree.  The prompt GEMM's instruction adds 32 products with fewer roundings;
// its chains of three instructions (six where K is 4096 and more, but not in 64-row tiles of widths that end within a tile) join one
// total.
// The flash attention adds its accumulators to a second set every 256 keys.
#include "ae_internal.h"
#include "attn_merge.h"
#include "gemm_epilogue.h"
#include "packed.h"
#include "step_inputs.h"

namespace ae {

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Loads are waited for by counting those behind them: the compiler may not change their order here.
__device__ __forceinline__ void keep_order() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

struct F32Args {
  const float *W[3];    // row-major sources: q, k, v (EPI_QKV), gate, up (EPI_SWIGLU), or one
  int seg_nb[3];        // EPI_QKV: exclusive end of each source in row-blocks
  int N, K;             // output rows of a source (EPI_QKV: of all), inner dimension (multiple of 8)
  int NB;               // row-blocks of 16 output rows
  const float *X;       // activations, row r at X + r * ldx
  int ldx, rows, row0;  // output row m reads activation row row0 + m
  const u32x4 *Xp;      // prompt GEMM: activations in three bf16 planes (see below) of RB row-blocks
  u32x4 *Xp_out;        // ... EPI_SWIGLU: and its output
  int RB;
  const float *ssq_in;  // NORM: [P_in][16] partial sums of x^2
  int P_in;
  float eps;
  const float *bias;
  float *Y;             // EPI_QKV: q; EPI_RESID: residual stream, updated in place
  int ldy;
  float *Xo;            // output times gain_out for the next GEMM (nullable), with partial sums of x^2
  int ldxo;
  const float *gain_out;
  float *ssq_out;
  float *amax_val, *lse_sum;
  int32_t *amax_idx;
  float lse_inv_t;
  const float2 *rope_tab;
  float *Kc, *Vc;       // this layer's cache (layouts of kernels_attn.hip)
  int pos0, n_ctx, hd;
  const int32_t *gate;
  int splits;           // EPI_PART: pieces of K, piece s -> Y + s * rows * N
  // prompt GEMM, EPI_QKV and EPI_SWIGLU: tiles behind the first `whole` (`tail` of them) are made in tail_splits pieces of K,
  // tile t's piece s -> tail_part, for f32_tail_kernel
  int whole, tail, tail_splits;
  f32x4 *tail_part;
};
enum { EPI_PART = 4 };  // prompt GEMM: raw partial sums over a piece of K

// Weight row that lane m of row-block nb feeds, and its source.  The rows of every q and k head are
// taken in rotary-pair order: tile j of a head holds rows 8j..8j+7 and their partners hd/2+8j.., so
// that a pair sits in lanes l and l^32 of one accumulator.
struct F32Rows {
  const float *base;   // the same for all lanes
  int row;             // this lane's row behind it
};
template <int EPI>
__device__ __forceinline__ F32Rows f32_weight_rows(const F32Args &a, int nb, int m) {
  if (EPI == EPI_QKV) {
    int si = 0, nbs = nb;
    if (nb >= a.seg_nb[0]) { si = 1; nbs = nb - a.seg_nb[0]; }
    if (nb >= a.seg_nb[1]) { si = 2; nbs = nb - a.seg_nb[1]; }
    if (si < 2) {
      const int bph = a.hd >> 4, head = nbs / bph, j = nbs % bph;
      return F32Rows{a.W[si] + (size_t)head * a.hd * a.K, m < 8 ? 8 * j + m : (a.hd >> 1) + 8 * j + m - 8};
    }
    return F32Rows{a.W[si] + (size_t)nbs * 16 * a.K, m};
  }
  return F32Rows{a.W[0] + (size_t)nb * 16 * a.K, min(m, a.N - 1 - nb * 16)};
}
template <int EPI>
__device__ __forceinline__ const float *f32_weight_row(const F32Args &a, int nb, int m) {
  const F32Rows r = f32_weight_rows<EPI>(a, nb, m);
  return r.base + (size_t)r.row * a.K;
}

template <int EPI>
__device__ __forceinline__ EpiPre f32_epi_prefetch(const F32Args &a, int nb, int g, int row, bool row_ok) {
  EpiPre p;
  p.a = make_float4(0.f, 0.f, 0.f, 0.f);
  p.b = make_float4(1.f, 1.f, 1.f, 1.f);
  if (EPI == EPI_QKV) {
    if (nb < a.seg_nb[1]) {   // (cos, sin) of the lane's two rotary pairs at the row's slot
      const int nbs = nb < a.seg_nb[0] ? nb : nb - a.seg_nb[0], j = nbs % (a.hd >> 4);
      const float2 *t = a.rope_tab + (size_t)(a.pos0 + (row_ok ? row : 0)) * (a.hd >> 1) + 8 * j + 4 * (g & 1);
      p.a = *reinterpret_cast<const float4 *>(t);
      p.b = *reinterpret_cast<const float4 *>(t + 2);
    }
  } else if (EPI == EPI_RESID || EPI == EPI_STORE) {
    const int n = nb * 16 + 4 * g;
    if (row_ok && n < a.N) {
      if (EPI == EPI_RESID) p.a = *reinterpret_cast<const float4 *>(a.Y + (size_t)row * a.ldy + n);
      else if (a.bias) p.a = *reinterpret_cast<const float4 *>(a.bias + n);
      if (a.Xo && a.gain_out) p.b = *reinterpret_cast<const float4 *>(a.gain_out + n);
    }
  }
  return p;
}

// s = accumulator of row-block nb (EPI_SWIGLU: of the gate, u = of the up projection); the lane holds
// output columns 16*nb + 4g .. +3 of activation row `row`.  Only the LM head (amax_val set) may have a
// number of columns that is no multiple of 8.  Every lane of the wave must call this (it shuffles).
template <int EPI>
__device__ __forceinline__ void f32_epi(const F32Args &a, f32x4 s, f32x4 u, int nb, int g, int m, int row, bool row_ok,
                                        float rinv, const EpiPre &pre) {
  const int n = nb * 16 + 4 * g;
  const bool ok = row_ok && n < a.N;
  if (EPI == EPI_PART) {
    if (ok) *reinterpret_cast<f32x4 *>(a.Y + ((size_t)blockIdx.y * a.rows + row) * a.N + n) = s;
  } else if (EPI == EPI_SWIGLU) {
    if (ok)
      *reinterpret_cast<float4 *>(a.Y + (size_t)row * a.ldy + n) =
          make_float4(silu_dev(s[0] * rinv) * (u[0] * rinv), silu_dev(s[1] * rinv) * (u[1] * rinv),
                      silu_dev(s[2] * rinv) * (u[2] * rinv), silu_dev(s[3] * rinv) * (u[3] * rinv));
  } else if (EPI == EPI_QKV) {
    int si = 0, nbs = nb;
    if (nb >= a.seg_nb[0]) { si = 1; nbs = nb - a.seg_nb[0]; }
    if (nb >= a.seg_nb[1]) { si = 2; nbs = nb - a.seg_nb[1]; }
    const int hd = a.hd, bph = hd >> 4, head = nbs / bph, j = nbs % bph, slot = a.pos0 + row;
    float4 o = make_float4(s[0] * rinv, s[1] * rinv, s[2] * rinv, s[3] * rinv);
    if (si < 2) {
      const float sgn = g < 2 ? -1.f : 1.f;   // first half: a*c - b*s; second half: b*c + a*s
      const float p0 = __shfl_xor(o.x, 32, 64), p1 = __shfl_xor(o.y, 32, 64);
      const float p2 = __shfl_xor(o.z, 32, 64), p3 = __shfl_xor(o.w, 32, 64);
      o.x = o.x * pre.a.x + sgn * p0 * pre.a.y;
      o.y = o.y * pre.a.z + sgn * p1 * pre.a.w;
      o.z = o.z * pre.b.x + sgn * p2 * pre.b.y;
      o.w = o.w * pre.b.z + sgn * p3 * pre.b.w;
      const int dcol = (g < 2 ? 0 : hd >> 1) + 8 * j + 4 * (g & 1);
      if (row_ok) {
        if (si == 0) *reinterpret_cast<float4 *>(a.Y + (size_t)row * a.ldy + head * hd + dcol) = o;
        else *reinterpret_cast<float4 *>(a.Kc + (((size_t)head * (hd >> 3) + (dcol >> 3)) * a.n_ctx + slot) * 8 + (dcol & 7)) = o;
      }
    } else if (row_ok) {
      *reinterpret_cast<float4 *>(a.Vc + ((size_t)head * a.n_ctx + slot) * hd + j * 16 + 4 * g) = o;
    }
  } else if (EPI == EPI_STORE && a.amax_val) {   // LM head: logits, argmax and softmax partials of the row-block
    float v[4] = {s[0] * rinv, s[1] * rinv, s[2] * rinv, s[3] * rinv};
    float bv = -INFINITY;
    int bi = 0x7fffffff;
    float *yp = a.Y + (size_t)row * a.ldy + n;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (row_ok && n + e < a.N) {
        yp[e] = v[e];
        if (v[e] > bv) { bv = v[e]; bi = n + e; }
      } else {
        v[e] = -INFINITY;
      }
    }
#pragma unroll
    for (int o = 16; o < 64; o <<= 1) {
      const float ov = __shfl_xor(bv, o, 64);
      const int oi = __shfl_xor(bi, o, 64);
      if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
    }
    if (g == 0) { a.amax_val[(size_t)m * a.NB + nb] = bv; a.amax_idx[(size_t)m * a.NB + nb] = bi; }
    if (a.lse_sum) {
      float t = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) t += v[e] == -INFINITY ? 0.f : expf((v[e] - bv) * a.lse_inv_t);   // NaN stays NaN
      t += __shfl_xor(t, 16, 64);
      t += __shfl_xor(t, 32, 64);
      if (g == 0) a.lse_sum[(size_t)m * a.NB + nb] = t;
    }
  } else if (EPI == EPI_STORE && a.N % 8 != 0) {   // LM head without partials (a sampled draft token)
    if (row_ok)
      for (int e = 0; e < 4; ++e)
        if (n + e < a.N) a.Y[(size_t)row * a.ldy + n + e] = s[e] * rinv;
  } else {
    const float4 o = make_float4(s[0] * rinv + pre.a.x, s[1] * rinv + pre.a.y, s[2] * rinv + pre.a.z, s[3] * rinv + pre.a.w);
    float ssq = 0.f;
    if (ok) {
      *reinterpret_cast<float4 *>(a.Y + (size_t)row * a.ldy + n) = o;
      if (a.Xo) {
        ssq = o.x * o.x + o.y * o.y + o.z * o.z + o.w * o.w;
        *reinterpret_cast<float4 *>(a.Xo + (size_t)row * a.ldxo + n) =
            make_float4(o.x * pre.b.x, o.y * pre.b.y, o.z * pre.b.z, o.w * pre.b.w);
      }
    }
    if (a.ssq_out) {
      ssq += __shfl_xor(ssq, 16, 64);
      ssq += __shfl_xor(ssq, 32, 64);
      if (g == 0) a.ssq_out[(size_t)nb * 16 + m] = ssq;
    }
  }
}

// ------------------------------------------------------------------ decode GEMM (1..16 rows)
// HBM-bound: each weight is read once.  A workgroup owns one block of 16 weight rows (gate/up: one of each) and all
// of K, dealt to its waves in chunks of 64 in two parts; a wave keeps a chunk (4 KB; gate/up: 8 KB) in flight.  (Twice as
// much takes 1 % longer, four times 6 %: fewer workgroups fit.)
// The rows of a row-major matrix lie a power of two apart, so workgroups that walk K in step ask the same few memory
// channels: each starts at a chunk of its own (7B widths, microseconds: o / down 29.6 -> 25.5, draft fc 35.0 -> 23.9,
// a draft token's LM head 105 -> 95; gate/up 76 -> 74 and QKV 42 -> 40 were spread by themselves).
// The address unit takes 16 lanes at a time and a cycle for every line they touch: with a row a lane, as the products
// want the weights, 64 cycles for 1 KB (a CU then gets 16 bytes a cycle at most).  So eight lanes read the 128 bytes of a row
// one after the other, straight into LDS, and the products take them from there.
// Cutting the chains at 16 products with one total per matrix is free; four totals cost 5 % (registers).
// What lies behind the end of K is out of range of the loads and read as zeros.
template <int EPI, bool NORM, int NW, bool GATED>
__global__ __launch_bounds__(NW * 64) void gemm_f32_kernel(const F32Args a) {
  constexpr int NA = EPI == EPI_SWIGLU ? 2 : 1;                // matrices
  constexpr int VM = 2 * NA + 2;                               // loads of half a chunk
  constexpr int CH = NW == 8 ? 4 : 2;                          // loads per chain of products
  // [wave][matrix][slot] for each half of a chunk: arrays of their own, so that the compiler can tell a read of one from a
  // load into the other
  __shared__ u32x4 r0[NW * NA * 128], r1[NW * NA * 128];
  if constexpr (GATED) AE_GATE(a.gate);
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 4, m = lane & 15;
  const int nb = blockIdx.x, K = a.K;
  const bool row_ok = m < a.rows;
  const int xrow = a.row0 + (row_ok ? m : a.rows - 1);   // rows beyond the block re-read the last row

  EpiPre pre{};
  if (w == 0) pre = f32_epi_prefetch<EPI>(a, nb, g, m, row_ok);

  constexpr int kRange = 0x7ffffff0;
  __amdgpu_buffer_rsrc_t rw[2];
  unsigned vw[2][2];
  int kw[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int r = h * 8 + (lane >> 3);
    kw[h] = 4 * ((lane & 7) ^ (r >> 1));   // slot r * 8 + q holds piece q ^ (r / 2) of row r: reads without conflicts
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const F32Rows t = EPI == EPI_SWIGLU ? F32Rows{a.W[i] + (size_t)nb * 16 * K, min(r, a.N - 1 - nb * 16)} : f32_weight_rows<EPI>(a, nb, r);
      rw[i] = __builtin_amdgcn_make_buffer_rsrc((void *)t.base, 0, kRange, 0x00020000);
      vw[i][h] = ((unsigned)t.row * K + kw[h]) * 4;
    }
  }
  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void *)a.X, 0, kRange, 0x00020000);
  const unsigned vx = ((unsigned)xrow * a.ldx + 4 * g) * 4;
  const int as = m * 8 + (g ^ (m >> 1));   // where this lane's weights are: piece g, and piece 4 + g at as ^ 4

  const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 acc[NA][4], tot[NA];
  u32x4 xb[2][2];
#pragma unroll
  for (int i = 0; i < NA; ++i) tot[i] = zero;
  const int NC = (K + 63) / 64, rot = (int)((unsigned)nb * 7u % (unsigned)NC);
  auto first_k = [&](int c, int half) {   // chunks behind the last one read nothing
    const int r = c + rot;
    return c < NC ? (r < NC ? r : r - NC) * 64 + half * 32 : K;
  };
  auto issue_w = [&](int c, int half, u32x4 *slot) {
    const int k = first_k(c, half);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const bool in = k + kw[h] < K;
#pragma unroll
      for (int i = 0; i < NA; ++i)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rw[i], (__attribute__((address_space(3))) void *)(slot + (w * NA + i) * 128 + h * 64), 16,
                                                 in ? vw[i][h] : kRange, k * 4, 0, 0);
    }
  };
  auto issue_x = [&](int c, int half, u32x4 (&x)[2]) {
    const int k = first_k(c, half);
#pragma unroll
    for (int j = 0; j < 2; ++j) x[j] = __builtin_amdgcn_raw_buffer_load_b128(rx, k + 16 * j + 4 * g < K ? vx + 64 * j : kRange, k * 4, 0);
  };
  auto part = [&](int c, int half, u32x4 *slot, u32x4 (&x)[2]) {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xf70 | VM);   // vmcnt: all but the part behind
    asm volatile("" ::: "memory");
    f32x4 wv[NA][2];
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) wv[i][j] = __builtin_bit_cast(f32x4, slot[(w * NA + i) * 128 + (j ? as ^ 4 : as)]);
#pragma unroll
    for (int i = 0; i < NA; ++i) asm volatile("" : "+v"(wv[i][0]), "+v"(wv[i][1]));   // read before the slot is filled again
    issue_w(c + NW, half, slot);
    keep_order();
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int n = half * 2 + j;
      const f32x4 xv = __builtin_bit_cast(f32x4, x[j]);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < NA; ++i) acc[i][e] = mfma_f32(wv[i][j][e], xv[e], n % CH == 0 ? zero : acc[i][e]);
      if (n % CH == CH - 1) {
#pragma unroll
        for (int i = 0; i < NA; ++i) tot[i] += (acc[i][0] + acc[i][1]) + (acc[i][2] + acc[i][3]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    issue_x(c + NW, half, x);
    keep_order();
  };
  issue_w(w, 0, r0);
  keep_order();
  issue_x(w, 0, xb[0]);
  keep_order();
  issue_w(w, 1, r1);
  keep_order();
  issue_x(w, 1, xb[1]);
  keep_order();

  // 1/rms of every row from the producer's partial sums of x^2, summed by wave 0 in a fixed order
  __shared__ float rinv_s[16];
  if (NORM && w == 0) {
    const float4 *pp = reinterpret_cast<const float4 *>(a.ssq_in);
    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
    for (int i = lane; i < a.P_in * 4; i += 64) {   // lane l covers rows 4*(l%4)..+3
      const float4 v = pp[i];
      t.x += v.x; t.y += v.y; t.z += v.z; t.w += v.w;
    }
#pragma unroll
    for (int o = 4; o < 64; o <<= 1) {
      t.x += __shfl_xor(t.x, o, 64); t.y += __shfl_xor(t.y, o, 64);
      t.z += __shfl_xor(t.z, o, 64); t.w += __shfl_xor(t.w, o, 64);
    }
    if (lane < 4) {
      rinv_s[lane * 4 + 0] = 1.0f / sqrtf(t.x / (float)K + a.eps);
      rinv_s[lane * 4 + 1] = 1.0f / sqrtf(t.y / (float)K + a.eps);
      rinv_s[lane * 4 + 2] = 1.0f / sqrtf(t.z / (float)K + a.eps);
      rinv_s[lane * 4 + 3] = 1.0f / sqrtf(t.w / (float)K + a.eps);
    }
  }

  for (int c = w; c < NC; c += NW) {
    part(c, 0, r0, xb[0]);
    part(c, 1, r1, xb[1]);
  }
  __builtin_amdgcn_s_waitcnt(0xf70);   // vmcnt(0): no load into LDS outlives the loop
#pragma unroll
  for (int i = 0; i < NA; ++i) r0[(w * NA + i) * 128 + lane] = __builtin_bit_cast(u32x4, tot[i]);   // the wave's own part of the ring
  __syncthreads();
  if (w != 0) return;
  f32x4 t[NW][NA];
#pragma unroll
  for (int ww = 0; ww < NW; ++ww)
#pragma unroll
    for (int i = 0; i < NA; ++i) t[ww][i] = __builtin_bit_cast(f32x4, r0[(ww * NA + i) * 128 + lane]);
#pragma unroll
  for (int o = 1; o < NW; o *= 2)
#pragma unroll
    for (int ww = 0; ww < NW; ww += 2 * o)
#pragma unroll
      for (int i = 0; i < NA; ++i) t[ww][i] += t[ww + o][i];
  const f32x4 s = t[0][0], u = t[0][NA - 1];
  f32_epi<EPI>(a, s, u, nb, g, m, m, row_ok, NORM ? rinv_s[xrow] : 1.f, pre);
}

static F32Args f32_args(const GemmLaunch &L) {
  F32Args a{};
  const Mat &W = *L.W;
  for (int i = 0; i < 3; ++i) a.W[i] = (const float *)(W.part[i] ? W.part[i] : W.rowmajor);
  a.K = W.K;
  a.N = L.epi == EPI_SWIGLU ? W.N / 2 : W.N;
  a.NB = (a.N + 15) / 16;
  int end = 0;
  for (int i = 0; i < 3; ++i) a.seg_nb[i] = end += L.epi == EPI_QKV ? L.seg_N[i] / 16 : 0;
  if (L.epi == EPI_QKV) { a.NB = end; a.N = end * 16; }
  a.X = (const float *)L.Xp; a.ldx = L.ldx; a.rows = L.rows; a.row0 = L.row0;
  a.ssq_in = L.ssq_in; a.P_in = L.P_in; a.eps = L.eps;
  a.bias = L.bias;
  a.Y = L.Y[0]; a.ldy = L.ldy[0];
  a.Xo = (float *)L.Xp_out; a.ldxo = L.ldxo; a.gain_out = L.gain_out; a.ssq_out = L.ssq_out;
  if (L.epi == EPI_SWIGLU) { a.Y = (float *)L.Xp_out; a.ldy = L.ldxo; a.Xo = nullptr; }
  a.amax_val = L.amax_val; a.amax_idx = L.amax_idx;
  a.lse_sum = L.amax_val ? L.lse_sum : nullptr; a.lse_inv_t = L.lse_inv_t;
  a.rope_tab = L.rope_tab; a.Kc = (float *)L.Kc; a.Vc = (float *)L.Vc;
  a.pos0 = L.pos0; a.n_ctx = L.n_ctx; a.hd = L.hd;
  a.gate = L.gate;
  return a;
}

template <int EPI, bool NORM, int NW>
static void launch_f32_waves(const F32Args &a, hipStream_t s) {
  if (a.gate) gemm_f32_kernel<EPI, NORM, NW, true><<<a.NB, NW * 64, 0, s>>>(a);
  else gemm_f32_kernel<EPI, NORM, NW, false><<<a.NB, NW * 64, 0, s>>>(a);
}

template <int EPI, bool NORM>
static void launch_f32_cfg(const F32Args &a, hipStream_t s) {
  if (a.K >= 1024) launch_f32_waves<EPI, NORM, 8>(a, s);   // at least two pieces of 64 for each of 8 waves
  else launch_f32_waves<EPI, NORM, 4>(a, s);
}

void launch_gemm_f32(const GemmLaunch &L, hipStream_t s) {
  const F32Args a = f32_args(L);
  const bool norm = L.ssq_in != nullptr;
  if (L.epi == EPI_QKV) launch_f32_cfg<EPI_QKV, true>(a, s);
  else if (L.epi == EPI_SWIGLU) launch_f32_cfg<EPI_SWIGLU, true>(a, s);
  else if (L.epi == EPI_RESID) launch_f32_cfg<EPI_RESID, false>(a, s);
  else if (norm) launch_f32_cfg<EPI_STORE, true>(a, s);
  else launch_f32_cfg<EPI_STORE, false>(a, s);
}

// ------------------------------------------------------------------ prompt GEMM
// Products of float32 numbers on the bf16 matrix instruction.  2^24 x = hi + mid + lo in bf16 (round to nearest even; the
// remainders are exact) holds all 24 bits of x: without the factor the last part of what lies below 2^-110 would fall under
// bf16's smallest number.  Of the nine products the three smallest are left out: up to 2^-24.2 of the whole, 2^-27.4 in the
// root mean square, of either sign.  The instruction takes 6 x 16 cycles for what v_mfma_f32_16x16x4_f32 takes 256 for, and rounds once
// for several products where that rounds each.  Activations come split ("planes", written by the kernels before), weights are
// split on the way.
//
// Planes: Xp[kt][rb][hi, mid, lo][slot = row * 4 + k octet] of 16 bytes, the packed form of packed.h with three parts; what
// lies behind the end of K in the last k-tile is zero.  A number that has no such parts (2^103 and more, Inf, NaN) is kept as it
// is in mid and lo, its hi is a NaN: sums that meet one come out not finite and are made again in float32.
constexpr float kSplitScale = 0x1p24f, kSumScale = 0x1p-48f;
__device__ __forceinline__ uint32_t pack_bf16(float x0, float x1) {
  bf16x2 h;
  h[0] = (__bf16)x0; h[1] = (__bf16)x1;
  uint32_t p = __builtin_bit_cast(uint32_t, h);
  asm("" : "+v"(p));   // (else every half is converted a second time where its value is needed)
  return p;
}
// x0, x1: the numbers times 2^24
__device__ __forceinline__ void split3(float x0, float x1, uint32_t (&p)[3]) {
  p[0] = pack_bf16(x0, x1);
  const float r0 = x0 - __uint_as_float(p[0] << 16), r1 = x1 - __uint_as_float(p[0] & 0xffff0000u);
  p[1] = pack_bf16(r0, r1);
  p[2] = pack_bf16(r0 - __uint_as_float(p[1] << 16), r1 - __uint_as_float(p[1] & 0xffff0000u));
}
constexpr uint32_t kAsItIs = 0x7fffu;   // hi of a number without parts
constexpr int kPlanePieces = 192;   // 16-byte pieces of a row-block and k-tile

// Products a * b at four consecutive k (k0 % 4 == 0) of row m of the row-block whose first tile is at xp; kts: pieces from k-tile
// to k-tile.  The parts are those of the product itself, not of the float32 number that it rounds to.
__device__ __forceinline__ void planes_store4(u32x4 *xp, int m, int k0, f32x4 a, f32x4 b, size_t kts) {
  uint32_t p[2][3];
  bool odd = false;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const float a0 = a[2 * h], a1 = a[2 * h + 1], b0 = b[2 * h] * kSplitScale, b1 = b[2 * h + 1] * kSplitScale;
    const float x0 = a0 * b0, x1 = a1 * b1;
    p[h][0] = pack_bf16(x0, x1);
    const float r0 = fmaf(a0, b0, -__uint_as_float(p[h][0] << 16)), r1 = fmaf(a1, b1, -__uint_as_float(p[h][0] & 0xffff0000u));
    p[h][1] = pack_bf16(r0, r1);
    p[h][2] = pack_bf16(r0 - __uint_as_float(p[h][1] << 16), r1 - __uint_as_float(p[h][1] & 0xffff0000u));
    odd |= !(fabsf(x0) < 0x1p127f) | !(fabsf(x1) < 0x1p127f);
  }
  if (odd) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (fabsf(a[e] * (b[e] * kSplitScale)) < 0x1p127f) continue;
      const uint32_t u = __float_as_uint(a[e] * b[e]), q[3] = {kAsItIs, u >> 16, u & 0xffffu};
#pragma unroll
      for (int n = 0; n < 3; ++n) p[e >> 1][n] = e & 1 ? (p[e >> 1][n] & 0xffffu) | q[n] << 16 : (p[e >> 1][n] & 0xffff0000u) | q[n];
    }
  }
  const int g = (k0 & 31) >> 3, half = (k0 & 7) >> 2;
#pragma unroll
  for (int n = 0; n < 3; ++n) reinterpret_cast<u32x2 *>(xp + (size_t)(k0 >> 5) * kts + n * 64 + m * 4 + g)[half] = u32x2{p[0][n], p[1][n]};
}
__device__ __forceinline__ f32x4 planes_load4(const u32x4 *xp, int m, int k0, size_t kts) {
  u32x2 v[3];
#pragma unroll
  for (int n = 0; n < 3; ++n)
    v[n] = reinterpret_cast<const u32x2 *>(xp + (size_t)(k0 >> 5) * kts + n * 64 + m * 4 + ((k0 & 31) >> 3))[(k0 & 7) >> 2];
  f32x4 x;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    uint32_t q[3];
#pragma unroll
    for (int n = 0; n < 3; ++n) q[n] = e & 1 ? v[n][e >> 1] >> 16 : v[n][e >> 1] & 0xffffu;
    x[e] = q[0] == kAsItIs ? __uint_as_float(q[1] << 16 | q[2])
                           : (__uint_as_float(q[0] << 16) + (__uint_as_float(q[1] << 16) + __uint_as_float(q[2] << 16))) * (1.f / kSplitScale);
  }
  return x;
}

// Epilogue of a wave's tiles (two weight row-blocks, J activation row-blocks).
template <int EPI, int J>
__device__ __forceinline__ void f32_dense_epilogue(const F32Args &a, const f32x4 (&tot)[2][J], int nb_t, int row_t, int w, int g, int m) {
  constexpr int STEP = EPI == EPI_SWIGLU ? 2 : 1;
#pragma unroll
  for (int i = 0; i < 2; i += STEP) {
    const int nb = EPI == EPI_SWIGLU ? nb_t + w : nb_t + w * 2 + i;
    if (nb >= a.NB) continue;
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int row = row_t + j * 16 + m;
      const bool row_ok = row < a.rows;
      if (EPI == EPI_SWIGLU) {
        const int n = nb * 16 + 4 * g;
        const f32x4 s = tot[0][j], u = tot[1][j];
        if (row_ok && n < a.N)
          planes_store4(a.Xp_out + (size_t)(row >> 4) * kPlanePieces, m, n,
                        f32x4{silu_dev(s[0]), silu_dev(s[1]), silu_dev(s[2]), silu_dev(s[3])}, u, (size_t)a.RB * kPlanePieces);
        continue;
      }
      const EpiPre pre = f32_epi_prefetch<EPI>(a, nb, g, row, row_ok);
      f32_epi<EPI>(a, tot[i][j], tot[i][j], nb, g, m, row, row_ok, 1.f, pre);
    }
  }
}

// Workgroup tile: 128 weight rows (gate/up: 64 of each) x 16*J activation rows; each of the 4 waves owns two
// weight row-blocks and all J activation row-blocks.  Stages of 32 k go straight into LDS, weights three stages ahead,
// activations one.  While a stage is multiplied the weights of the next one are split, vector instructions between the
// matrix instructions: an MFMA of 16 cycles leaves room for two.  7B widths, 333 rows, against the float32 instruction, in
// tiles of 48 rows: gate/up 649 -> 356 + 5 us (the last tiles in pieces of K), QKV 408 -> 203 + 6, o / down 247 -> 140 on average; the
// factor of the split takes 16 of 118 vector instructions a stage (J = 3) and 6, 4 and 3 us of these.  With the activations split here
// too (44 vector instructions more a stage; whole tiles, without the factor: 382 and 238 us) 478 / 295.  What is left of the matrix rate
// (40 %): 3.3 vector instructions an MFMA at J = 3, latencies that two waves a SIMD do not cover, clocks of 2.05 GHz.  Such a prompt
// now takes tiles of 64 rows (one layer, 48 -> 64 rows in one process: gate/up 348 + 5 -> 330 + 9, QKV 193 + 6 -> 188 + 10).
template <int EPI, int J, bool LONG>
__global__ __launch_bounds__(256, 2) void gemm_f32_dense_kernel(const F32Args a) {
  constexpr int TM = 16 * J, CH = LONG ? 6 : 3;             // CH: stages in a chain of products
  constexpr int NX = (3 * J + 3) / 4;                       // activation tiles of 1 KB that a wave loads per stage
  // Activations of two stages [row-block][hi, mid, lo][lane], weights of three as they are [wave][row-block][slot]: arrays
  // of their own, so that the compiler can tell a read of one from a load into another.
  __shared__ u32x4 x0[J * kPlanePieces], x1[J * kPlanePieces], a0[4 * 256], a1[4 * 256], a2[4 * 256];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4, m = lane & 15;
  // the activation tiles of one weight tile run side by side on one XCD (ids go round the 8 XCDs) and share it in its L2
  constexpr int NBT = EPI == EPI_SWIGLU ? 4 : 8;            // output row-blocks per workgroup
  const int NT = (a.NB + NBT - 1) / NBT, MT = (a.rows + TM - 1) / TM;
  int id = blockIdx.x, count = NT * MT, piece = blockIdx.y, pieces = a.splits;
  const bool behind = EPI != EPI_PART && a.tail > 0 && id >= a.whole;   // a piece of one of the last tiles
  if (EPI != EPI_PART && a.tail > 0) {
    count = behind ? a.tail * a.tail_splits : a.whole;
    id -= behind ? a.whole : 0;
  }
  const int per = (count + 7) >> 3;
  int v = (id & 7) * per + (id >> 3);
  if ((id >> 3) >= per || v >= count) return;
  if (behind) {
    pieces = a.tail_splits;
    piece = v / a.tail;
    v = a.whole + v % a.tail;
  }
  const int nb_t = v / MT * NBT, row_t = (v % MT) * TM;
  // this workgroup's piece of K, in stages of 32
  int NS = (a.K + 95) / 96 * 3, lo = 0;                     // in threes
  if (EPI == EPI_PART || behind) {
    const int np = NS / 3;
    lo = np * piece / pieces * 3;
    NS = np * (piece + 1) / pieces * 3 - lo;
  }
  const int K = min(a.K, (lo + NS) * 32) - lo * 32;

  // Operands come through buffer loads: a base for the wave from the piece's first k on, a byte offset a lane, the stage in
  // a scalar; pieces behind the end of K are out of range and read as zeros.  Eight lanes take the 128 bytes of a weight row
  // one after the other: with a row a lane, as the products want them, the address unit takes four times as long.
  constexpr int kRange = 0x7ffffff0;
  const size_t kts = (size_t)a.RB * kPlanePieces;
  const unsigned kts_b = a.RB * (kPlanePieces * 16u);
  const int q = lane & 7;
  __amdgpu_buffer_rsrc_t ra[2];
  unsigned va[2][2], vx[NX];
  int ka[2];
  // row-blocks behind the last one of the chunk are not read
  const u32x4 *xbase = a.Xp + (size_t)lo * kts + (size_t)(row_t >> 4) * kPlanePieces;
  const int rbs = min(J, a.RB - (row_t >> 4));
  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void *)xbase, 0, -1, 0x00020000);
#pragma unroll
  for (int i = 0; i < NX; ++i) vx[i] = (min(w + 4 * i, 3 * rbs - 1) * 64 + m * 4 + g) * 16;   // in lane order in LDS
#pragma unroll
  for (int h = 0; h < 2; ++h) ka[h] = 4 * (q ^ ((h * 8 + (lane >> 3)) >> 1));   // slot r * 8 + q holds piece q ^ (r / 2) of row r
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r = h * 8 + (lane >> 3);
      F32Rows t;
      if (EPI == EPI_SWIGLU) {   // a gate and an up block
        const int nb = min(nb_t + w, a.NB - 1);
        t = F32Rows{a.W[i] + (size_t)nb * 16 * a.K, min(r, a.N - 1 - nb * 16)};
      } else {
        t = f32_weight_rows<EPI>(a, min(nb_t + w * 2 + i, a.NB - 1), r);
      }
      ra[i] = __builtin_amdgcn_make_buffer_rsrc((void *)(t.base + lo * 32), 0, kRange, 0x00020000);
      va[i][h] = ((unsigned)t.row * a.K + ka[h]) * 4;
    }
  auto issue_a = [&](int st, u32x4 *slot) {
    const int s = min(st, NS) * 128;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const bool in = st * 32 + ka[h] < K;
#pragma unroll
      for (int i = 0; i < 2; ++i)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(ra[i], (__attribute__((address_space(3))) void *)(slot + w * 256 + i * 128 + h * 64),
                                                 16, in ? va[i][h] : kRange, s, 0, 0);
    }
  };
  auto issue_x = [&](int st, u32x4 *slot) {   // stages without k repeat the last one (its weights are zeros)
    const unsigned s = (unsigned)min(st, (K + 31) / 32 - 1) * kts_b;
#pragma unroll
    for (int i = 0; i < NX; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (__attribute__((address_space(3))) void *)(slot + min(w + 4 * i, 3 * J - 1) * 64),
                                               16, (int)vx[i], s, 0, 0);
  };
  // every wave waits for its own loads (all but the 4 newest, weights that have two stages left), then for the others
  auto gate = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xf74);   // vmcnt(4)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  const int as = m * 8 + ((2 * g) ^ (m >> 1));   // where this lane's weights are in a tile
  f32x4 raw[2][2];   // weights of the stage that is split next
  auto read_raw = [&](const u32x4 *slot) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 2; ++e) raw[i][e] = __builtin_bit_cast(f32x4, slot[w * 256 + i * 128 + (as ^ e)]);
  };
  auto split = [&](u32x4 (&f)[2][3]) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      uint32_t p[4][3];
#pragma unroll
      for (int e = 0; e < 4; ++e) split3(raw[i][e >> 1][e % 2 * 2] * kSplitScale, raw[i][e >> 1][e % 2 * 2 + 1] * kSplitScale, p[e]);
#pragma unroll
      for (int n = 0; n < 3; ++n) {
        f[i][n] = u32x4{p[0][n], p[1][n], p[2][n], p[3][n]};
        asm volatile("" : "+v"(f[i][n]));   // here, not where it is used
      }
    }
  };
  // acc: chains of CH stages of the large products, joined in tot; sml: the small ones, whose roundings do not matter
  const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 acc[2][J], tot[2][J], sml[2][J];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < J; ++j) acc[i][j] = tot[i][j] = sml[i][j] = zero;
  u32x4 fa[2][2][3];   // split weights of stages st and st+1
  // Stage st: products with the activations xs, beside them the splitting of the weights of stage st+1 (in raw).  x1st: room for
  // the activations of stage st+1; a2nd: weights of stage st+2; far: room for those of stage st+3.
  auto stage = [&](int st, int u, const u32x4 *xs, u32x4 *x1st, const u32x4 *a2nd, u32x4 *far) __attribute__((always_inline)) {
    issue_x(st + 1, x1st);
    keep_order();
    issue_a(st + 3, far);
    keep_order();
    const u32x4 *sb = xs + lane;
    const u32x4 (&f)[2][3] = fa[u & 1];
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const u32x4 b0 = sb[(j * 3 + 0) * 64], b1 = sb[(j * 3 + 1) * 64], b2 = sb[(j * 3 + 2) * 64];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        if (u % CH == 0) tot[i][j] += acc[i][j];
        acc[i][j] = mfma_bf16(f[i][0], b0, u % CH == 0 ? zero : acc[i][j]);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) sml[i][j] = mfma_bf16(f[i][2], b0, sml[i][j]);
#pragma unroll
      for (int i = 0; i < 2; ++i) sml[i][j] = mfma_bf16(f[i][0], b2, sml[i][j]);
#pragma unroll
      for (int i = 0; i < 2; ++i) sml[i][j] = mfma_bf16(f[i][1], b1, sml[i][j]);
#pragma unroll
      for (int i = 0; i < 2; ++i) sml[i][j] = mfma_bf16(f[i][1], b0, sml[i][j]);
#pragma unroll
      for (int i = 0; i < 2; ++i) sml[i][j] = mfma_bf16(f[i][0], b1, sml[i][j]);
    }
    split(fa[(u + 1) & 1]);
    __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
#pragma unroll
    for (int n = 0; n < 12 * J; ++n) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, (96 + 12 * J - 1) / (12 * J), 0);
      if (n % 4 == 0 && n / 4 < 3 * (J - 1)) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xf70 | (NX + 4));   // vmcnt: all but what this stage asked for
    asm volatile("" ::: "memory");
    read_raw(a2nd);
    gate();
  };
  issue_a(0, a0);
  issue_a(1, a1);
  issue_x(0, x0);
  keep_order();
  issue_a(2, a2);
  gate();
  read_raw(a0);
  split(fa[0]);
  read_raw(a1);
  auto first3 = [&](int st) __attribute__((always_inline)) {
    stage(st, 0, x0, x1, a2, a0);
    stage(st + 1, 1, x1, x0, a0, a1);
    stage(st + 2, 2, x0, x1, a1, a2);
  };
  auto second3 = [&](int st) __attribute__((always_inline)) {
    stage(st + 3, 3, x1, x0, a2, a0);
    stage(st + 4, 4, x0, x1, a0, a1);
    stage(st + 5, 5, x1, x0, a1, a2);
  };
  // Sixes, then three where they are left (of three stages alone those behind the last one multiply zeros).  A way out in the
  // middle of the loop costs 40 registers of copies, which long chains at J = 4 do not have.
  int st = 0;
  if constexpr (J == 1) {
    for (; st < NS; st += 6) {
      first3(st);
      if (st + 3 >= NS) break;
      second3(st);
    }
  } else {
    do {
      first3(st);
      second3(st);
      st += 6;
    } while (st + 6 <= NS);
    if (st < NS) first3(st);
  }
  __builtin_amdgcn_s_waitcnt(0xf70);   // vmcnt(0): no load into LDS outlives the loop
  bool odd = false;
#pragma unroll
  for (int j = 0; j < J; ++j)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      tot[i][j] = (tot[i][j] + (acc[i][j] + sml[i][j])) * kSumScale;
      const f32x4 d = tot[i][j] - tot[i][j];
      odd |= row_t + j * 16 + m < a.rows && !((d[0] + d[1]) + (d[2] + d[3]) == 0.f);
    }
  if (__any(odd)) {   // Inf or NaN somewhere, a number without parts, or a sum above 2^80: these again in float32
#pragma unroll 1
    for (int j = 0; j < J; ++j) {
      const u32x4 *xp = xbase + min(j, rbs - 1) * kPlanePieces;
      const float *wp[2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
        wp[i] = (EPI == EPI_SWIGLU ? a.W[i] + (size_t)min((nb_t + w) * 16 + m, a.N - 1) * a.K
                                   : f32_weight_row<EPI>(a, min(nb_t + w * 2 + i, a.NB - 1), m)) + lo * 32;
      f32x4 s[2] = {zero, zero};
#pragma unroll 1
      for (int k = 4 * g; k - 4 * g < K; k += 16) {
        const f32x4 b = k < K ? planes_load4(xp, m, k, kts) : zero;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const f32x4 wv = k < K ? *reinterpret_cast<const f32x4 *>(wp[i] + k) : zero;
#pragma unroll
          for (int e = 0; e < 4; ++e) s[i] = mfma_f32(wv[e], b[e], s[i]);
        }
      }
#pragma unroll
      for (int jj = 0; jj < J; ++jj)
        if (jj == j)
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (!(tot[i][jj][e] - tot[i][jj][e] == 0.f)) tot[i][jj][e] = s[i][e];
    }
  }
  if (EPI != EPI_PART && pieces > 1) {
    f32x4 *out = a.tail_part + (((size_t)piece * a.tail + v - a.whole) * 4 + w) * (2 * J * 64) + lane;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < J; ++j) out[(i * J + j) * 64] = tot[i][j];
    return;
  }
  f32_dense_epilogue<EPI, J>(a, tot, nb_t, row_t, w, g, m);
}

// Adds the pieces of a tile whose K was split and runs the GEMM's epilogue on it.
template <int EPI, int J>
__global__ __launch_bounds__(256) void f32_tail_kernel(const F32Args a) {
  constexpr int NBT = EPI == EPI_SWIGLU ? 4 : 8;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, MT = (a.rows + 16 * J - 1) / (16 * J), v = a.whole + (int)blockIdx.x;
  const f32x4 *in = a.tail_part + ((size_t)blockIdx.x * 4 + w) * (2 * J * 64) + lane;
  const size_t stride = (size_t)a.tail * 4 * (2 * J * 64);
  f32x4 tot[2][J];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < J; ++j) tot[i][j] = in[(i * J + j) * 64];
  for (int s = 1; s < a.tail_splits; ++s)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < J; ++j) tot[i][j] += in[s * stride + (i * J + j) * 64];
  f32_dense_epilogue<EPI, J>(a, tot, v / MT * NBT, (v % MT) * 16 * J, w, lane >> 4, lane & 15);
}

// Tiles behind the last full round of 512 workgroups (two per compute unit), and the pieces that K of each is dealt to where
// that fills the round: at most half as many tiles as it has places, 16 stages a piece at least, room for the pieces in max_part.  7B widths, 333
// rows in tiles of 48: QKV (512 + 160 tiles, 3 pieces) 238 -> 204 + 7 us, gate/up (1024 + 180, 2 pieces) 382 -> 360 + 6.  In the 64-row
// tiles that such a prompt takes, 64 and 8 tiles are cut into eight pieces each.
struct F32Tail {
  int tiles = 0, pieces = 1;
};
static F32Tail f32_tail(long tiles, int K, int J, size_t max_part) {
  F32Tail t;
  const int left = (int)(tiles % 512), room = left ? 512 / left : 0, longest = (K + 31) / 32 / 16, S = room < longest ? room : longest;
  if (left > 0 && S > 1 && (size_t)left * S * 2048 * J <= max_part) {
    t.tiles = left;
    t.pieces = S < 8 ? S : 8;
  }
  return t;
}

// Widths that end with a tile.
template <int EPI>
static bool f32_whole(const F32Args &a) { return a.N % (EPI == EPI_SWIGLU ? 64 : 128) == 0 && a.K % 32 == 0; }

template <int EPI, int J>
static void launch_f32_dense_tile(F32Args a, hipStream_t s, size_t max_part) {
  constexpr int NBT = EPI == EPI_SWIGLU ? 4 : 8;
  const int tiles = (a.NB + NBT - 1) / NBT * ((a.rows + 16 * J - 1) / (16 * J));
  const F32Tail t = EPI == EPI_PART ? F32Tail() : f32_tail(tiles, a.K, J, max_part);
  a.whole = tiles - t.tiles;
  a.tail = t.tiles;
  a.tail_splits = t.tiles ? t.pieces : 0;
  const dim3 grid((a.whole + 7) / 8 * 8 + (a.tail * a.tail_splits + 7) / 8 * 8, a.splits);
  // the joins of a chain cost vector instructions and, of a long sum, roundings: half as many there (a 7B gate/up sum 21 instead of
  // 43; at J = 4 of whole widths alone, 500 rows 1.25e-6 -> 1.20e-6 off float64)
  if (a.K >= 4096 && (J < 4 || f32_whole<EPI>(a))) gemm_f32_dense_kernel<EPI, J, true><<<grid, 256, 0, s>>>(a);
  else gemm_f32_dense_kernel<EPI, J, false><<<grid, 256, 0, s>>>(a);
  if constexpr (EPI != EPI_PART) {
    if (a.tail > 0) f32_tail_kernel<EPI, J><<<a.tail, 256, 0, s>>>(a);
  }
}

// Microseconds of a GEMM in tiles of 16 * J rows and S pieces of K (EPI_PART).  A round of 512 workgroups takes 84, 118, 136 or 160 us
// for K = 4096 with J = 1 .. 4 (narrow tiles split their weights for fewer products), one of at most 256, alone on their
// compute units, 0.65 of that; tiles behind the last full round are cut (f32_tail) or a round of their own; a piece of K is
// written and added.  Meant for the order of plans, not for their times (0.6 of the measured ones at 20 rows of 7B, 0.85 to 1.03 from 160
// on): what it picks is 0.6, 0.6, 1.0 and 2.1 % off the best of all plans on average (7B, 13B, 2048 x 5632, 1024 x 2816; 20 to 2048 rows).  The
// pass behind cut tiles is charged 5 us; it takes 4 to 6 with J <= 2, 5 to 8 with 3, 6 to 10 with 4, which charged to them changes
// nothing of that (0.6, 0.6, 0.8, 2.0 %).
static double f32_dense_cost(bool part, long NT, const F32Args &a, int J, int S, size_t max_part) {
  static constexpr double kRound[5] = {0, 84, 118, 136, 160};
  const long tiles = NT * ((a.rows + 16 * J - 1) / (16 * J));
  const double c = kRound[J] * a.K / 4096;
  const auto rounds = [](long w) { return (double)(w / 512) + (w % 512 == 0 ? 0.0 : w % 512 <= 256 ? 0.65 : 1.0); };
  if (part) return rounds(tiles * S) * c / S + 0.9 * S + (double)S * a.rows * a.N * 4 / 5e6;
  const F32Tail t = f32_tail(tiles, a.K, J, max_part);
  return rounds(tiles - t.tiles) * c + (t.tiles ? rounds((long)t.tiles * t.pieces) * c / t.pieces + 5 : 0);
}

// The same by tiles per compute unit times rows of a tile over pieces, the older rule, for widths that end within a tile.  It is 14, 14, 7
// and 11 % off the best plan there (4104 x 11016, 2056 x 5640, 1032 x 2824, 5128 x 13832; 20 to 2048 rows), mostly by tiles of too few rows up
// to 500 rows; f32_dense_cost would be 4, 7, 2 and 4 % off (pieces of 33 or 41 tiles do not fill the 8 XCDs alike, which it does
// not count).  The tests of the tile shapes hold these widths to this rule, which reaches all shapes within 1000 rows.
static double f32_tile_count(long NT, const F32Args &a, int J, int S) {
  static constexpr double kPerRow[5] = {0, 1.4, 1.1, 1.0, 1.0};
  const long tiles = NT * ((a.rows + 16 * J - 1) / (16 * J)) * S;
  return (double)((tiles + 255) / 256 * J) / S * kPerRow[J] * (tiles <= 256 ? 1.25 : 1.0) * (1.0 + 0.03 * S);
}

// Rows of a tile and (EPI_PART) pieces of K, by f32_dense_cost.  (By f32_tile_count, which takes narrow tiles to be dearer by 10
// to 40 % and a round to have 256 places, 7B, 2 layers: 64 rows 984 us, 100 1255, 128 1297, 200 1691, 333 2206, 400 3019, 600 3848;
// so 841, 1074, 1102, 1556, 2155, 2499, 3487.)
template <int EPI>
static int launch_f32_dense_cfg(F32Args a, hipStream_t s, size_t max_part = 0) {   // returns the pieces of K
  const long NT = EPI == EPI_SWIGLU ? (a.NB + 3) / 4 : (a.NB + 7) / 8;
  const bool whole = f32_whole<EPI>(a);
  int best = 4;
  double cost = 1e30;
  for (int J = 4; J >= 1; --J)
    for (int S = 1; S <= (EPI == EPI_PART ? 8 : 1); ++S) {
      if (S > 1 && (a.K < S * 256 || (size_t)S * a.rows * a.N > max_part)) break;
      const double c = whole ? f32_dense_cost(EPI == EPI_PART, NT, a, J, S, max_part) : f32_tile_count(NT, a, J, S);
      if (c < cost) { cost = c; best = J; a.splits = S; }
    }
  if (best == 4) launch_f32_dense_tile<EPI, 4>(a, s, max_part);
  else if (best == 3) launch_f32_dense_tile<EPI, 3>(a, s, max_part);
  else if (best == 2) launch_f32_dense_tile<EPI, 2>(a, s, max_part);
  else launch_f32_dense_tile<EPI, 1>(a, s, max_part);
  return a.splits;
}

// Normalised row (x / rms * gain) -> planes, 256 threads; ss: this thread's share of the sum of squares.
__device__ __forceinline__ void norm_row_planes(const float *x, float ss, int d, const float *gain, float eps, u32x4 *xp, int m, size_t kts) {
  __shared__ float red[4];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  const float rn = 1.0f / sqrtf(((red[0] + red[1]) + (red[2] + red[3])) / (float)d + eps);
  for (int k = threadIdx.x * 4; k < d; k += 1024) {
    const f32x4 v = *reinterpret_cast<const f32x4 *>(x + k), gn = *reinterpret_cast<const f32x4 *>(gain + k);
    planes_store4(xp, m, k, v * rn, gn, kts);
  }
}

// Adds the partial sums of a row to its residual (or to the bias) and, where Xp is set, normalises the new row for the next GEMM.
__global__ __launch_bounds__(256) void sum_rmsnorm_f32_kernel(const float *part, int splits, size_t stride, const float *base,
                                                              size_t base_ld, int d, const float *gain, float eps, float *x,
                                                              u32x4 *Xp, size_t kts) {
  const size_t r = blockIdx.x;
  float ss = 0.f;
  for (int k = threadIdx.x * 4; k < d; k += 1024) {
    f32x4 v = *reinterpret_cast<const f32x4 *>(part + r * d + k);   // one rounding at the residual's magnitude
    for (int p = 1; p < splits; ++p) v += *reinterpret_cast<const f32x4 *>(part + p * stride + r * d + k);
    if (base) v += *reinterpret_cast<const f32x4 *>(base + r * base_ld + k);
    *reinterpret_cast<f32x4 *>(x + r * d + k) = v;
    ss += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
  }
  if (Xp) norm_row_planes(x + r * d, ss, d, gain, eps, Xp + (r >> 4) * kPlanePieces, r & 15, kts);
}

// [RMSNorm(x_r) * gain ; embedding of the token behind slot r, where emb is set] -> planes
__global__ __launch_bounds__(256) void norm_cat_f32_kernel(const float *x, int d, const float *gain, float eps, const float *emb,
                                                           const int32_t *next_ids, u32x4 *Xp, size_t kts) {
  const size_t r = blockIdx.x;
  u32x4 *xp = Xp + (r >> 4) * kPlanePieces;
  float ss = 0.f;
  for (int k = threadIdx.x * 4; k < d; k += 1024) {
    const f32x4 v = *reinterpret_cast<const f32x4 *>(x + r * d + k);
    ss += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
  }
  norm_row_planes(x + r * d, ss, d, gain, eps, xp, r & 15, kts);
  if (!emb) return;
  const float *e = emb + (size_t)next_ids[r] * d;
  const f32x4 one = f32x4{1.f, 1.f, 1.f, 1.f};
  for (int k = threadIdx.x * 4; k < d; k += 1024) planes_store4(xp, r & 15, d + k, *reinterpret_cast<const f32x4 *>(e + k), one, kts);
}

void launch_norm_cat_f32(const float *x, int rows, int d, const float *gain, float eps, const void *emb, const int32_t *next_ids,
                         void *Xp, int RB, hipStream_t s) {
  norm_cat_f32_kernel<<<rows, 256, 0, s>>>(x, d, gain, eps, (const float *)emb, next_ids, (u32x4 *)Xp, (size_t)RB * kPlanePieces);
}

size_t planes_bytes(int rows, int K) { return (size_t)(rows + 15) / 16 * ((K + 31) / 32) * kPlanePieces * 16; }

static F32Args f32_dense_args(const GemmLaunch &L, int RB) {
  F32Args a = f32_args(L);
  a.Xp = (const u32x4 *)L.Xp;
  a.Xp_out = (u32x4 *)L.Xp_out;
  a.RB = RB;
  a.splits = 1;
  return a;
}

void launch_gemm_f32_dense(const GemmLaunch &L, int RB, float *part, size_t max_part, hipStream_t s) {
  F32Args a = f32_dense_args(L, RB);
  a.tail_part = (f32x4 *)part;
  if (L.epi == EPI_QKV) launch_f32_dense_cfg<EPI_QKV>(a, s, max_part);
  else launch_f32_dense_cfg<EPI_SWIGLU>(a, s, max_part);
}

void launch_gemm_f32_resid_norm(const GemmLaunch &L, int RB, float *part, size_t max_part, const float *base, size_t base_ld, float *x,
                                const float *gain, void *Xp_out, hipStream_t s) {
  F32Args a = f32_dense_args(L, RB);
  a.Y = part;
  const int S = launch_f32_dense_cfg<EPI_PART>(a, s, max_part);
  sum_rmsnorm_f32_kernel<<<a.rows, 256, 0, s>>>(part, S, (size_t)a.rows * a.N, base, base_ld, a.N, gain, L.eps, x, (u32x4 *)Xp_out,
                                                (size_t)RB * kPlanePieces);
}

// ------------------------------------------------------------------ attention, 1..16 rows
// One workgroup = one KV head x 64 keys fixed by absolute slot, 16 keys per wave; the query rows that share
// the KV head go in tiles of 16.  K operand: lane (key m, g) reads d-octets 4c+g of its key, as cached.  V
// operand: lane (m, g) reads head-dim elements m*VT.. of keys 4g..4g+3, the keys whose probabilities it
// holds: all loads are 128 bits wide and issued up front, no shuffles in between.
constexpr int kF32AttnKeys = 64;

// V rows j >= live of a lane's four keys lie behind the end of the block: rolled back or left by an earlier sequence,
// perhaps not finite.  Their probabilities are 0, but 0 * Inf is not.  (Only the last key tile of a launch has any.)
template <int N>
__device__ __forceinline__ void clear_dead_rows(f32x4 (&v)[4][N], int live) {
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < N; ++i) v[j][i] = j < live ? v[j][i] : f32x4{0.f, 0.f, 0.f, 0.f};
}

template <int HD, int NG, bool GATED>
__global__ __launch_bounds__(256 * NG) void attn_f32_kernel(const float *q, int rows, int pos0, int H, int Hkv, int n_ctx,
                                                       const float *Kc, const float *Vc, float *part, float *out,
                                                       float scale_log2e, const int32_t *gate) {
  constexpr int C = HD / 32, VT = HD / 16;
  __shared__ float reds[NG][4][16][HD + 4];   // (rows of HD floats lie on the same banks, where 16 lanes write 16 of them: 7B 6.8 us, so 6.1)
  __shared__ float wms[NG][4][16], wls[NG][4][16];
  __shared__ ChunkMerge<HD, NG> mrg;
  if constexpr (GATED) AE_GATE(gate);
  // a group of four waves takes a chunk
  const int tid = threadIdx.x & 255, gi = NG > 1 ? threadIdx.x >> 8 : 0, lane = tid & 63, w = tid >> 6, g = lane >> 4, m = lane & 15;
  const int kh = blockIdx.x, chunk = NG > 1 ? gi : blockIdx.y, n_chunks = gridDim.y;
  const int G = H / Hkv, R = rows * G, MT = (R + 15) / 16;
  float (&red)[4][16][HD + 4] = reds[gi];
  float (&wm)[4][16] = wms[gi], (&wl)[4][16] = wls[gi];
  const int kbase = chunk * kF32AttnKeys + w * 16;
  const bool active = kbase < pos0 + rows;   // does this wave own any visible key?

  f32x4 kreg[C][2], vreg[4][VT / 4];
  if (active) {
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const float *kp = Kc + (((size_t)kh * (HD / 8) + 4 * c + g) * n_ctx + kbase + m) * 8;
      kreg[c][0] = *reinterpret_cast<const f32x4 *>(kp);
      kreg[c][1] = *reinterpret_cast<const f32x4 *>(kp + 4);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float *vp = Vc + ((size_t)kh * n_ctx + kbase + 4 * g + j) * HD + m * VT;
#pragma unroll
      for (int i = 0; i < VT / 4; ++i) vreg[j][i] = *reinterpret_cast<const f32x4 *>(vp + 4 * i);
    }
  }
  for (int mt = 0; mt < MT; ++mt) {
    const int r = mt * 16 + m, rc = r < R ? r : R - 1;
    float mx = -INFINITY, lsum = 0.f;
    f32x4 O[VT];
#pragma unroll
    for (int dt = 0; dt < VT; ++dt) O[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (active) {
      const float *qp = q + ((size_t)(rc / G) * H + kh * G + rc % G) * HD + g * 8;
      f32x4 qv[C][2];
#pragma unroll
      for (int c = 0; c < C; ++c) {
        qv[c][0] = *reinterpret_cast<const f32x4 *>(qp + c * 32);
        qv[c][1] = *reinterpret_cast<const f32x4 *>(qp + c * 32 + 4);
      }
      f32x4 S0 = f32x4{0.f, 0.f, 0.f, 0.f}, S1 = S0;
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          S0 = mfma_f32(kreg[c][0][e], qv[c][0][e], S0);
          S1 = mfma_f32(kreg[c][1][e], qv[c][1][e], S1);
        }
      // causal mask: query row r / G sees slots <= pos0 + r / G
      const int limit = r < R ? pos0 + r / G : -1;
      float p[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        p[e] = kbase + 4 * g + e <= limit ? (S0[e] + S1[e]) * scale_log2e : -INFINITY;
        mx = fmaxf(mx, p[e]);
      }
      mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        p[e] = mx > -INFINITY ? __builtin_amdgcn_exp2f(p[e] - mx) : 0.f;
        lsum += p[e];
      }
      lsum += __shfl_xor(lsum, 16, 64);
      lsum += __shfl_xor(lsum, 32, 64);
      if (kbase + 16 > pos0 + rows) clear_dead_rows(vreg, pos0 + rows - kbase - 4 * g);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int dt = 0; dt < VT; ++dt) O[dt] = mfma_f32(vreg[j][dt >> 2][dt & 3], p[j], O[dt]);
    }
    // O[dt][i] is head-dim element (4g + i) * VT + dt of row m
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int t = 0; t < VT / 4; ++t)
        *reinterpret_cast<f32x4 *>(&red[w][m][(4 * g + i) * VT + 4 * t]) =
            f32x4{O[4 * t][i], O[4 * t + 1][i], O[4 * t + 2][i], O[4 * t + 3][i]};
    if (g == 0) { wm[w][m] = mx; wl[w][m] = lsum; }
    __syncthreads();
    {   // combine the four waves in a fixed order
      const int m2 = tid >> 4, seg = tid & 15, r2 = mt * 16 + m2;
      if (r2 < R) {
        const float ms = fmaxf(fmaxf(wm[0][m2], wm[1][m2]), fmaxf(wm[2][m2], wm[3][m2]));
        float wgt[4], l = 0.f;
#pragma unroll
        for (int ww = 0; ww < 4; ++ww) {
          wgt[ww] = wm[ww][m2] > -INFINITY ? __builtin_amdgcn_exp2f(wm[ww][m2] - ms) : 0.f;
          l = fmaf(wgt[ww], wl[ww][m2], l);
        }
        // one workgroup holds the whole context: the result itself, as the merge of a single partial gives it
        const bool whole = NG == 1 && n_chunks == 1;
        float *res = out + ((size_t)(r2 / G) * H + kh * G + r2 % G) * HD;
        float *dst = NG > 1 ? mrg.o[gi][m2] : whole ? res : part + (((size_t)kh * n_chunks + chunk) * R + r2) * (HD + 2);
#pragma unroll
        for (int i = 0; i < HD / 16; ++i) {
          float o = 0.f;
#pragma unroll
          for (int ww = 0; ww < 4; ++ww) o = fmaf(wgt[ww], red[ww][m2][seg * (HD / 16) + i], o);
          dst[seg * (HD / 16) + i] = whole ? o / l : o;
        }
        if (seg == 0 && NG > 1) { mrg.mx[gi][m2] = ms; mrg.l[gi][m2] = l; }
        else if (seg == 0 && !whole) { dst[HD] = ms; dst[HD + 1] = l; }
      }
    }
    __syncthreads();
    if constexpr (NG > 1) {   // (the next tile writes mrg behind its own barrier)
      const int m2 = threadIdx.x / (HD / 4), k0 = threadIdx.x % (HD / 4) * 4, r2 = mt * 16 + m2;
      if (m2 < 16 && r2 < R) {
        const float4 o = mrg.merged(m2, k0);
        *reinterpret_cast<float4 *>(out + ((size_t)(r2 / G) * H + kh * G + r2 % G) * HD + k0) = o;
      }
    }
  }
}

template <int HD, bool GATED>
static void launch_attention_f32_cfg(const float *q, int rows, int pos0, const ae_config &c, const float *Kc, const float *Vc,
                                     float *part, float *out, hipStream_t s, const int32_t *gate) {
  const int n_chunks = (pos0 + rows + kF32AttnKeys - 1) / kF32AttnKeys;
  // Two chunks in one workgroup spare the merge (the smallest model's verification of 5 rows behind 100 slots 105 -> 96 us).  Three and four give nothing
  // (103 -> 101 us, as contexts that they do not concern), nor do heads of 128 elements (431.8 us both): what a
  // compute unit then reads takes as long as the launch.
  const bool two = HD == 64 && n_chunks == 2;
  const auto launch = [&](auto *kernel, int ng) {
    kernel<<<dim3(c.n_kv_heads, ng > 1 ? 1 : n_chunks), 256 * ng, 0, s>>>(q, rows, pos0, c.n_heads, c.n_kv_heads, kv_capacity(c), Kc, Vc, part, out,
                                                                          1.4426950408889634f / sqrtf((float)HD), gate);
  };
  if (two) launch(attn_f32_kernel<HD, HD == 64 ? 2 : 1, GATED>, 2);
  else launch(attn_f32_kernel<HD, 1, GATED>, 1);
  if (n_chunks > 1 && !two) launch_attention_merge(part, rows, n_chunks, c, out, true, s, gate);
}

void launch_attention_f32(const float *q, int rows, int pos0, const ae_config &c, const void *kv_layer, size_t v_off,
                          float *part, float *out, hipStream_t s, const int32_t *gate) {
  const float *Kc = (const float *)kv_layer, *Vc = (const float *)((const char *)kv_layer + v_off);
  if (c.head_dim == 128) {
    if (gate) launch_attention_f32_cfg<128, true>(q, rows, pos0, c, Kc, Vc, part, out, s, gate);
    else launch_attention_f32_cfg<128, false>(q, rows, pos0, c, Kc, Vc, part, out, s, gate);
  } else {
    if (gate) launch_attention_f32_cfg<64, true>(q, rows, pos0, c, Kc, Vc, part, out, s, gate);
    else launch_attention_f32_cfg<64, false>(q, rows, pos0, c, Kc, Vc, part, out, s, gate);
  }
}

int attn_f32_chunk_keys() { return kF32AttnKeys; }

// ------------------------------------------------------------------ causal attention of a prompt chunk
// A wave owns 16 (row, query head of the KV head's group) pairs and walks the visible keys 16 at a time with an
// online softmax (operand mapping of attn_f32_kernel).  Every 256 keys the running output joins a second
// accumulator.  Late (long) tiles are scheduled first; every wave is independent.
template <int HD>
__global__ __launch_bounds__(256) void attn_prefill_f32_kernel(const float *q, int rows, int pos0, int H, int Hkv, int n_ctx,
                                                               const float *Kc, const float *Vc, u32x4 *Xp, size_t kts,
                                                               float scale_log2e) {
  constexpr int C = HD / 32, VT = HD / 16;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, g = lane >> 4, m = lane & 15;
  const int kh = blockIdx.x, G = H / Hkv, R = rows * G;
  const int r0 = (((int)gridDim.y - 1 - (int)blockIdx.y) * 4 + w) * 16;
  if (r0 >= R) return;   // wave-uniform
  const bool rok = r0 + m < R;
  const int r = rok ? r0 + m : R - 1, row = r / G, head = kh * G + r % G, limit = pos0 + row;
  const int last_key = pos0 + min(r0 + 15, R - 1) / G;   // last slot any row of the wave sees
  f32x4 qv[C][2], kreg[C][2], vreg[4][VT / 4];
  const float *qp = q + ((size_t)row * H + head) * HD + g * 8;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    qv[c][0] = *reinterpret_cast<const f32x4 *>(qp + c * 32);
    qv[c][1] = *reinterpret_cast<const f32x4 *>(qp + c * 32 + 4);
  }
  auto load_k = [&](int kb) {
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const float *kp = Kc + (((size_t)kh * (HD / 8) + 4 * c + g) * n_ctx + kb + m) * 8;
      kreg[c][0] = *reinterpret_cast<const f32x4 *>(kp);
      kreg[c][1] = *reinterpret_cast<const f32x4 *>(kp + 4);
    }
  };
  auto load_v = [&](int kb) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float *vp = Vc + ((size_t)kh * n_ctx + kb + 4 * g + j) * HD + m * VT;
#pragma unroll
      for (int i = 0; i < VT / 4; ++i) vreg[j][i] = *reinterpret_cast<const f32x4 *>(vp + 4 * i);
    }
  };
  float mx = -INFINITY, lsum = 0.f, ltot = 0.f;
  f32x4 O[VT], T[VT];
#pragma unroll
  for (int dt = 0; dt < VT; ++dt) O[dt] = T[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  load_k(0);
  load_v(0);
  const int last_kb = last_key & ~15;
  for (int kb = 0; kb <= last_key; kb += 16) {
    const int kb_next = min(kb + 16, last_kb);   // the last step re-requests its own tiles (ignored)
    f32x4 S0 = f32x4{0.f, 0.f, 0.f, 0.f}, S1 = S0;
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        S0 = mfma_f32(kreg[c][0][e], qv[c][0][e], S0);
        S1 = mfma_f32(kreg[c][1][e], qv[c][1][e], S1);
      }
    __builtin_amdgcn_sched_barrier(0);
    load_k(kb_next);
    __builtin_amdgcn_sched_barrier(0);
    float p[4], bmax = -INFINITY;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      p[e] = kb + 4 * g + e <= limit ? (S0[e] + S1[e]) * scale_log2e : -INFINITY;
      bmax = fmaxf(bmax, p[e]);
    }
    bmax = fmaxf(bmax, __shfl_xor(bmax, 16, 64));
    bmax = fmaxf(bmax, __shfl_xor(bmax, 32, 64));
    const float mnew = fmaxf(mx, bmax);   // finite from the first block on: slot 0 is visible to every row
    const float alpha = __builtin_amdgcn_exp2f(mx - mnew);
    float bsum = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      p[e] = __builtin_amdgcn_exp2f(p[e] - mnew);
      bsum += p[e];
    }
    lsum = lsum * alpha + bsum;   // this lane's share: the four lane groups are added at the end
    ltot *= alpha;
    mx = mnew;
#pragma unroll
    for (int dt = 0; dt < VT; ++dt) {
      O[dt] *= alpha;
      T[dt] *= alpha;
    }
    if (kb + 16 > pos0 + rows) clear_dead_rows(vreg, pos0 + rows - kb - 4 * g);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int dt = 0; dt < VT; ++dt) O[dt] = mfma_f32(vreg[j][dt >> 2][dt & 3], p[j], O[dt]);
    __builtin_amdgcn_sched_barrier(0);
    load_v(kb_next);
    __builtin_amdgcn_sched_barrier(0);
    if ((kb & 255) == 240) {
#pragma unroll
      for (int dt = 0; dt < VT; ++dt) {
        T[dt] += O[dt];
        O[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      ltot += lsum;
      lsum = 0.f;
    }
  }
  ltot += lsum;
  ltot += __shfl_xor(ltot, 16, 64);
  ltot += __shfl_xor(ltot, 32, 64);
  if (rok) {
    u32x4 *xp = Xp + (size_t)(row >> 4) * kPlanePieces;
#pragma unroll 1   // (unrolled, the handling of large numbers makes the kernel long)
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int t = 0; t < VT / 4; ++t) {
        f32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (T[4 * t + e][i] + O[4 * t + e][i]) / ltot;
        planes_store4(xp, row & 15, head * HD + (4 * g + i) * VT + 4 * t, o, f32x4{1.f, 1.f, 1.f, 1.f}, kts);
      }
  }
}

void launch_attention_prefill_f32(const float *q, int rows, int pos0, const ae_config &c, const void *kv_layer, size_t v_off,
                                  void *Xp, int RB, hipStream_t s) {
  const int G = c.n_heads / c.n_kv_heads, R = rows * G, HD = c.head_dim;
  const dim3 grid(c.n_kv_heads, (R + 63) / 64);
  const size_t kts = (size_t)RB * kPlanePieces;
  const float scale = 1.4426950408889634f / sqrtf((float)HD);
  const float *Kc = (const float *)kv_layer, *Vc = (const float *)((const char *)kv_layer + v_off);
  if (HD == 128)
    attn_prefill_f32_kernel<128><<<grid, 256, 0, s>>>(q, rows, pos0, c.n_heads, c.n_kv_heads, kv_capacity(c), Kc, Vc, (u32x4 *)Xp, kts, scale);
  else
    attn_prefill_f32_kernel<64><<<grid, 256, 0, s>>>(q, rows, pos0, c.n_heads, c.n_kv_heads, kv_capacity(c), Kc, Vc, (u32x4 *)Xp, kts, scale);
}

// ------------------------------------------------------------------ row producers
// Embedding rows -> residual stream, x * gain and the row's sum of x^2 (gain == nullptr: the rows alone)
__global__ __launch_bounds__(256) void embed_f32_kernel(const float *emb, const BlockIds ids, int d, const float *gain, float *x,
                                                        float *Xo, float *ssq) {
  __shared__ float red[4];
  const int r = blockIdx.x;
  const float *src = emb + (size_t)block_id(ids, r) * d;
  float ss = 0.f;
  for (int k = threadIdx.x * 4; k < d; k += 1024) {
    const float4 v = *reinterpret_cast<const float4 *>(src + k);
    *reinterpret_cast<float4 *>(x + (size_t)r * d + k) = v;
    if (gain) {
      ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
      const float4 gn = *reinterpret_cast<const float4 *>(gain + k);
      *reinterpret_cast<float4 *>(Xo + (size_t)r * d + k) = make_float4(v.x * gn.x, v.y * gn.y, v.z * gn.z, v.w * gn.w);
    }
  }
  if (!gain) return;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  if (threadIdx.x == 0) ssq[r] = (red[0] + red[1]) + (red[2] + red[3]);
}

void launch_embed_f32(const void *emb, const BlockIds &ids, int rows, int d, const float *gain, float *x, void *Xo, float *ssq,
                      hipStream_t s) {
  embed_f32_kernel<<<rows, 256, 0, s>>>((const float *)emb, ids, d, gain, x, (float *)Xo, ssq);
}

// cat[r] = [feature row r ; embedding of the token that FOLLOWS slot r]  (Sec. 2.2)
__global__ __launch_bounds__(256) void draft_cat_f32_kernel(const float *feat, int feat_ld, const float *emb,
                                                            const int32_t *next_ids, int d, float *cat, const DraftInputs in) {
  const int r = blockIdx.x;
  if (r == 0 && in.st) store_draft_inputs(in);
  const float *e = emb + (size_t)next_ids[r] * d, *f = feat + (size_t)r * feat_ld;
  float *o = cat + (size_t)r * 2 * d;
  for (int k = threadIdx.x * 4; k < d; k += 1024) {
    *reinterpret_cast<float4 *>(o + k) = *reinterpret_cast<const float4 *>(f + k);
    *reinterpret_cast<float4 *>(o + d + k) = *reinterpret_cast<const float4 *>(e + k);
  }
}

void launch_draft_cat_f32(const float *feat, int feat_ld, const void *emb, const int32_t *next_ids, int rows, int d, void *cat,
                          hipStream_t s, const DraftInputs &in) {
  draft_cat_f32_kernel<<<rows, 256, 0, s>>>(feat, feat_ld, (const float *)emb, next_ids, d, (float *)cat, in);
}

}  // namespace ae
