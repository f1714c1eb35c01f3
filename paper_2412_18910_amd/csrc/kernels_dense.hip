// Dense prompt pass (first iteration of Algorithm 1 of arxiv 2412.18910 on a long prompt):
// the only place of the method where the matrix cores, not HBM, are the limit.
//
// The prompt is processed in chunks of up to a few thousand rows.  Activations of a chunk
// live in the packed bf16 hi/lo form of the decode step, extended to many row-blocks
// (Xp[kt][rb][h][64], see packed.h); weights are the same k-major MFMA tiles the decode
// GEMMs stream.  Kernels:
//  * gemm_dense_kernel: a workgroup of 4 or 8 waves makes a tile of 128 to 512 weight rows x 32 to 128
//    activation rows (dense_plan).  Each wave owns 2 to 4 weight row-blocks (A operands: buffer loads straight
//    from the tiled matrix into registers, one coalesced 1 KB burst per tile, three k-tiles ahead) and
//    multiplies them with all activation row-blocks, which go straight into an LDS ring of four k-tiles
//    (64 KB for 128 rows).  At 4 x 8 row-blocks, 64 MFMAs per wave and k-tile against 16 LDS reads, which are
//    issued one step ahead of the MFMAs that use them; two waves feed every matrix pipe (<= 256 registers);
//    tiles are handed out XCD-aware; epilogues are those of the decode GEMM.
//  * attn_prefill_kernel: causal flash attention straight off the tiled KV cache; a wave owns
//    16 or 32 (row, head) pairs of one KV head and walks the visible keys 32 at a time with an
//    online softmax in the log2 domain; no partials, no merge, packed output.
//  * embedding, 1/rms finalisation and the draft head's [feature ; embedding] input.
#include "ae_internal.h"
#include "dense_tile.h"
#include "gemm_epilogue.h"
#include "packed.h"

namespace ae {

constexpr int EPI_PART = 4;   // raw float32 sums over a piece of K -> a.part[piece][row][N]

// DM = activation row-blocks per workgroup, DN = weight row-blocks per wave, NW = waves; EPI_PART: K is split over workgroups
// (gridDim.y pieces).  The waves lie along the weights alone: with two groups of waves along the rows (half the LDS
// reads, each weight tile loaded twice) 100 rows of 7B gate/up took 52 us instead of 46, the vector cache being what is short.
template <int EPI, bool NORM, int DM, int DN, int NW>
__global__ __launch_bounds__(NW * 64, 2) void gemm_dense_kernel(const GemmArgs a) {
  // ring of four k-tiles of B, [DM][2][64] pieces each: arrays of their own, so that the compiler can tell a read of
  // one from a load into another
  __shared__ u32x4 b0[DM * 128], b1[DM * 128], b2[DM * 128], b3[DM * 128];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, m = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: keeps operand bases in scalar registers
  // Workgroup -> tile.  Workgroups are handed to the 8 XCDs round-robin (id % 8) and each XCD
  // has its own L2, so XCD x takes a contiguous share of the tile list, and the list runs
  // through panels of 8 weight tiles with the activation tile advancing every 8 entries: the
  // ~64 workgroups resident on an XCD then cover about 8 x 8 tiles and share their operands in
  // that L2 (7B gate/up GEMM over 2048 rows: 1.4 GB fetched from HBM instead of 3.3 GB with
  // the plain row-major order).
  const int NT = (a.NBtot + NW * DN - 1) / (NW * DN), MT = (a.rows + DM * 16 - 1) / (DM * 16);
  const int per = (NT * MT + 7) >> 3;
  const int v = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
  if (v >= NT * MT) return;
  constexpr int PN = 8;
  const int full = (NT / PN) * PN * MT;
  int tn, tm;
  if (v < full) {
    const int r = v % (PN * MT);
    tn = (v / (PN * MT)) * PN + r % PN;
    tm = r / PN;
  } else {
    const int r = v - full, pn = NT % PN;
    tn = (NT / PN) * PN + r % pn;
    tm = r / pn;
  }
  const int rb0 = tm * DM;
  // a workgroup hanging over the end of the matrix slides back (recomputes, stores nothing new)
  const int nbw = min(tn * (NW * DN), a.NBtot - NW * DN) + w * DN;
  const size_t kts = (size_t)a.RB * 128;
  // Operands come through buffer loads: resource descriptor and per-k-tile byte offset in
  // scalar registers, one fixed per-lane offset register each.  All reads are in range: the descriptors' sizes
  // do not cover a position that is in the scalar offset.
  // The DM row-blocks of one k-tile are 2*DM tiles of 64 contiguous pieces; a wave loads its own (dense_slot) straight
  // into LDS in lane order, so its accesses are conflict-free.
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void *)a.W, 0, a.w_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void *)a.Xp, 0, a.xp_bytes, 0x00020000);
  const unsigned wl = lane * 16;                                         // per-lane byte offset
  const unsigned kstride_b = a.NBtot * 1024u, kts_b = a.RB * 2048u;      // bytes per k-tile
  unsigned wq = nbw * 1024u, xq = rb0 * 2048u;           // first k-tile (uniform)
  int NK = a.KT;   // k-tiles, a multiple of 4
  if (EPI == EPI_PART) {   // a piece of K in units of 4 k-tiles
    const int u0 = a.KT / 4 * (int)blockIdx.y / (int)gridDim.y, u1 = a.KT / 4 * ((int)blockIdx.y + 1) / (int)gridDim.y;
    wq += u0 * 4 * kstride_b;
    xq += u0 * 4 * kts_b;
    NK = (u1 - u0) * 4;
  }

  f32x4 acc[DN][DM];
#pragma unroll
  for (int i = 0; i < DN; ++i)
#pragma unroll
    for (int j = 0; j < DM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Three k-tiles are in flight while one is multiplied: A tiles on their way into register sets, B tiles into LDS
  // without passing registers.  (Through registers only one stage fitted beside the 128 accumulators; waits on
  // loads one stage old and the LDS writes kept the matrix pipes at 60 % of a 7B gate/up GEMM over 2048 rows.)
  // 7B widths, 2048 rows: gate/up 597 -> 548 us, QKV 346 -> 319, o/down 225 -> 213 on average.
  constexpr int XI = (DM * 2 + NW - 1) / NW, VM = XI + DN;   // B tiles per wave, loads per wave and k-tile
  u32x4 w0[DN], w1[DN], w2[DN], w3[DN];
  auto put = [&](u32x4 *slot, u32x4 (&wr)[DN], int kt) {   // k-tiles behind the last repeat it (ignored)
    const unsigned k = min(kt, NK - 1);
#pragma unroll
    for (int i = 0; i < XI; ++i) {
      const int t = dense_slot(w, i, NW, DM);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (__attribute__((address_space(3))) void *)(slot + t * 64), 16, wl,
                                               xq + k * kts_b + dense_source(t, rb0, a.RB) * 1024, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < DN; ++i) wr[i] = __builtin_amdgcn_raw_buffer_load_b128(rw, wl + i * 1024, wq + k * kstride_b, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  // Every wave waits for its own loads of the k-tile that comes next (all but the 2 * VM of the two k-tiles behind
  // it), then for the other waves: the k-tile is in LDS, and the slot multiplied last is free.
  auto gate = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xf70 | ((2 * VM) & 15) | ((2 * VM) >> 4 << 14));   // vmcnt(2 * VM)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  // MFMAs of one k-tile.  The B tiles of step t+1 are read from LDS while the 2*DN MFMAs of
  // step t run; the sched_group_barrier sequence pins that interleaving.
  auto multiply = [&](const u32x4 (&wr)[DN], const u32x4 *slot) {
    const u32x4 *bcur = slot + lane;
    u32x4 f[2][2];
    f[0][0] = bcur[0];
    f[0][1] = bcur[64];
#pragma unroll
    for (int t = 0; t < DM; ++t) {
      if (t + 1 < DM) {
        f[(t + 1) & 1][0] = bcur[(t + 1) * 128];
        f[(t + 1) & 1][1] = bcur[(t + 1) * 128 + 64];
      }
#pragma unroll
      for (int i = 0; i < DN; ++i) acc[i][t] = mfma_bf16(wr[i], f[t & 1][0], acc[i][t]);
#pragma unroll
      for (int i = 0; i < DN; ++i) acc[i][t] = mfma_bf16(wr[i], f[t & 1][1], acc[i][t]);
    }
    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);        // DS reads of step 0
#pragma unroll
    for (int t = 0; t < DM; ++t) {
      if (t + 1 < DM) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);   // DS reads of step t+1
      __builtin_amdgcn_sched_group_barrier(0x008, 2 * DN, 0);             // MFMAs of step t
    }
  };
  put(b0, w0, 0);
  put(b1, w1, 1);
  put(b2, w2, 2);
  for (int kt = 0; kt < NK; kt += 4) {
    gate();
    put(b3, w3, kt + 3);
    multiply(w0, b0);
    gate();
    put(b0, w0, kt + 4);
    multiply(w1, b1);
    gate();
    put(b1, w1, kt + 5);
    multiply(w2, b2);
    gate();
    put(b2, w2, kt + 6);
    multiply(w3, b3);
  }
  __builtin_amdgcn_s_waitcnt(0xf70);   // vmcnt(0): no load into LDS outlives the loop

  constexpr int STEP = EPI == EPI_SWIGLU ? 2 : 1;
#pragma unroll
  for (int i = 0; i < DN; i += STEP) {
    const int nb = nbw + i;
    if (nb < tn * (NW * DN)) continue;   // slid-back duplicate of a neighbour's row-block
#pragma unroll
    for (int j = 0; j < DM; ++j) {
      const int rb = rb0 + j, row = rb * 16 + m;
      if (rb * 16 >= a.rows) break;   // wave-uniform: behind the rows, and where DM does not divide them behind the buffers
      const bool row_ok = row < a.rows;
      if (EPI == EPI_PART) {
        if (row_ok)
          *reinterpret_cast<f32x4 *>(a.part + (((size_t)blockIdx.y * a.rows + row) * a.NBtot + nb) * 16 + 4 * g) = acc[i][j];
        continue;
      }
      const float rinv = NORM && row_ok ? a.rinv[row] : 1.f;
      epi_tile<EPI, true>(a, acc[i][j], acc[i + STEP - 1][j], nb, g, m, rb, row_ok, rinv, kts);
    }
  }
}

template <int EPI, bool NORM, int DM, int DN, int NW>
static void launch_dense_tile(const GemmArgs &a, int splits, hipStream_t s) {
  const int tiles = ((a.NBtot + NW * DN - 1) / (NW * DN)) * ((a.rows + DM * 16 - 1) / (DM * 16));
  gemm_dense_kernel<EPI, NORM, DM, DN, NW><<<dim3((tiles + 7) / 8 * 8, splits), NW * 64, 0, s>>>(a);
}

// How a GEMM is laid out on the chip: waves (4 or 8) and weight row-blocks of each (dn), activation row-blocks of a workgroup
// (dm, exact: a prompt of 100 rows multiplies 7, not 8), pieces of K (0: whole K, and the epilogue in the same kernel).
struct DensePlan {
  int nw = 8, dn = 2, dm = 8, splits = 0;
};

// Microseconds that a plan takes, fitted to 9600 launches (7B, 13B and 8B-GQA widths, 20 to 4096 rows).  Measured again (4876 plans, 216
// GEMMs): the plan it picks is 2.3, 1.1 and 1.1 % off the best of all on average, its microseconds are 0.78 to 1.21 of the
// measured ones.  Workgroups go round-robin to the 8 XCDs of 32 compute units.  A
// k-tile of a workgroup costs what is largest of its products (5 ns for 16 x 16 x 32, hi and lo), what it takes through the
// vector cache (16 ns a KB: 64 GB/s a compute unit, by lines in flight) and the weights' share of HBM.  Pieces are
// written at 3.8 TB/s when all workgroups end at once, and a pass adds them; whole K pays for its epilogue, and for
// o and down for the launch that sums x^2.  One workgroup of four waves alone on a compute unit is 12 % slower at the
// products; of those that run for several rounds 4 x 4 tiles (two workgroups a unit) are ahead for gate/up (7B, 2048 rows: 528 us, 8 x 2 537, 8 x 4
// 526; 4096 rows 988, 1011), 8 x 2 for the rest (QKV, 2048 rows: 297, 4 x 4 301; o and down together 395, 435).
static double dense_cost(const GemmArgs &a, int epi, const DensePlan &p) {
  const int n = p.nw * p.dn, S = p.splits > 0 ? p.splits : 1;
  const long tiles = (long)((a.NBtot + n - 1) / n) * ((a.rows + p.dm * 16 - 1) / (p.dm * 16));
  const long rounds = ((tiles + 7) / 8 * S + 31) / 32;
  double e = 1.0 + 0.02 * (8 - p.dm);
  if (p.nw == 4 && rounds == 1) e *= 1.116;
  else if (p.nw == 8 && rounds > 1) e *= p.dn == 4 ? 1.04 : epi == EPI_SWIGLU ? 1.02 : 1.0;
  const double active = (double)tiles * S / rounds, products = n * p.dm * 4.98 * e, cache = (n + 2 * p.dm) * 15.84,
               memory = n * 0.128 * (active < 256 ? active : 256);   // 8 TB/s: ramps are in the constant
  double k = products > cache ? products : cache;
  if (memory > k) k = memory;
  const double out = (double)a.rows * a.NBtot * 64;   // bytes of one float32 result
  const double t = 6.9 + rounds * (a.KT / (double)S) * k * 1e-3;
  if (p.splits > 0) return t + S * out / 3.8e6 + 5.4 + (S + 1) * out / 6.6e6;
  return t + out * (epi == EPI_QKV ? 1 : epi == EPI_SWIGLU ? 0.5 : 3) / 10.9e6 + (epi == EPI_QKV || epi == EPI_SWIGLU ? 0 : 5.5);
}

// Plans by the number of tiles, the older rule, for what dense_cost was not fitted to: K below 3072, a last chunk of one row-block, and whole K
// of the draft head's input projection (once a prompt: 200 us of 2048 rows of 7B either way).  At K below 3072 it is the slower one: 2048 x 5632
// 18 % off the best plan on average, dense_cost 1.7; 1024 x 2816 28 %, 2.5 (20 to 4096 rows): the line could lie lower.  Less than 384 tiles of 256 weight rows x 64 rows
// would leave compute units idle (256, two workgroups each): pieces of K.  Else 128-row tiles, or 64-row ones (0.55 of
// their time) where these fill rounds of 512 workgroups better; one round of them in workgroups of eight waves, which
// take the activations through the vector cache once instead of twice.
static DensePlan plan_by_tiles(const GemmArgs &a, size_t part_floats) {
  DensePlan best;
  const long nt = (a.NBtot + 15) / 16, t8 = nt * ((a.rows + 127) / 128), t4 = nt * ((a.rows + 63) / 64);
  if (t4 < 384) {
    const long mt = a.rows > 64 ? (a.rows + 127) / 128 : 1;
    double cost = 1e30;
    for (int dn = 2; dn <= 3; ++dn) {
      if (a.NBtot < 8 * dn) break;
      const long tiles = (a.NBtot + 8 * dn - 1) / (8 * dn) * mt;
      for (int S = 1; S <= 16 && S <= a.KT / 8; ++S) {   // a piece: two passes of the k-loop at least
        if ((size_t)S * a.rows * a.NBtot * 16 > part_floats) break;
        const double c = (double)((tiles * S + 255) / 256) * dn / S + 0.005 * S;   // rounds x work of a piece, its pass
        if (c < cost) { cost = c; best = DensePlan{8, dn, a.rows > 64 ? 8 : 4, S}; }
      }
    }
    if (best.splits) return best;
  }
  const double c8 = (double)((t8 + 511) / 512), c4 = 0.55 * (double)((t4 + 511) / 512);
  const long t48 = (nt + 1) / 2 * ((a.rows + 63) / 64);
  if (c4 < c8 && t4 <= 512 && t48 > 192 && t48 <= 256) return DensePlan{8, 4, 4, 0};
  return DensePlan{4, 4, c4 < c8 ? 4 : 8, 0};
}

// Short prompts: few tiles, all of the weights to read.  K is cut so that all compute units read, but in as few pieces as that
// takes: writing and adding them was a third of a 7B layer of 100 rows (gate/up 4 pieces of 384 weight rows 46 + 9 us, now 2 of 192
// 46 + 6; QKV 8 of 384 31 + 10, now 4 of 192 29 + 7; o and down 16 of 256 24 + 8, now 8 of 128 20 + 6).  Long prompts: whole K, the
// rows in tiles that fill their last round.
static DensePlan dense_plan(const GemmArgs &a, int epi, size_t part_floats) {
  const DensePlan by_tiles = plan_by_tiles(a, part_floats);
  if (a.KT < 96 || a.rows <= 16 || (epi == EPI_STORE && by_tiles.splits == 0)) return by_tiles;
  static constexpr int kSplit[4][2] = {{4, 2}, {4, 3}, {8, 2}, {8, 3}}, kWhole[3][2] = {{8, 2}, {8, 4}, {4, 4}};   // waves, dn
  DensePlan best = by_tiles;
  double cost = 1e30;
  auto consider = [&](const DensePlan &p) {
    if (a.NBtot < p.nw * p.dn) return;
    const double c = dense_cost(a, epi, p);
    if (c < cost) { cost = c; best = p; }
  };
  for (int i = 0; i < (epi == EPI_STORE ? 0 : epi == EPI_SWIGLU ? 3 : 1); ++i)   // gate/up alone gains by the other two
    for (int dm = 4; dm <= 8; ++dm) consider(DensePlan{kWhole[i][0], kWhole[i][1], dm, 0});
  const int rbs = (a.rows + 15) / 16, mt = (rbs + 7) / 8;
  for (auto &w : kSplit)
    for (int S = 1; S <= 16 && (size_t)S * a.rows * a.NBtot * 16 <= part_floats; ++S)
      consider(DensePlan{w[0], w[1], (rbs + mt - 1) / mt, S});
  return best;
}

template <int DM>
static void launch_dense_part(const GemmArgs &a, const DensePlan &p, hipStream_t s) {
  if (p.nw == 4 && p.dn == 2) launch_dense_tile<EPI_PART, false, DM, 2, 4>(a, p.splits, s);
  else if (p.nw == 4) launch_dense_tile<EPI_PART, false, DM, 3, 4>(a, p.splits, s);
  else if (p.dn == 2) launch_dense_tile<EPI_PART, false, DM, 2, 8>(a, p.splits, s);
  else launch_dense_tile<EPI_PART, false, DM, 3, 8>(a, p.splits, s);
}

// Every plan ends in a launch, one without an instance of its own in the narrowest tile: 16 weight row-blocks, which all matrices have.
template <int EPI, bool NORM, int DM>
static void launch_dense_whole(const GemmArgs &a, const DensePlan &p, hipStream_t s) {
  if constexpr (EPI == EPI_SWIGLU || DM == 4 || DM == 8)   // else plan_by_tiles alone
    if (p.nw == 4) return launch_dense_tile<EPI, NORM, DM, 4, 4>(a, 1, s);
  if constexpr (EPI == EPI_SWIGLU || DM == 4)
    if (p.nw == 8 && p.dn == 4) return launch_dense_tile<EPI, NORM, DM, 4, 8>(a, 1, s);
  launch_dense_tile<EPI, NORM, DM, 2, 8>(a, 1, s);
}

// Adds the pieces of one 16x16 tile (EPI_SWIGLU: of a gate and an up tile) per wave and runs the GEMM's epilogue on it.
template <int EPI>
__global__ __launch_bounds__(256) void dense_finish_kernel(const GemmArgs a, int splits) {
  constexpr int STEP = EPI == EPI_SWIGLU ? 2 : 1;
  const int lane = threadIdx.x & 63, g = lane >> 4, m = lane & 15;
  const int NU = a.NBtot / STEP, v = blockIdx.x * 4 + (threadIdx.x >> 6), nb = v % NU * STEP, rb = v / NU;
  const int row = rb * 16 + m;
  const bool row_ok = row < a.rows;
  if (rb * 16 >= a.rows) return;   // wave-uniform
  const float *p = a.part + ((size_t)(row_ok ? row : a.rows - 1) * a.NBtot + nb) * 16 + 4 * g;
  const size_t stride = (size_t)a.rows * a.NBtot * 16;
  f32x4 t = *reinterpret_cast<const f32x4 *>(p), u = t;
  if (STEP == 2) u = *reinterpret_cast<const f32x4 *>(p + 16);
#pragma unroll 4
  for (int i = 1; i < splits; ++i) {
    t += *reinterpret_cast<const f32x4 *>(p + i * stride);
    if (STEP == 2) u += *reinterpret_cast<const f32x4 *>(p + i * stride + 16);
  }
  epi_tile<EPI, true>(a, t, u, nb, g, m, rb, row_ok, a.rinv[row], (size_t)a.RB * 128);
}

// Row of a workgroup of the kernels that pack a row each.  Neighbouring rows share lines of a packed tile, so they go to
// one XCD (workgroups are handed out round-robin to the eight), whose L2 puts the lines together: the 16 rows of a row-block,
// or four, which share 64 bytes, where the row-blocks are too few for all of the chip.  Tiles in lane order, 7B widths,
// microseconds in row order -> so (row-major tiles, which these kernels alone would want): sum of K pieces, 100 rows 8.9 -> 7.9
// (7.6), 333 13.3 -> 11.1 (10.0), 1100 27.0 -> 19.2 (18.0); draft input, 333 rows 17.3 -> 12.8 (10.0), 1100 44.3 -> 28.2 (25.5),
// 2048 78.7 -> 51.4 (45.5); embedding, 1100 rows 23.1 -> 17.2 (18.2), 2048 40.0 -> 24.8 (29.0).  What lane order costs the
// first two the GEMMs gain several times over (a layer of 2048 rows 24 us).
constexpr int packed_row_groups(int rows) { return rows > 512 ? (rows + 127) / 128 * 128 : (rows + 31) / 32 * 32; }
__device__ __forceinline__ int packed_row() {
  const int b = blockIdx.x, sh = gridDim.x > 512 ? 4 : 2;   // rows beside each other: 16 or 4
  return (((b >> (3 + sh)) * 8 + (b & 7)) << sh) + ((b >> 3) & ((1 << sh) - 1));
}

// Adds the pieces of a row to its residual (x, updated in place) or to the bias, leaves row * gain packed for the next
// GEMM and the row's 1/rms.
__global__ __launch_bounds__(1024) void dense_sum_rows_kernel(const GemmArgs a, int splits, float *rinv, float eps) {
  __shared__ float red[16];
  const int r = packed_row(), d = a.NBtot * 16;
  if (r >= a.rows) return;
  const float *p = a.part + (size_t)r * d;
  const size_t stride = (size_t)a.rows * d;
  float *x = a.seg[0].Y ? a.seg[0].Y + (size_t)r * a.seg[0].ldy : nullptr;
  float ss = 0.f;
  for (int k = threadIdx.x * 4; k < d; k += 4096) {
    f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
    if (x) v = *reinterpret_cast<const f32x4 *>(x + k);
    else if (a.bias) v = *reinterpret_cast<const f32x4 *>(a.bias + k);
    for (int i = 0; i < splits; i += 4) {   // by fours: loads in flight together, one rounding at the residual's magnitude
      f32x4 q = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 t = *reinterpret_cast<const f32x4 *>(p + min(i + j, splits - 1) * stride + k);
        q += i + j < splits ? t : f32x4{0.f, 0.f, 0.f, 0.f};
      }
      v += q;
    }
    if (x) *reinterpret_cast<f32x4 *>(x + k) = v;
    ss += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
    const f32x4 gn = *reinterpret_cast<const f32x4 *>(a.gain_out + k);
    packed_store4<true>(a.Xp_out + (size_t)(r >> 4) * 128, r & 15, k, v[0] * gn[0], v[1] * gn[1], v[2] * gn[2], v[3] * gn[3],
                  (size_t)a.RB * 128);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) t += red[i];
    rinv[r] = 1.0f / sqrtf(t / (float)d + eps);
  }
}

template <int EPI, bool NORM>
static void launch_dense_cfg(const GemmArgs &a, const DensePlan &p, hipStream_t s) {
  if constexpr (EPI == EPI_STORE) {   // plan_by_tiles
    if (p.nw == 8) launch_dense_tile<EPI, NORM, 4, 4, 8>(a, 1, s);
    else if (p.dm == 4) launch_dense_tile<EPI, NORM, 4, 4, 4>(a, 1, s);
    else launch_dense_tile<EPI, NORM, 8, 4, 4>(a, 1, s);
  } else {
    switch (p.dm) {
      case 4: launch_dense_whole<EPI, NORM, 4>(a, p, s); break;
      case 5: launch_dense_whole<EPI, NORM, 5>(a, p, s); break;
      case 6: launch_dense_whole<EPI, NORM, 6>(a, p, s); break;
      case 7: launch_dense_whole<EPI, NORM, 7>(a, p, s); break;
      default: launch_dense_whole<EPI, NORM, 8>(a, p, s); break;
    }
  }
}

bool launch_gemm_dense(const GemmLaunch &L, int RB, const float *rinv, hipStream_t s, float *part, size_t part_floats,
                       float *rinv_out) {
  GemmArgs a{};
  a.W = (const u32x4 *)L.W->tiled;
  a.NBtot = L.W->N / 16;
  a.KT = L.W->K / 32;
  a.Xp = (const u32x4 *)L.Xp;
  a.rows = L.rows;
  a.RB = RB;
  a.w_bytes = (int)((size_t)L.W->N * L.W->K * 2);
  a.xp_bytes = (int)((size_t)L.W->K * RB * 64);
  a.rinv = rinv;
  a.bias = L.bias;
  a.Xp_out = (u32x4 *)L.Xp_out; a.gain_out = L.gain_out; a.ssq_out = L.ssq_out;
  int end = 0;
  for (int i = 0; i < 3; ++i) {
    if (i < L.nseg) end += L.seg_N[i] / 16;
    a.seg[i] = GemmSeg{i < L.nseg ? L.Y[i] : nullptr, i < L.nseg ? L.ldy[i] : 0, i < L.nseg ? end : 0x7fffffff};
  }
  a.rope_tab = L.rope_tab; a.Kc = (uint16_t *)L.Kc; a.Vc = (uint16_t *)L.Vc;
  a.pos0 = L.pos0; a.n_ctx = L.n_ctx; a.hd = L.hd;
  a.part = part;
  const DensePlan p = dense_plan(a, L.epi, part_floats);
  const int S = p.splits;
  if (S > 0) {
    switch (p.dm) {
      case 2: launch_dense_part<2>(a, p, s); break;
      case 3: launch_dense_part<3>(a, p, s); break;
      case 4: launch_dense_part<4>(a, p, s); break;
      case 5: launch_dense_part<5>(a, p, s); break;
      case 6: launch_dense_part<6>(a, p, s); break;
      case 7: launch_dense_part<7>(a, p, s); break;
      default: launch_dense_part<8>(a, p, s); break;
    }
    const int rb = (a.rows + 15) / 16;
    if (L.epi == EPI_QKV) dense_finish_kernel<EPI_QKV><<<(a.NBtot * rb + 3) / 4, 256, 0, s>>>(a, S);
    else if (L.epi == EPI_SWIGLU) dense_finish_kernel<EPI_SWIGLU><<<(a.NBtot / 2 * rb + 3) / 4, 256, 0, s>>>(a, S);
    else dense_sum_rows_kernel<<<packed_row_groups(a.rows), 1024, 0, s>>>(a, S, rinv_out, L.eps);
    return true;
  }
  if (L.epi == EPI_QKV) launch_dense_cfg<EPI_QKV, true>(a, p, s);
  else if (L.epi == EPI_SWIGLU) launch_dense_cfg<EPI_SWIGLU, true>(a, p, s);
  else if (L.epi == EPI_RESID) launch_dense_cfg<EPI_RESID, false>(a, p, s);
  else launch_dense_cfg<EPI_STORE, false>(a, p, s);
  return false;
}

// ------------------------------------------------------------------ 1/rms of every row
// ssq: [RB][P][16] partial sums of x^2 -> rinv[rb*16 + m]; one workgroup per row-block,
// 16 threads per row, fixed summation order.
__global__ __launch_bounds__(256) void rinv_finalize_kernel(const float *ssq, int P, int K, float eps, float *rinv) {
  __shared__ float sh[256];
  const int rb = blockIdx.x, m = threadIdx.x & 15, pg = threadIdx.x >> 4;
  float t = 0.f;
#pragma unroll 16   // loads in flight, not one after the other
  for (int p = pg; p < P; p += 16) t += ssq[((size_t)rb * P + p) * 16 + m];
  sh[threadIdx.x] = t;
  __syncthreads();
  if (threadIdx.x < 16) {
    float tot = 0.f;
    for (int i = 0; i < 16; ++i) tot += sh[i * 16 + threadIdx.x];
    rinv[rb * 16 + threadIdx.x] = 1.0f / sqrtf(tot / (float)K + eps);
  }
}

void launch_rinv_finalize(const float *ssq, int RBused, int P, int K, float eps, float *rinv, hipStream_t s) {
  rinv_finalize_kernel<<<RBused, 256, 0, s>>>(ssq, P, K, eps, rinv);
}

// ------------------------------------------------------------------ packed-form producers
__device__ __forceinline__ void bf16_to_float8(const uint16_t *p, float (&v)[8]) {
  const u32x4 raw = *reinterpret_cast<const u32x4 *>(p);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = __uint_as_float(raw[i] << 16);
    v[2 * i + 1] = __uint_as_float(raw[i] & 0xffff0000u);
  }
}

// Embedding rows -> float residual stream, packed(x * gain) and the row's sum of x^2 ([rb][1][16]).
__global__ __launch_bounds__(256) void embed_dense_kernel(const uint16_t *emb, const int32_t *ids, int rows, int d, const float *gain,
                                                          float *x, u32x4 *Xp, size_t kts, float *ssq) {
  __shared__ float red[4];
  const int r = packed_row(), rb = r >> 4, m = r & 15;
  if (r >= rows) return;
  const uint16_t *src = emb + (size_t)ids[r] * d;
  u32x4 *xp = Xp + (size_t)rb * 128;
  float ss = 0.f;
  for (int k0 = threadIdx.x * 4; k0 < d; k0 += 1024) {
    const uint2 raw = *reinterpret_cast<const uint2 *>(src + k0);
    const float v0 = __uint_as_float(raw.x << 16), v1 = __uint_as_float(raw.x & 0xffff0000u);
    const float v2 = __uint_as_float(raw.y << 16), v3 = __uint_as_float(raw.y & 0xffff0000u);
    ss += v0 * v0 + v1 * v1 + v2 * v2 + v3 * v3;
  }
  for (int k0 = threadIdx.x * 8; k0 < d; k0 += 2048) {   // d is a multiple of 256
    float v[8], y[8];
    bf16_to_float8(src + k0, v);
    *reinterpret_cast<float4 *>(x + (size_t)r * d + k0) = make_float4(v[0], v[1], v[2], v[3]);
    *reinterpret_cast<float4 *>(x + (size_t)r * d + k0 + 4) = make_float4(v[4], v[5], v[6], v[7]);
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = v[e] * gain[k0 + e];
    packed_store8(xp, m, k0, y, kts);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  if (threadIdx.x == 0) ssq[r] = (red[0] + red[1]) + (red[2] + red[3]);
}

void launch_embed_dense(const void *emb, const int32_t *ids_dev, int rows, int d, const float *gain, float *x, void *Xp,
                        int RB, float *ssq, hipStream_t s) {
  embed_dense_kernel<<<packed_row_groups(rows), 256, 0, s>>>((const uint16_t *)emb, ids_dev, rows, d, gain, x, (u32x4 *)Xp, (size_t)RB * 128, ssq);
}

// Draft head input of every slot of the chunk whose next token is known (Eq. 2):
// [RMSNorm(x_r) * gain ; embedding of the following token] -> packed, K = 2d.
__global__ __launch_bounds__(256) void draft_cat_dense_kernel(const float *x, int rows, int d, const float *gain, float eps,
                                                              const uint16_t *emb, const int32_t *next_ids, u32x4 *Xp,
                                                              size_t kts) {
  __shared__ float red[4];
  const int r = packed_row(), rb = r >> 4, m = r & 15;
  if (r >= rows) return;
  const float *xr = x + (size_t)r * d;
  float ss = 0.f;
  for (int k0 = threadIdx.x * 4; k0 < d; k0 += 1024) {
    const float4 v = *reinterpret_cast<const float4 *>(xr + k0);
    ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  const float rinv = 1.0f / sqrtf(((red[0] + red[1]) + (red[2] + red[3])) / (float)d + eps);
  u32x4 *xp = Xp + (size_t)rb * 128;
  const uint16_t *e = emb + (size_t)next_ids[r] * d;
  for (int k0 = threadIdx.x * 8; k0 < d; k0 += 2048) {
    float y[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = xr[k0 + e] * rinv * gain[k0 + e];
    packed_store8(xp, m, k0, y, kts);
    bf16_to_float8(e + k0, y);
    packed_store8(xp, m, d + k0, y, kts);
  }
}

void launch_draft_cat_dense(const float *x, int rows, int d, const float *gain, float eps, const void *emb,
                            const int32_t *next_ids, void *Xp, int RB, hipStream_t s) {
  draft_cat_dense_kernel<<<packed_row_groups(rows), 256, 0, s>>>(x, rows, d, gain, eps, (const uint16_t *)emb, next_ids, (u32x4 *)Xp, (size_t)RB * 128);
}

// ------------------------------------------------------------------ causal attention of a prompt chunk
// q: float [rows][H*HD] of the chunk (already rotated); chunk row i sits at slot pos0 + i and
// sees slots 0..pos0+i of the tiled cache (which already holds the chunk's own K and V).
// Pairs (row, query head of the KV head's group) are numbered r = row*G + head%G; a wave owns
// MT tiles of 16 consecutive pairs, a workgroup 64*MT pairs, and walks the visible keys 32 at a time with an
// online softmax.  The K and V tiles of a step (16 KB at head_dim 128) are shared through
// double-buffered LDS: read by every wave for itself they take the whole 64 bytes a cycle of the vector cache.
// Per step the softmax is worth about as many cycles as the products, and the waves of a workgroup are in the same
// phase, so each wave runs the two side by side: the scores of step s+1 (buffer: K of s+1 beside V of s) are
// multiplied while the probabilities of step s are worked out.  The mask is applied only where the diagonal
// crosses the tile, rescaling only where a maximum grew, row sums stay per lane until the end, maxima are exchanged
// by row swaps.
__device__ __forceinline__ float max_across_groups(float v) {   // maximum over the four lane groups (l, l^16, l^32, l^48)
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

template <int HD, int MT>
__global__ __launch_bounds__(256, 2) void attn_prefill_kernel(const float *q, int rows, int pos0, int H, int Hkv, int n_ctx,
                                                              const u32x4 *Kc, const u32x4 *Vc, u32x4 *Xp_out, size_t kts,
                                                              float scale_log2e) {
  constexpr int DT = HD / 32, VT = HD / 16, KP = 2 * DT * 64, VP = VT * 64, NL = KP / 256;   // 16-byte pieces of a step
  __shared__ u32x4 kv[2][KP + VP];   // K tiles [2][DT][64] of step s+1, V tiles [VT][64] of step s
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4, m = lane & 15;
  const int kh = blockIdx.x, G = H / Hkv, R = rows * G;
  // Long tiles (late rows) first; with at most two workgroups per compute unit all are resident at once, and the
  // second half of the list runs the other way so that every unit gets a long and a short one.
  const int T = gridDim.y, y = blockIdx.y, half = (T + 1) / 2;
  const int tile = (int)(gridDim.x * gridDim.y) > 512 || y < half ? T - 1 - y : y - half;
  const int r0 = (tile * 4 + w) * (16 * MT);
  int row[MT], head[MT], limit[MT], clear_kb[MT];
  bool rok[MT];
  u32x4 qh[MT][DT], ql[MT][DT];
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    const int r = r0 + t * 16 + m;
    rok[t] = r < R;
    const int rr = rok[t] ? r : R - 1;
    row[t] = rr / G;
    head[t] = kh * G + rr % G;
    limit[t] = pos0 + row[t];   // last slot this lane's row may see
    clear_kb[t] = pos0 + min(r0 + t * 16, R - 1) / G - 31;   // steps up to here are visible to every row of the tile
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const float *src = q + ((size_t)row[t] * H + head[t]) * HD + dt * 32 + g * 8;
      const float4 a = *reinterpret_cast<const float4 *>(src), b = *reinterpret_cast<const float4 *>(src + 4);
      uint32_t h0, h1, h2, h3, l0, l1, l2, l3;
      split2(a.x * scale_log2e, a.y * scale_log2e, h0, l0);
      split2(a.z * scale_log2e, a.w * scale_log2e, h1, l1);
      split2(b.x * scale_log2e, b.y * scale_log2e, h2, l2);
      split2(b.z * scale_log2e, b.w * scale_log2e, h3, l3);
      qh[t][dt] = u32x4{h0, h1, h2, h3};
      ql[t][dt] = u32x4{l0, l1, l2, l3};
    }
  }
  // last slot any row of the wave sees (a wave behind the last pair only helps to load); last step of the workgroup
  const int last_key = r0 < R ? pos0 + min(r0 + 16 * MT - 1, R - 1) / G : -1;
  const int last_step = (pos0 + min((tile + 1) * (64 * MT) - 1, R - 1) / G) >> 5;

  float mx[MT], lsum[MT];
  f32x4 O[MT][VT];
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    mx[t] = -INFINITY;
    lsum[t] = 0.f;
#pragma unroll
    for (int dt = 0; dt < VT; ++dt) O[t][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // the K tiles of a step are contiguous in the cache, and so are its V tiles; steps behind the last repeat it (ignored)
  const u32x4 *kp = Kc + (size_t)kh * (n_ctx / 16) * DT * 64 + tid, *vp = Vc + (size_t)kh * (n_ctx / 32) * VP + tid;
  u32x4 sa[2 * NL], sb[2 * NL];
  auto issue_k = [&](u32x4 *st, int s) {
#pragma unroll
    for (int i = 0; i < NL; ++i) st[i] = kp[(size_t)min(s, last_step) * KP + i * 256];
  };
  auto issue = [&](u32x4 (&st)[2 * NL], int s) {   // K of step s+1, V of step s
    issue_k(st, s + 1);
#pragma unroll
    for (int i = 0; i < NL; ++i) st[NL + i] = vp[(size_t)min(s, last_step) * VP + i * 256];
  };
  auto stash = [&](const u32x4 (&st)[2 * NL], int buf) {
#pragma unroll
    for (int i = 0; i < 2 * NL; ++i) kv[buf][tid + i * 256] = st[i];
  };
  auto scores = [&](f32x4 (&S)[MT][2], const u32x4 *ks) {
#pragma unroll
    for (int t = 0; t < MT; ++t) S[t][0] = S[t][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const u32x4 k0 = ks[dt * 64], k1 = ks[(DT + dt) * 64];
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        S[t][0] = mfma_bf16(k0, qh[t][dt], S[t][0]);
        S[t][1] = mfma_bf16(k1, qh[t][dt], S[t][1]);
      }
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        S[t][0] = mfma_bf16(k0, ql[t][dt], S[t][0]);
        S[t][1] = mfma_bf16(k1, ql[t][dt], S[t][1]);
      }
    }
  };
  // step s: S holds its scores, N receives those of step s+1
  auto step = [&](int s, int buf, f32x4 (&S)[MT][2], f32x4 (&N)[MT][2]) {
    const int kb = s * 32;
    if (kb > last_key) return;   // wave-uniform
    const u32x4 *ks = kv[buf] + lane, *vs = ks + KP;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      if (kb > clear_kb[t]) {
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
          for (int e = 0; e < 4; ++e) S[t][kt][e] = kb + kt * 16 + 4 * g + e <= limit[t] ? S[t][kt][e] : -INFINITY;
      }
      float bmax = fmaxf(fmaxf(fmaxf(S[t][0][0], S[t][0][1]), fmaxf(S[t][0][2], S[t][0][3])),
                         fmaxf(fmaxf(S[t][1][0], S[t][1][1]), fmaxf(S[t][1][2], S[t][1][3])));
      bmax = max_across_groups(bmax);
      if (__any(bmax > mx[t])) {   // finite from the first step on: slot 0 is visible to every row
        const float mnew = fmaxf(mx[t], bmax), alpha = __builtin_amdgcn_exp2f(mx[t] - mnew);
        mx[t] = mnew;
        lsum[t] *= alpha;
#pragma unroll
        for (int dt = 0; dt < VT; ++dt) O[t][dt] *= alpha;
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    scores(N, ks);
    u32x4 ph[MT], pl[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      float bsum = 0.f;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          S[t][kt][e] = __builtin_amdgcn_exp2f(S[t][kt][e] - mx[t]);
          bsum += S[t][kt][e];
        }
      lsum[t] += bsum;   // this lane's share of the row
      // P^T as B operand: k-slot e of lane group g = key 16*(e/4) + 4g + e%4 of the 32-key block
      uint32_t h0, h1, h2, h3, l0, l1, l2, l3;
      split2(S[t][0][0], S[t][0][1], h0, l0);
      split2(S[t][0][2], S[t][0][3], h1, l1);
      split2(S[t][1][0], S[t][1][1], h2, l2);
      split2(S[t][1][2], S[t][1][3], h3, l3);
      ph[t] = u32x4{h0, h1, h2, h3};
      pl[t] = u32x4{l0, l1, l2, l3};
    }
    // interleave: K tiles ahead of their products, about 3 vector instructions to an MFMA
    __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
    for (int i = 0; i < 4 * DT * MT / 2; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
      __builtin_amdgcn_sched_group_barrier(0x402, 7, 0);
      if (i % 2 == 0) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int dt = 0; dt < VT; dt += 2) {   // two tiles at a time: four products between the two of an accumulator
      const u32x4 v0 = vs[dt * 64], v1 = vs[(dt + 1) * 64];
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        O[t][dt] = mfma_bf16(v0, ph[t], O[t][dt]);
        O[t][dt + 1] = mfma_bf16(v1, ph[t], O[t][dt + 1]);
      }
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        O[t][dt] = mfma_bf16(v0, pl[t], O[t][dt]);
        O[t][dt + 1] = mfma_bf16(v1, pl[t], O[t][dt + 1]);
      }
    }
    __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
    for (int i = 0; i < VT * MT / 2; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
      if (i < VT - 4) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
  };
  f32x4 SA[MT][2], SB[MT][2];
  issue_k(sb, 0);
#pragma unroll
  for (int i = 0; i < NL; ++i) kv[1][tid + i * 256] = sb[i];
  issue(sa, 0);
  issue(sb, 1);
  __syncthreads();
  scores(SA, kv[1] + lane);
  stash(sa, 0);
  __syncthreads();
  for (int s = 0; s <= last_step; s += 2) {
    issue(sa, s + 2);
    __builtin_amdgcn_sched_barrier(0);
    step(s, 0, SA, SB);
    __builtin_amdgcn_sched_barrier(0);
    stash(sb, 1);
    __syncthreads();
    issue(sb, s + 3);
    __builtin_amdgcn_sched_barrier(0);
    step(s + 1, 1, SB, SA);
    __builtin_amdgcn_sched_barrier(0);
    stash(sa, 0);
    __syncthreads();
  }
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    lsum[t] += __shfl_xor(lsum[t], 16, 64);
    lsum[t] += __shfl_xor(lsum[t], 32, 64);
    if (rok[t]) {
      const float inv = 1.0f / lsum[t];
      u32x4 *xp = Xp_out + (size_t)(row[t] >> 4) * 128;
#pragma unroll
      for (int dt = 0; dt < VT; ++dt)
        packed_store4<true>(xp, row[t] & 15, head[t] * HD + dt * 16 + 4 * g, O[t][dt][0] * inv, O[t][dt][1] * inv,
                      O[t][dt][2] * inv, O[t][dt][3] * inv, kts);
    }
  }
}

template <int MT>
static void launch_attention_prefill_tiles(const float *q, int rows, int pos0, const ae_config &c, const void *kv_layer,
                                           size_t v_off, void *Xp_out, int RB, hipStream_t s) {
  const int G = c.n_heads / c.n_kv_heads, R = rows * G, HD = c.head_dim;
  const dim3 grid(c.n_kv_heads, (R + 64 * MT - 1) / (64 * MT));
  const float scale_log2e = 1.4426950408889634f / sqrtf((float)HD);
  const u32x4 *Kc = (const u32x4 *)kv_layer, *Vc = (const u32x4 *)((const char *)kv_layer + v_off);
  const int cap = kv_capacity(c);
  if (HD == 128)
    attn_prefill_kernel<128, MT><<<grid, 256, 0, s>>>(q, rows, pos0, c.n_heads, c.n_kv_heads, cap, Kc, Vc, (u32x4 *)Xp_out,
                                                     (size_t)RB * 128, scale_log2e);
  else
    attn_prefill_kernel<64, MT><<<grid, 256, 0, s>>>(q, rows, pos0, c.n_heads, c.n_kv_heads, cap, Kc, Vc, (u32x4 *)Xp_out,
                                                    (size_t)RB * 128, scale_log2e);
}

// Two tiles a wave read each K and V tile from LDS half as often, one tile a wave gives twice the workgroups.  The
// larger reuse pays where the walks are long (most keys lie before the chunk) and there is work for all 256 compute
// units: 32 heads of 128, 2048 rows, 83 us with one tile and 96 with two without a context, 310 and 286 behind 2048 or
// 4096 slots, 1633 rows (416 workgroups of two tiles a wave) behind 6144 slots 456 and 438; 100 rows 7.6 and 11.6.
void launch_attention_prefill(const float *q, int rows, int pos0, const ae_config &c, const void *kv_layer, size_t v_off,
                              void *Xp_out, int RB, hipStream_t s) {
  const long wgs = (long)c.n_kv_heads * ((rows * (c.n_heads / c.n_kv_heads) + 127) / 128);
  if (pos0 >= rows && wgs >= 384) launch_attention_prefill_tiles<2>(q, rows, pos0, c, kv_layer, v_off, Xp_out, RB, s);
  else launch_attention_prefill_tiles<1>(q, rows, pos0, c, kv_layer, v_off, Xp_out, RB, s);
}

}  // namespace ae
