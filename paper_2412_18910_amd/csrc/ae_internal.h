// Internal declarations of libadaeagle (gfx950).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <string>
#include <tuple>
#include <vector>

#include "adaeagle.h"

namespace ae {

constexpr int kMaxRows = 16;       // rows of one verify / prefill block (one MFMA tile)
constexpr int kAttnChunk = 256;    // keys per split-KV workgroup (fixed by absolute slot)
constexpr int kMaxSplits = 64;     // n_ctx_max / kAttnChunk upper bound
constexpr int kMfmaKeysPerWave = 64;                     // bf16 matrix-core attention: keys per wave,
constexpr int kMfmaAttnChunk = 4 * kMfmaKeysPerWave;     // keys per workgroup (4 waves)
constexpr int kMaxLdlpHidden = 1024;
constexpr int kDenseMinPrompt = 17;   // prompts of one 16-row block go through the decode kernels

// Device-resident step state.  The host mirrors kv_len (it learns it at every accept).
struct DevState {
  int32_t n_acc;            // result of the last accept
  int32_t bonus;
  int32_t k_next;           // Eq. 3 result for the next step
  float y_next;             // LDLP scalar before rounding
  int32_t draft_ids[kMaxRows];
  int32_t override_ids[kMaxRows];
  // Device-gated DDD chain (reset together with override_ids): every kernel of a draft token
  // past the predicted length reads draft_live at entry and returns when it is 0; draft_len
  // counts the tokens drafted.
  int32_t draft_live;
  int32_t draft_len;
  int32_t block[kMaxRows];  // ids of the verify block
  int32_t argmax[kMaxRows]; // per-row argmax of the last LM-head call
  double u_draft[kMaxRows];
  double u_accept[kMaxRows];
  float cum_logp;           // log-probability of the current draft sequence (DDD exit rule)
  float draft_lp[kMaxRows]; // per-token log-probabilities
};
static_assert(offsetof(DevState, u_draft) % 8 == 0, "doubles must stay aligned");

// Pinned host memory that the device writes and the host polls: a copy of the device state, and flag words that a
// kernel sets behind its last write (release, system scope).  A flag holds the number of the request it answers.
struct HostMirror {
  DevState st;
  alignas(64) uint32_t published;   // state copies
  uint32_t imported;                // feature rows taken over (ae_set_state)
  uint32_t decision;                // DDD rule behind a draft token: number << 1 | go on
};

// Launch whose own result is returned, whatever error was pending before it: such an error stays pending (a failed
// launch itself leaves none behind).
template <typename... P, typename... A>
hipError_t launch_checked(void (*kernel)(P...), dim3 grid, dim3 block, hipStream_t s, A... args) {
  std::tuple<P...> typed(args...);
  const hipError_t e = std::apply(
      [&](P &...p) {
        void *ptrs[] = {(void *)&p...};
        return hipLaunchKernel((const void *)kernel, grid, block, ptrs, 0, s);
      },
      typed);
  if (e != hipSuccess) (void)hipGetLastError();
  return e;
}

// A kernel launched with a non-null gate pointer does nothing when *gate == 0.
#define AE_GATE(gate)                          \
  do {                                         \
    if ((gate) != nullptr && *(gate) == 0) return; \
  } while (0)

// Weight matrix handle: row-major source plus (bf16 fast path) the re-tiled copy.
struct Mat {
  const void *rowmajor = nullptr;  // caller's [N,K]
  void *tiled = nullptr;           // ctx-owned MFMA-tile layout, bf16 only
  const void *part[3] = {nullptr, nullptr, nullptr};   // float32: row-major sources of a fused matrix
  int N = 0, K = 0;
};

struct LayerW {
  const float *attn_norm = nullptr, *ffn_norm = nullptr;
  Mat wq, wk, wv, wo, w_gate, w_up, w_down;
  Mat f_qkv, f_gu;   // fused [q;k;v] and [gate,up]: bf16 tiled (gate and up row-blocks interleaved), float32 by parts
};

}  // namespace ae

struct ae_ctx {
  ae_config cfg{};
  hipStream_t stream = nullptr;
  int device = 0;
  bool fast = false;            // bf16 weights and cache (else float32)
  std::string err;

  // weights
  const void *tok_emb = nullptr;
  const float *final_norm = nullptr;
  ae::Mat lm_head, draft_fc, ldlp_in;
  const float *draft_fc_b = nullptr, *ldlp_b_in = nullptr, *ldlp_b_res = nullptr;
  const void *ldlp_w_res = nullptr;
  const float *ldlp_w_out = nullptr, *ldlp_b_out = nullptr;
  std::vector<ae::LayerW> layers;  // n_layers target layers + the draft layer last
  std::vector<void *> owned;       // device allocations to free

  // KV cache: per layer K in d-group-major layout, V row-major (see kernels_attn.hip)
  void *kv = nullptr;
  size_t kv_layer_stride = 0;      // bytes between layers
  size_t kv_v_offset = 0;          // bytes from a layer's K to its V
  float2 *rope_tab = nullptr;      // [n_ctx_max][head_dim/2] (cos, sin)
  float *kv_stage = nullptr;       // this device's address of the library's static staging array

  // activations (float, kMaxRows rows each)
  float *x = nullptr, *q = nullptr;
  float *F = nullptr;              // feature rows (post final norm)
  float *logits = nullptr;         // [k_max+1][V]
  float *dlogits = nullptr;        // [k_max][V]
  float *attn_part = nullptr;      // split-KV partials
  float *ldlp_z = nullptr;         // LDLP hidden vector
  // GEMM inputs (bf16: packed B operands; float32: 16 rows, row-major) and RMSNorm partial sums
  void *xp_a = nullptr, *xp_f = nullptr, *xp_att = nullptr, *xp_h = nullptr, *xp_cat = nullptr;
  float *ssq_a = nullptr, *ssq_f = nullptr;
  float *amax_val = nullptr;       // LM-head argmax partials [16][vocab/16]
  int32_t *amax_idx = nullptr;
  float *lse_sum = nullptr;        // LM-head softmax partials [16][vocab/16] (DDD rule)
  int Pa = 0;                      // number of valid partial-sum rows in ssq_a
  double *prob = nullptr;          // T>0 scratch: segment / row statistics of the sampling kernels
  int32_t *hist = nullptr;         // device token history by slot
  ae::DevState *st = nullptr;      // device state
  ae::HostMirror *hm = nullptr;    // pinned host memory the device writes; hm_dev: its address on the device
  ae::HostMirror *hm_dev = nullptr;
  float *h_rows = nullptr;         // pinned: two exported rows (logits, feature, K/V); h_rows_dev: on the device
  float *h_rows_dev = nullptr;
  float *h_feat = nullptr;         // pinned: the feature row of ae_set_state; read by request feat_seq
  float *h_feat_dev = nullptr;
  uint32_t feat_seq = 0;
  size_t row_floats = 0;           // floats of such a row, a multiple of kExportPiece; a flag word per piece follows the two
  // rows fetched one after the other (ae_get_logits, ae_get_draft_logits): the last one, and the one behind it, on its way
  const float *last_row = nullptr, *ahead_row = nullptr;
  uint32_t ahead_seq = 0;
  int row_half = 0;                // of h_rows, where the last row went
  int logit_rows = 0, draft_rows = 0;   // rows that the last verification, prompt or draft wrote
  uint32_t seq = 0;                // number of the last request to the device

  // dense prompt pass: chunk buffers, allocated at the first long prompt (pxa normalised rows, pxh FFN rows, pxcat draft head
  // input, pxatt attention output, packed or float32 planes; pxf and the partial sums are bf16 only)
  int prefill_mode = 0;            // AE_PREFILL_AUTO / _BLOCKS / _DENSE
  int dense_chunk = 0;             // rows per dense pass (multiple of 128); 0: as ensure_dense has it
  int dense_limit = 0;             // 0, or what a chunk is held to because more could not be had
  int dense_cap = 0;               // rows the buffers below hold
  std::vector<void *> dense_owned;
  float *px = nullptr, *pq = nullptr, *prinv = nullptr, *pssq_a = nullptr, *pssq_f = nullptr;
  void *pxa = nullptr, *pxf = nullptr, *pxatt = nullptr, *pxh = nullptr, *pxcat = nullptr;
  float *ppart = nullptr;          // sums over pieces of K of the GEMMs that split it
  size_t ppart_floats = 0;

  // host-side state machine
  int kv_len = 0, dlen = 0, nF = 0;
  int cur_k = 0, cur_k_last = 0, block_rows = 0;
  int ddd_mode = AE_DDD_DEVICE;    // AE_DDD_HOST / AE_DDD_DEVICE
  bool k_on_device = false;        // the last draft's length is only known on the device (st->draft_len)
  const int32_t *gate = nullptr;   // gate of the kernels being enqueued (device-gated DDD chain), else nullptr
  int32_t pending = 0;
  bool have_pending = false, have_draft = false, have_verify = false, k_next_valid = false;
  int k_next = 0;
  float y_next = 0.f;
  std::vector<int32_t> h_hist;     // host mirror of the token history
  std::vector<int32_t> h_block;

  // per-kernel event timing of the gate/up GEMM launches (see ae_set_kernel_timing)
  bool ktime = false;
  std::vector<hipEvent_t> kt_ev;   // pairs (begin, end)
  int kt_used = 0;
  double kt_total_us = 0.0;
  long long kt_count = 0;

  // profiling
  bool profiling = false;
  hipEvent_t ev[5] = {nullptr, nullptr, nullptr, nullptr, nullptr};
  ae_phase_times last_times{};
};

namespace ae {

// Where the embedding kernels take the ids of their rows from: a device array; or the block of a verification, put
// together and recorded in st->block on the way: host values (v), or hist[kv_len] and the draft tokens.
struct BlockIds {
  const int32_t *ids = nullptr;
  DevState *st = nullptr;
  const int32_t *hist = nullptr;
  int32_t kv_len = 0, v[kMaxRows] = {};
};
// Host inputs of a draft (-1: no override); they travel as kernel arguments.  st == nullptr: none.
struct DraftInputs {
  DevState *st = nullptr;
  int32_t override_ids[kMaxRows] = {}, n_u = 0;
  double u[kMaxRows] = {};
};
// Rows that argmax_finish normalises beside its own work (the features of a forward).
struct NormRows {
  const float *x = nullptr, *gain = nullptr;
  float *out = nullptr;
  int rows = 0, d = 0;
  float eps = 0.f;
};
// Greedy acceptance evaluated by the LDLP's input kernel (st == nullptr: not).
struct GreedyAccept {
  DevState *st = nullptr;
  int32_t *hist = nullptr;
  int kv_len = 0, rows = 0, k_on_device = 0;
};

// ---- dtype-independent kernels (kernels_generic.hip); all launches are asynchronous on `s` ----
void launch_rmsnorm(const float *x, const float *g, int rows, int d, float eps, float *out, hipStream_t s);
// k_on_device: the draft length is st->draft_len (the block is padded to `rows` rows)
void launch_accept_greedy(DevState *st, int32_t *hist, int kv_len, int rows, bool k_on_device, hipStream_t s);
// z0 = W_in [e ; f] + b_in (Eq. 3 input layer), e and f read in place; st_nacc != nullptr: slot and
// row relative to the acceptance result in *st_nacc; ga.st: the greedy acceptance is evaluated here first
void launch_ldlp_in(const void *W, const float *bias, const void *emb, int dtype, const int32_t *hist, const float *F, int d,
                    int in_mode, int h, int slot, int f_row, const DevState *st_nacc, const GreedyAccept &ga, float *z0,
                    hipStream_t s);
// also copies the whole device state to `mirror` and answers request `seq` there
void launch_ldlp_tail(const float *z0, const void *w_res, int dtype, const float *b_res, const float *w_out,
                      const float *b_out, int h, int n_res, int k_max, int cls, DevState *st, HostMirror *mirror,
                      uint32_t seq, hipStream_t s);
// mirror->st = *st, written by the device itself, as the answer to request `seq`
void launch_publish_state(const DevState *st, HostMirror *mirror, uint32_t seq, hipStream_t s);
// F[0..d) = feat[0..d) (pinned host memory), hist2[0..2) = two ids, then mirror->imported = seq
hipError_t launch_set_state(const float *feat, int d, float *F, int32_t *hist2, int32_t last_tok, int32_t pending, HostMirror *mirror,
                            uint32_t seq, hipStream_t s);
// dst[0..n) = src[0..n), dst in pinned host memory; flags[p] = seq behind piece p of kExportPiece floats
constexpr size_t kExportPiece = 4096;
hipError_t launch_export_row(const float *src, size_t n, float *dst, uint32_t *flags, uint32_t seq, hipStream_t s);
void launch_rope_table(float2 *tab, int n_pos, int head_dim, float base, hipStream_t s);
void launch_fill_zero(void *p, size_t bytes, hipStream_t s);

// ---- attention (kernels_attn.hip) ----
size_t kv_layer_bytes(const ae_config &c);
size_t kv_v_offset_bytes(const ae_config &c);
int kv_capacity(const ae_config &c);   // n_ctx_max rounded up to a whole attention chunk
// bf16 MFMA attention over the tiled cache layout (kernels_attn_mfma.hip)
void attention_mfma_setup();   // once per context set-up: dynamic LDS limit of the kernels
void launch_attention_mfma(const float *q, int rows, int pos0, const ae_config &c, const void *kv_layer, size_t v_off,
                           float *part, void *Xp_out, hipStream_t s, const int32_t *gate = nullptr);
// merge of split-KV partials (log2-domain maxima) into the input of the output projection: packed bf16 hi/lo, or
// float32 rows [rows][n_heads * head_dim]
void launch_attention_merge(const float *part, int rows, int n_chunks, const ae_config &c, void *out, bool f32, hipStream_t s,
                            const int32_t *gate);
void launch_kv_import(void *kv_layer, size_t v_off, const ae_config &c, const float *k_dev, const float *v_dev, int n,
                      bool tiled, hipStream_t s);
hipError_t launch_kv_export(const void *kv_layer, size_t v_off, const ae_config &c, int which, int slot, float *out_dev,
                            bool tiled, hipStream_t s);
size_t attn_part_floats(const ae_config &c);

// ---- T > 0 sampling (kernels_sample.hip) ----
size_t sample_scratch_doubles(int V);   // size of the scratch that sampling and acceptance take
// k = draft tokens the block holds room for (rows - 1); k_on_device: only the first
// st->draft_len of them were drafted (padded block of the device-gated DDD chain); u: k + 1 uniforms
void launch_accept_sample(const float *tl, const float *dl, int V, int k, bool k_on_device, float T, DevState *st,
                          int32_t *hist, int kv_len, const double *u, double *prob, hipStream_t s);

// ---- bf16 decode GEMMs (kernels_mfma.hip) ----
// Row-block nb of a row-major [N,K] matrix -> row-block nb_off + nb*nb_stride of a fused
// k-major tiled matrix with NBtot row-blocks.
void launch_retile(const void *rowmajor, int N, int K, void *tiled, int NBtot, int nb_off, int nb_stride, int perm_hd,
                   hipStream_t s);
enum { EPI_STORE = 0, EPI_RESID = 1, EPI_SWIGLU = 2, EPI_QKV = 3 };
struct GemmLaunch {
  const Mat *W = nullptr;         // fused matrix: N = all output rows, K
  const void *Xp = nullptr;       // activations: packed (bf16) or float32 rows of stride ldx
  int ldx = 0, ldxo = 0;          // float32: row strides of Xp and Xp_out
  int rows = 0, row0 = 0;         // output row m reads packed row row0 + m
  const float *ssq_in = nullptr;  // != nullptr: fused RMSNorm, [P_in][16] partial sums of x^2
  int P_in = 0;
  float eps = 0.f;
  const float *bias = nullptr;
  int epi = EPI_STORE;
  int nseg = 1;                   // output segments (q | k | v)
  float *Y[3] = {nullptr, nullptr, nullptr};
  int ldy[3] = {0, 0, 0};
  int seg_N[3] = {0, 0, 0};
  void *Xp_out = nullptr;         // output for the next GEMM, in the form of its Xp
  const float *gain_out = nullptr;
  float *ssq_out = nullptr;
  float *amax_val = nullptr;      // LM head: argmax partials per row and row-block [16][N/16]
  int32_t *amax_idx = nullptr;
  float *lse_sum = nullptr;       // with amax_val: sum of exp((x - block max) * lse_inv_t) per row and row-block
  float lse_inv_t = 1.f;
  // EPI_QKV: rotary embedding + KV append fused into the epilogue
  const float2 *rope_tab = nullptr;
  void *Kc = nullptr, *Vc = nullptr;
  int pos0 = 0, n_ctx = 0, hd = 0;
  const int32_t *gate = nullptr;  // see AE_GATE
};
void launch_gemm_mfma(const GemmLaunch &L, hipStream_t s);
void gemm_mfma_setup(int num_cus);   // once per context set-up: compute-unit count for the shape table
// Where the kernel that fixes a draft token leaves that token's embedding: row `row`, second
// half (k = d .. 2d-1) of the draft head's packed input.  Xp == nullptr: nowhere.
struct DraftCat {
  const void *emb = nullptr;   // embedding table [V][d]
  void *Xp = nullptr;          // packed (bf16) or float32 rows [16][2d]
  int d = 0, row = 0, f32 = 0;
};
// DDD bookkeeping folded into the kernel that fixes draft token i: the token's
// log-probability under softmax(logits / T) from the LM-head epilogue's row-block statistics
// (block maxima `val`, block sums `lse_sum`), the running sum, the drafted length and the exit
// rule for the next token (st->draft_live = 0 when i + 1 >= k and the sum is below theta).  lse_sum == nullptr: rule off.
struct DddFinish {
  const float *val = nullptr, *lse_sum = nullptr;
  const float *logits = nullptr;   // the token's logit row
  int NB = 0, k = 0;
  float inv_t = 1.f, theta = 0.f;
  uint32_t *flag = nullptr;        // nullable: host word that receives seq << 1 | (the rule goes on)
  uint32_t seq = 0;
};
void launch_argmax_finish(const float *val, const int32_t *idx, int NB, int rows, DevState *st, int pick_i, hipStream_t s,
                          const int32_t *gate = nullptr, DraftCat cat = DraftCat(), DddFinish ddd = DddFinish(),
                          const NormRows &norm = NormRows());
// temperature > 0: draft token i by inverse CDF, and what launch_argmax_finish does with a greedy one
void launch_sample_draft(const float *logits, int V, float T, DevState *st, int i, double *scratch, hipStream_t s,
                         const int32_t *gate, DraftCat cat, DddFinish ddd);
void launch_embed_packed(const void *emb, const BlockIds &ids, int rows, int d, const float *gain, float *x,
                         void *Xp, float *ssq, hipStream_t s);
void launch_pack_rows(const float *src, int ld, int rows, int K, const float *gain, void *Xp, hipStream_t s);
void launch_draft_cat_packed(const float *feat, int feat_ld, const void *emb, const int32_t *next_ids, int rows, int d,
                             void *Xp, hipStream_t s, const DraftInputs &in);

// ---- dense prompt pass (kernels_dense.hip); packed buffers hold RB row-blocks ----
// Same GemmLaunch as the decode GEMM (rows = rows of the chunk, row0 unused); rinv != nullptr
// folds RMSNorm in (1/rms per row, from launch_rinv_finalize or rinv_out below).  part: room for
// part_floats floats, used where K is split.  Returns true if so: EPI_RESID and EPI_STORE (L.gain_out
// set, Y stored for EPI_RESID only) have then left 1/rms (with L.eps) of every output row in rinv_out,
// else partial sums of x^2 in L.ssq_out.
bool launch_gemm_dense(const GemmLaunch &L, int RB, const float *rinv, hipStream_t s, float *part, size_t part_floats,
                       float *rinv_out = nullptr);
void launch_rinv_finalize(const float *ssq, int RBused, int P, int K, float eps, float *rinv, hipStream_t s);
void launch_embed_dense(const void *emb, const int32_t *ids_dev, int rows, int d, const float *gain, float *x, void *Xp,
                        int RB, float *ssq, hipStream_t s);
void launch_draft_cat_dense(const float *x, int rows, int d, const float *gain, float eps, const void *emb,
                            const int32_t *next_ids, void *Xp, int RB, hipStream_t s);
void launch_attention_prefill(const float *q, int rows, int pos0, const ae_config &c, const void *kv_layer, size_t v_off,
                              void *Xp_out, int RB, hipStream_t s);

// ---- float32 models (kernels_f32.hip) ----
void launch_gemm_f32(const GemmLaunch &L, hipStream_t s);         // 1..16 rows, all epilogues and fusions
// Prompt GEMMs, any number of rows; activations in planes of RB row-blocks (kernels_f32.hip), already normalised: EPI_QKV
// and EPI_SWIGLU (planes out); part: room for max_part floats, used where the last tiles are made in pieces of K
void launch_gemm_f32_dense(const GemmLaunch &L, int RB, float *part, size_t max_part, hipStream_t s);
// x = Xp . W^T + base (row stride base_ld, nullable), Xp_out = RMSNorm(x) * gain (nullable); part: room for max_part
// floats, at least rows * N
void launch_gemm_f32_resid_norm(const GemmLaunch &L, int RB, float *part, size_t max_part, const float *base, size_t base_ld, float *x,
                                const float *gain, void *Xp_out, hipStream_t s);
// [RMSNorm(x) * gain ; embedding of the token that follows (emb == nullptr: no second half)] -> planes
void launch_norm_cat_f32(const float *x, int rows, int d, const float *gain, float eps, const void *emb, const int32_t *next_ids,
                         void *Xp, int RB, hipStream_t s);
size_t planes_bytes(int rows, int K);   // activations of K columns
void launch_attention_f32(const float *q, int rows, int pos0, const ae_config &c, const void *kv_layer, size_t v_off,
                          float *part, float *out, hipStream_t s, const int32_t *gate = nullptr);
int attn_f32_chunk_keys();   // keys per split-KV workgroup
void launch_attention_prefill_f32(const float *q, int rows, int pos0, const ae_config &c, const void *kv_layer, size_t v_off,
                                  void *Xp, int RB, hipStream_t s);
void launch_embed_f32(const void *emb, const BlockIds &ids, int rows, int d, const float *gain, float *x, void *Xo, float *ssq,
                      hipStream_t s);
void launch_draft_cat_f32(const float *feat, int feat_ld, const void *emb, const int32_t *next_ids, int rows, int d, void *cat,
                          hipStream_t s, const DraftInputs &in);

}  // namespace ae
