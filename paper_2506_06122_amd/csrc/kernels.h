// Host-callable launchers of every device kernel in the library.  All launches are
// asynchronous on the given stream; pointers are device memory unless noted.
#pragma once
#include "common.h"

// ---- plain one-op-per-kernel path (any storage type; used for fp32 models and as the
// ---- cross-check path for bf16) -------------------------------------------------------
struct GatherRows;
// x[r] = the embedding of tokens[r]; with gather (a decode step) of the row gathered on the way
template <typename T>
void launch_embed(const T* table, const int* tokens, const GatherRows* gather, float* x, int rows, int hidden, hipStream_t s);

// out[r] = x[r] * gain * rsqrt(mean(x[r]^2) + eps)
void launch_rmsnorm_f32(const float* x, const float* gain, float* out, int rows, int hidden, float eps,
                        hipStream_t s);

// out[m][n] = sum_k h[m][k] w[n][k] (+ residual[m][n], which may be out); w is T [N][K].  h = a, or with a gain
// RMSNorm(a) * gain; rows_index (optional) selects the rows of a.  glu (with a gain): w holds N gate rows,
// then N up rows, and out = silu(gate) * up.
struct LinearArgs {
  const float* a;
  int lda;
  const int* rows_index;
  const float* gain;
  float eps;
  float* out;
  int ldo;
  const float* residual;  // row stride ldo
  int M, N, K;
};
template <typename T>
void launch_linear_simple(const LinearArgs& p, const T* w, bool glu, hipStream_t s);

// rotary embedding of q (in place) and k, then k and v of every row go to the row's page
// plain path: bias and per-head RMSNorm of the fused [q | k | v] rows, in place (NULL parts are skipped)
void launch_qkv_bias_norm(float* qkv, const float* bias, const float* q_gain, const float* k_gain, float eps,
                          int rows, int n_q_heads, int n_kv_heads, int dh, hipStream_t s);
template <typename KT>
void launch_rope_kvwrite(float* qkv, const float* cos_sin, const int* row_pos, const int* row_slot,
                         const int* page_table, int max_pages, KT* kv_pool, KvGeom geom, int layer, int rows,
                         int n_q_heads, hipStream_t s);

// causal grouped-query attention of each row over cached positions 0..pos of its slot.  decode: every row is
// another slot's next position; takes rows as the projection (and launch_qkv_bias_norm) left them, rotates
// and caches itself
template <typename KT>
void launch_attention_simple(const float* qkv, const float* cos_sin, float* out, const int* row_pos,
                             const int* row_slot, const int* page_table, int max_pages, KT* kv_pool, KvGeom geom,
                             int layer, int rows, int n_q_heads, bool decode, hipStream_t s);

// top-k routing: idx/wt [rows][top_k]; ties to the lower expert index; wt = softmax of the selected logits
void launch_moe_route(const float* router_logits, int* idx, float* wt, int rows, int n_experts, int top_k,
                      hipStream_t s);
// act[(r,j)][f] = silu(Wg_e h_r)[f] * (Wu_e h_r)[f], e = idx[r][j]; w_gate_up is [E][2*Fe][hidden]
template <typename T>
void launch_moe_gate_up_simple(const float* h, const T* w_gate_up, const int* idx, float* act, int rows,
                               int top_k, int hidden, int expert_ffn, hipStream_t s);
// x[r][n] += sum_j wt[r][j] * (Wd_e act_(r,j))[n]; w_down is [E][hidden][Fe]
template <typename T>
void launch_moe_down_simple(const float* act, const T* w_down, const int* idx, const float* wt, float* x,
                            int rows, int top_k, int hidden, int expert_ffn, hipStream_t s);

// copies whole pages (all layers, all heads, K and V): pairs = (src_page, dst_page) x n
void launch_copy_pages(void* kv_pool, const int* pairs, int n_pairs, int n_layers, long long layer_stride_bytes,
                       long long page_stride_bytes, hipStream_t s);

// page_table[slot * max_pages + index] = page for n (slot, index, page) triples: the entries that
// changed on the host since the table was uploaded
void launch_patch_page_table(int* page_table, int max_pages, const int* triples, int n, hipStream_t s);

void launch_convert_to_f32(const void* src, int dtype, float* dst, long long n, hipStream_t s);

// ---- per-slot decode state -------------------------------------------------------------
struct SlotState {
  int* last_token;       // [slots]
  int* pos;              // [slots] cached positions so far = position of the next fed token
  int* step;             // [slots] response position of the next token to emit
  long long* sample_id;  // [slots]
  float* inv_temp;       // [slots]
  float* top_p;          // [slots]
};

// row r <- slot live[r]: token, position, slot, sampling parameters.  What changed on the host comes along from
// memory mapped for the device: the live list (host_live, kept in `live`), the step's forced tokens and
// sampler words (each may be NULL).
struct GatherRows {
  SlotState st;
  int rows;
  int* live;
  const int* host_live;
  const int* host_forced;
  const unsigned* host_uniform;
  int *token, *pos, *slot, *step, *forced;
  unsigned* uniform;
  float *inv_temp, *top_p;
  long long* sample_id;
};
// The token of row r.  One thread of a row stores; a kernel that reads the rows' tokens does this first, and saves a
// launch.
__device__ inline int gather_row(const GatherRows& a, int r, bool store) {
  const int sl = a.host_live ? a.host_live[r] : a.live[r];
  const int token = a.st.last_token[sl];
  if (store) {
    if (a.host_forced) a.forced[r] = a.host_forced[r];
    if (a.host_uniform) a.uniform[r] = a.host_uniform[r];
    if (a.host_live) a.live[r] = sl;
    a.token[r] = token;
    a.pos[r] = a.st.pos[sl];
    a.slot[r] = sl;
    a.inv_temp[r] = a.st.inv_temp[sl];
    a.top_p[r] = a.st.top_p[sl];
    a.sample_id[r] = a.st.sample_id[sl];
    a.step[r] = a.st.step[sl];
  }
  return token;
}
void launch_gather_decode_rows(const GatherRows& a, hipStream_t s);

// ---- sampling ---------------------------------------------------------------------------
constexpr int kMeetSpins = 128;  // looks of about 0.5 us; the parts of a row finish a phase within a few us of each other
struct SampleRows {
  const float* logits;      // [*][vocab]
  const int* logits_row;    // [rows] row of `logits` each draw reads, or NULL (identity)
  const float* inv_temp;    // [rows], or NULL: inv_temp_all for every row
  const float* top_p;       // [rows], or NULL: top_p_all for every row
  const unsigned* uniforms; // [rows] or NULL -> Philox(seed, sample_id, step)
  const long long* sample_id;  // [rows] (Philox only)
  const int* step;             // [rows] (Philox only)
  const int* forced;        // [rows] or NULL; entries outside [0, vocab) mean "draw"
  unsigned long long seed;
  float inv_temp_all, top_p_all;
  int* tokens;              // out [rows]
  float* logprobs;          // out [rows]
  unsigned long long* weight_sums;  // out [rows] or NULL
  // Scratch that lets a row's two sweeps over the vocabulary run on several workgroups (the
  // sums are integers, so the split changes nothing): both or neither.
  float* part_max = nullptr;               // [rows][kSampleHead]: maxima of the parts, then the words they meet at
  unsigned long long* seg_sums = nullptr;  // [rows][kSampleSegments]
  // any_nucleus = false promises that no row draws with top_p < 1; with it, `nucleus` is the scratch of
  // nucleus_rows rows that lets those rows' sweeps run on several workgroups too.
  bool any_nucleus = true;
  unsigned long long* nucleus = nullptr;   // [nucleus_rows][kNucleusScratch]
  int nucleus_rows = 0;
  int patience = kMeetSpins;               // looks of a part at the others' progress before it leaves its share to them
  // What the draw ends with, where asked for: the token and log-prob in host memory mapped for the
  // device, and the state of slot row_slot[r] (a negative one has none): its next position is
  // row_pos[r] + pos_step, the other fields follow from the row's own.
  int* host_tokens = nullptr;
  float* host_logprobs = nullptr;
  const int* row_slot = nullptr;
  const int* row_pos = nullptr;
  int pos_step = 0;
  SlotState slots{};
};
constexpr int kSampleParts = 64, kSampleSegments = 1024;
constexpr int kMeetWords = 16, kSampleHead = kSampleParts + kMeetWords + 2;  // 32-bit words: what the parts meet at, the random word
constexpr int kNucleusBins0 = 41 * 16;                           // exponents 0..40 x 4 mantissa bits
constexpr int kNucleusHist = kNucleusBins0 + 1024 + 512;         // the three histograms of a row
constexpr int kNucleusCounts = kNucleusHist + kSampleSegments / 2;  // behind 1024 32-bit counts: per part the ids it listed, 32 bits each
constexpr int kNucleusList = kNucleusCounts + kSampleParts / 2;  // the listed ids, shared out among the parts
constexpr int kNucleusListed = 8192;
constexpr int kNucleusScratch = kNucleusList + kNucleusListed;   // 64-bit words
struct KernelTimer;
// timer: brackets every launch under its kernel's name, or NULL
void launch_sample(SampleRows r, int rows, int vocab, hipStream_t s, KernelTimer* timer = nullptr);
void launch_philox_words(unsigned long long seed, const long long* ids, const unsigned* steps, unsigned* out,
                         int n, hipStream_t s);
// out[r] = log softmax(logits[r] * inv_temp)[target[r]]; target < 0 writes 0
void launch_logprob_gather(const float* logits, const int* target, float inv_temp, float* out, int rows,
                           int vocab, hipStream_t s);

// Copies of 4-byte words from host memory mapped for the device, all in one launch.
struct HostCopies {
  static constexpr int kMax = 12;
  int n = 0;
  const int* src[kMax];
  int* dst[kMax];
  int words[kMax];
  template <typename T>
  void add(T* to, const T* from, size_t count) {
    if (!count) return;
    src[n] = (const int*)from;
    dst[n] = (int*)to;
    words[n++] = (int)(count * sizeof(T) / 4);
  }
};
void launch_host_copies(const HostCopies& a, hipStream_t s);
// page_table[list[2 i]][0 .. list[2 i + 1]) = packed[i][..], rows of max_pages; list and packed as above
void launch_upload_page_rows(int* page_table, int max_pages, const int* list, const int* packed, int n, hipStream_t s);
