// Launchers of the matrix-core (bf16) path: packed-weight projections, fused row kernels
// and paged attention.  Pointers are device memory; launches are asynchronous.
#pragma once
#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "stream_plan.h"
#include "tile_grid.h"

// Kernels of a decode step take what their first loads need as leading scalar arguments, at most 14 dwords, and the rest
// as a struct behind them: the build asks for leading scalars to be preloaded into registers, where the struct is a read
// from memory away (streamed projections, 16 rows: 1536 x 1536 5.5 -> 5.2 us, 1536 x 8960 in 5 splits 9.9 -> 9.3).

// Epilogues of the projection kernels:
//   EPI_F32          out[m][n] fp32 (split-K planes allowed)
//   EPI_SWIGLU_BF16  every column tile holds 8 gates, then their 8 ups: act[m][f] = silu(gate) * up as bf16 hi/lo
//   EPI_RESID        stream kernel only: x[m][n] += result (fp32, in place); h = x * gain as
//                    bf16 hi/lo planes (the next projection's operand, not yet normalised);
//                    ssq_out[workgroup column][m] = sum of x^2 over the workgroup's columns
// Any stream-kernel epilogue first scales row m by rsqrt(sum_p rinv_ssq[p][m] / K + eps) when
// rinv_ssq is given: the second half of the RMSNorm of the projection's input.
//   EPI_LSE          tile kernel only, the teacher-forced log-prob pass: the result z = out *
//                    lse_scale never reaches memory; per (workgroup column, row) the kernel
//                    stores max z and sum exp(z - max) over the workgroup's columns, and the
//                    workgroup that owns column lse_target[m] stores that z (launch_lse_finish
//                    turns these into log-probs)
enum { EPI_F32 = 0, EPI_SWIGLU_BF16 = 1, EPI_RESID = 2, EPI_LSE = 3 };

// Fragment order of an activation plane [rows][K] (decode steps that stream the weights): the
// 16-row x 32-deep operand fragment of the 16x16x32 matrix instruction is stored as one
// contiguous 1 KiB block [lane][8] with lane = (k % 32 / 8) * 16 + row % 16, fragments ordered
// [row / 16][k / 32].  A wavefront then reads an operand fragment as whole cache lines, as it
// reads a weight fragment.  Rows are padded to a multiple of 16 (the pad is never written and
// what is read from it only reaches output rows that are not stored).
__host__ __device__ inline long long frag_offset(int m, int k, int k_tiles) {
  return (((long long)(m >> 4) * k_tiles + (k >> 5)) << 9) + ((((k >> 3) & 3) * 16 + (m & 15)) << 3) + (k & 7);
}

// Interleaved planes of an activation buffer [rows][K] (everything with more rows): a row is K / 32
// blocks of 128 bytes, each holding the hi parts of 32 elements and then their lo parts, so that
// one cache line carries both planes of a k-tile.
constexpr int kPlaneLo = 32;  // elements from a hi part to its lo part
__host__ __device__ inline long long plane_offset(int m, int k, int K) {
  return 2 * (long long)m * K + ((k >> 5) << 6) + (k & 31);
}

constexpr int kTicketStride = 32;  // a ticket has its 128-byte line to itself
constexpr int kDeviceScope = 16;   // cache policy of a buffer access at the scope of the device: sc1

struct GemmArgs {
  const void* a;     // activations as bf16 hi and lo parts: interleaved rows (plane_offset), or with `frag` two
  const void* a_lo;  // planes in fragment order; a_lo = first lo part
  bool frag = false; // stream kernel: `a`, `h` and the EPI_SWIGLU_BF16 result are in fragment order
  const void* w;     // packed bf16 weight, N/16 x K/32 fragments of 1 KiB
  void* out;         // EPI_F32: float [splits][M][ldo]; EPI_SWIGLU_BF16: bf16 [M][ldo] (ldo = N/2)
  int M, N, K, ldo;
  long long out_lo_offset = 0;  // EPI_SWIGLU_BF16: elements from a hi part of `out` to its lo part
  long long split_stride;  // floats between split planes (EPI_F32)
  int k_tiles_per_split;   // filled by the launcher
  TileGrid grid;           // tile kernel: the launch's blocks (launcher)
  // EPI_RESID with K splits: they meet in the launch (join_splits)
  float* join = nullptr;         // [joined tiles][splits] parts of a wavefront
  unsigned* tickets = nullptr;   // one per joined tile, kTicketStride apart, 0 between launches
  // input normalisation (stream kernel)
  const float* rinv_ssq = nullptr;  // [rinv_partials][ssq_stride] partial sums of squares of the input rows
  int rinv_partials = 0;
  int ssq_stride = 0;
  float eps = 0.f;
  // EPI_RESID
  float* x = nullptr;            // [M][N] residual stream, updated in place
  const float* gain = nullptr;   // [N] gain of the RMSNorm that follows
  uint16_t* h = nullptr;         // bf16 [M][N], first hi part
  long long h_lo_offset = 0;     // elements from a hi part of h to its lo part
  float* ssq_out = nullptr;      // [grid columns][ssq_stride]
  // grouped launch (mixture of experts, tile kernel): row block y works on rows
  // [block_row_begin[y], block_row_end[y]) of the expert-sorted order with the weights of
  // group_of_block[y]; row_map maps a sorted row to its source row in `a`.
  const int* group_of_block = nullptr;
  const int* block_row_begin = nullptr;
  const int* block_row_end = nullptr;
  const int* row_map = nullptr;
  long long group_stride16 = 0;  // 16-byte units between consecutive groups' packed weights
  int n_row_blocks = 0;
  // EPI_LSE
  const int* lse_target = nullptr;  // [M] target column of row m, or -1
  float lse_scale = 1.f;            // 1 / temperature
  float* lse_max = nullptr;         // [grid columns][lse_stride]
  float* lse_sum = nullptr;         // [grid columns][lse_stride]
  float* lse_tgt = nullptr;         // [M]
  int lse_stride = 0;
};

// Rows up to which a decode step streams the weights (gemm_stream_kernel).  Above that the activations every
// workgroup re-reads, and the narrow outputs' second row blocks once they no longer find idle CUs (hidden / 16 column
// tiles each: 256 workgroups at 2048), outweigh the two norm launches per layer that the path saves.  Step at 24 rows,
// streamed / as tiles: hidden 1024 1.13 / 1.46 ms, 1536 1.74 / 1.85, 2048 1.25 / 1.36 (16 layers), 2560 1.63 / 1.52 (16
// layers), 3584 4.49 / 4.25.
inline int stream_rows(int hidden) { return hidden <= 2048 ? 32 : 16; }

// How one projection is launched: kind 0 = gemm_stream_kernel, 1 = gemm_tile_kernel; shape = which of the
// kernel's configurations, nt = column tiles per workgroup, splits = K splits (planes, or joined with EPI_RESID).
struct GemmPlan {
  int kind, shape, nt, splits;
  const char* name;  // kernel name as a profiler shows it (without the argument list)
};
GemmPlan gemm_plan(int M, int N, int K, int epi, int max_splits);
GemmPlan gemm_plan_stream(int M, int N, int K, int epi, int max_splits);  // the stream kernel for M <= 32
GemmPlan gemm_plan_grouped(int epi, long long picks, int n_experts);      // experts' row blocks of moe_block_rows
// column parts per row that an EPI_LSE launch with this plan writes, and the most any plan writes
inline int lse_parts(const GemmPlan& pl, int N) { return ceil_div(N >> 4, pl.nt); }
inline int lse_parts_max(int N) { return ceil_div(N >> 4, 8); }
// out[m] = lse_tgt[m] - log sum_n exp(z[m][n]) from the parts of an EPI_LSE launch; 0 where target < 0
void launch_lse_finish(const float* lse_max, const float* lse_sum, const float* lse_tgt, const int* target,
                       int parts, int stride, int rows, float* out, hipStream_t s);
// returns the number of split planes written (EPI_F32; <= plan.splits)
int launch_gemm_bf16(GemmArgs a, int epi, const GemmPlan& plan, hipStream_t s);
// rows of src [N][K] -> fragments.  half < 0: row n to column tile tile_offset + n / 16; half = 0 or 1: row n to
// tile n / 8, columns 8 half .. 8 half + 7 (the gate and up matrices share tiles)
void launch_pack_weight(const void* src, void* dst, int N, int K, int tile_offset, int half, hipStream_t s);

// x[r] (+= sum of `splits` partial planes) ; h[r] = bf16(x[r] * gain * rsqrt(mean(x[r]^2) + eps)).
//   tokens != NULL : x[r] is first loaded from the bf16 embedding row tokens[r]
//   gather.rows    : the same for a decode step, whose rows are gathered on the way
//   rows_index != NULL : source row of x is rows_index[r], x is not written back (final norm)
struct RowNormArgs {
  float* x;
  const float* partial;     // [splits][rows][hidden] or NULL
  long long split_stride;
  int splits;
  const float* gain;
  uint16_t* h;              // bf16 hi and lo parts [rows][hidden], interleaved (plane_offset) unless h_frag
  long long h_lo_offset;    // elements from a hi part to its lo part
  float* ssq_out;           // when set: h = x * gain without the rsqrt factor, ssq_out[r] = sum x[r]^2
  bool h_frag = false;      // h in fragment order
  const int* tokens;
  GatherRows gather{};
  const uint16_t* embed;
  const int* rows_index;
  int rows, hidden;
  float eps;
  // mixture of experts: x[r] += sum_j moe_wt[r][j] * moe_y[moe_slot[r][j]] (picks in order)
  const float* moe_y = nullptr;    // [slots][hidden]
  const int* moe_slot = nullptr;   // [rows][moe_k]
  const float* moe_wt = nullptr;   // [rows][moe_k]
  int moe_k = 0;
};
void launch_row_norm(const RowNormArgs& a, hipStream_t s);

// What some model families do to q, k, v between the projection and the rotary embedding
// (head_dim 128 here: one wavefront holds one head as 64 rotary pairs).
struct QkvExtras {
  const float* bias = nullptr;    // [q | k | v] added to the projection, or NULL
  const float* q_gain = nullptr;  // [128] gains of an RMSNorm over each q head, or NULL
  const float* k_gain = nullptr;  // [128] the same for each k head
  float eps = 0.f;
};
// x0, x1 = elements i and i + 64 of one head, all 64 lanes of the wavefront taking part:
// adds the bias (element offset `off` of the fused row) and normalises the head.
__device__ inline void qkv_extras(const QkvExtras& e, int off, int i, const float* gain, float& x0, float& x1) {
  if (e.bias) {
    x0 += e.bias[off + i];
    x1 += e.bias[off + i + 64];
  }
  if (gain) {
    const float rinv = 1.0f / sqrtf(wave_sum(x0 * x0 + x1 * x1) / 128.0f + e.eps);
    x0 *= rinv * gain[i];
    x1 *= rinv * gain[i + 64];
  }
}

// Sums the split planes of the fused QKV projection, applies the rotary embedding to q and
// k, writes q as bf16 [rows][q_dim] (and optionally as fp32 into q_f32 [rows][q_f32_ld]) and
// stores k, v into the row's KV page (bf16, the pool's element order).
struct QkvPostArgs {
  const float* partial;
  long long split_stride;
  int splits;
  const float* cos_sin;
  const int *row_pos, *row_slot, *page_table;
  int max_pages;
  uint16_t* q_bf16;         // hi plane [rows][q_dim]
  long long q_lo_offset;    // elements to the lo plane
  float* q_f32;
  int q_f32_ld;
  uint16_t* kv_pool;
  KvGeom geom;
  int layer, rows, n_q_heads;
  QkvExtras extra;
};
void launch_qkv_post(const QkvPostArgs& a, hipStream_t s);

constexpr int GROUP_MEMBERS = 4;  // samples of one prompt that attend to its shared pages together

// Paged grouped-query attention on the matrix cores (KV_MATRIX pool, head_dim 128).
struct AttnArgs {
  const uint16_t* q;        // prefill: half-precision hi plane [rows][n_q_heads][128], rotary applied
  long long q_lo_offset;    // elements to its lo plane
  uint16_t* out;            // bf16 hi and lo parts [rows][n_q_heads * 128], interleaved (plane_offset) unless out_frag
  long long out_lo_offset;  // elements from a hi part to its lo part
  bool out_frag = false;    // decode: out in fragment order, K = n_q_heads * 128
  const uint16_t* kv_pool;
  KvGeom geom;
  const int* page_table;
  int max_pages, layer, n_q_heads;
  // decode: one row per sample
  const int *row_pos, *row_slot;
  int rows;
  int n_splits, split_tokens;      // KV range per workgroup (multiple of 128)
  bool wide = false;               // decode: workgroups of 8 wavefronts instead of 4
  float* part_o;                   // [rows][n_kv_heads][n_slots][16][128]
  float* part_ml;                  // [rows][n_kv_heads][n_slots][2][16]
  unsigned* tickets = nullptr;     // decode, plain: one per (row, KV head), kTicketStride apart, 0 between launches
  int n_slots = 0;                 // shared prompts: partial results per (row, KV head); 0: n_splits
  // decode with shared prompts (launch_attention_decode_grouped): the samples of one prompt
  // attend to the prompt's shared pages together - each key and value fragment is read once
  // for all of them - and every row attends alone only to what follows its row_t0.
  const int* row_t0 = nullptr;     // [rows] first position of the row's own range (0 = no shared part)
  int slot0 = 0;                   // partial slots [0, slot0) hold the shared part, [slot0, slot0 + n_splits) the own
  const int* grp_rows = nullptr;   // [n_groups][GROUP_MEMBERS] rows of a group's members, -1 = none
  const int* grp_len = nullptr;    // [n_groups] shared positions (a multiple of 32)
  const int* grp_slot = nullptr;   // [n_groups] page-table row of one member
  int n_groups = 0, n_splits_a = 0, split_tokens_a = 0;  // shared part: splits of split_tokens_a (multiple of 128)
  // decode (rotary, KV write and attention in one launch)
  const float* qkv_raw;            // fp32 [planes][rows][(n_q_heads + 2 n_kv_heads) * 128], projections before
                                   // rotary, as split-K planes that the kernel sums in ascending order
  int qkv_planes;                  // >= 1
  long long qkv_plane_stride;      // floats between planes
  const float* cos_sin;
  QkvExtras extra;                 // decode: bias / per-head norm of the new q, k, v
  uint16_t* kv_pool_w;
  // prefill: packed sequences
  const int *seq_row0, *seq_len, *seq_slot;
  const int* seq_pos0 = nullptr;   // position of each sequence's first row (NULL = 0): rows that
                                   // continue a cached context attend to it as well
  int n_seqs, max_seq_len;
};
void launch_attention_prefill(const AttnArgs& a, hipStream_t s);
const char* attention_prefill_name(const AttnArgs& a);  // the kernel it launches, as a profiler shows it
// Decode attention: the result is final; with several splits (a.n_splits > 1) it goes through the
// partial results and a.tickets.
void launch_attention_decode_fused(const AttnArgs& a, hipStream_t s);
// the same with shared prompts, partial results per (row, KV head, slot) for launch_attention_merge; needs n_q_heads / n_kv_heads <= 8 (4 members x heads <= 32 columns)
void launch_attention_decode_grouped(const AttnArgs& a, hipStream_t s);
void launch_attention_merge(const AttnArgs& a, hipStream_t s);

// ---- policy-gradient objective over packed rollouts (kernels_loss.hip) ----------------------
struct PolicyLossArgs {
  int n_seqs;
  long long total;            // tokens = cu_seqlens[n_seqs]
  const int* host_cu;         // [n_seqs + 1] and
  const float* host_rewards;  // [n_seqs], in host memory mapped for the device
  int* cu_seqlens;            // the same two on the device, filled by the first launch
  float* rewards;
  const float *logp_new, *logp_old, *logp_ref;  // [total]; logp_ref may be NULL
  const unsigned char* mask;  // [total] 1 = the token counts
  float gamma, kl_coef, reward_clip, adv_clip, eps_low, eps_high;
  float* grad;                // [total] d loss / d logp_new
  float* advantages;          // [total] or NULL
  int n_parts;                // workgroups that count the mask, at most kLossParts
  int* part_count;            // [n_parts] counted tokens
  float* part_sum;            // [n_seqs] sum over the sequence's tokens, in mapped host memory
  int* count;                 // [1] N, in mapped host memory
};
constexpr int kLossParts = 512;
// longest: tokens of the longest sequence
void launch_policy_loss(const PolicyLossArgs& p, int longest, hipStream_t s);

// ---- mixture-of-experts block on the matrix-core path ---------------------------------------
// Routing: sums the split planes of the router projection, picks the top_k experts of every
// row by (logit descending, expert index ascending), mixes with the softmax over the picked
// logits, and takes each pick's position inside its expert's list from an integer counter.
struct MoeRouteArgs {
  const float* partial;     // [splits][rows][n_experts] router logits (split planes)
  long long split_stride;
  int splits;
  int rows, n_experts, top_k;
  int* idx;                 // [rows][top_k] expert of pick j
  float* wt;                // [rows][top_k] mixing weight of pick j
  int* pos;                 // [rows][top_k] position of the pick inside its expert's list
  int* count;               // [n_experts], zero on entry: picks per expert
  int* route_log;           // optional copy of idx (parity hook)
};
void launch_moe_route_topk(const MoeRouteArgs& a, hipStream_t s);

// Plan of the grouped projections: expert-sorted slots, cut into row blocks.
struct MoePlanArgs {
  const int* count;         // [n_experts]
  const int* idx;           // [rows * top_k]
  const int* pos;           // [rows * top_k]
  int rows, n_experts, top_k, max_blocks, block_rows;
  int* row_map;             // [rows * top_k] slot -> source row
  int* slot_of;             // [rows * top_k] (row, pick) -> slot
  int* group_of_block;      // [max_blocks]
  int* block_row_begin;     // [max_blocks]
  int* block_row_end;       // [max_blocks]; unused blocks get begin = end = 0
};
void launch_moe_plan(const MoePlanArgs& a, hipStream_t s);
// Rows per block of the grouped projections, by the picks an expert gets on average; the columns go with them
// (gemm_plan_grouped).
constexpr int kMoeMinBlockRows = 32;
inline int moe_block_rows(long long picks, int n_experts) { return picks <= 14ll * n_experts ? 32 : 64; }
