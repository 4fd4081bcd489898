// Paged grouped-query attention on the matrix cores, head_dim 128, half-precision KV pages in
// the KV_MATRIX element order (common.h).  Queries and probabilities enter the matrix
// instructions as hi + lo half-precision pairs, so keys and values are the only rounded
// operands; the result leaves as hi + lo bf16 planes for the output projection.
//
// Decoding is memory-bound (paper section 2.1) and its attention streams every cached key
// and value once per step, so the kernels are built around that stream: each wavefront
// takes 32 cached positions at a time as sixteen contiguous 1 KiB loads (8 key fragments,
// 8 value fragments), computes transposed scores S^T = K q^T with 16x16x32 f16 matrix
// instructions (columns = the query rows that share the KV head), runs the online softmax
// on the fragment (per-column max and sum are a register reduction plus two cross-lane
// steps), and feeds the probabilities straight back as the B operand of O^T += V^T P^T.
// The value pages are stored in exactly the k-order in which a score fragment holds its
// probabilities, so P never moves between lanes.
//
//   decode  : one workgroup per (KV split, KV head, sample); columns = the G query heads;
//             the rotary embedding of the new query and key and the KV-page write ride in
//             the prologue; its 4 or 8 wavefronts interleave over the split's 32-position groups
//             and merge through LDS; of several splits per sample the last to finish joins the results.
//   decode, shared prompts (optional): in the same launch, workgroups of (split, KV head, up
//             to 4 samples of one prompt) take the prompt's shared pages with the members'
//             query heads as columns, and the per-sample workgroups start after those pages.
//   prefill : one wavefront per (16 or 32 query positions, query head); columns = positions;
//             causal limit per column; a sequence may continue a cached context (its rows
//             then attend to that context too).
#include "kernels_fast.h"

typedef __attribute__((__vector_size__(8 * sizeof(_Float16)))) _Float16 f16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
union Frag {
  uint4 u;
  f16x8 v;
  uint32_t w[4];
  uint16_t h[8];
};
#define MFMA16(a, b, c) __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0)

#define DH 128
#define GROUP_U4 512  // uint4 per 32-position group of one K (or V) block: 32 * 128 * 2 / 16
// Probabilities are scaled by 2^10 before they become half-precision operands, so that the
// small probabilities of a long, flat attention row stay in the normal range; the sums and the output
// accumulators carry the same factor, which the final normalisation divides out.
#define P_SCALE_LOG2 10.0f

// largest value / sum over the 4 lanes that hold a column (16 and 32 lanes apart), in each of them: swaps of
// rows and halves of the wavefront, a few cycles each, where exchanges through LDS cost some sixty
__device__ __forceinline__ float column_max(float x) {
  const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(h[0]), __uint_as_float(h[1]));
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float column_sum(float x) {
  const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(h[0]) + __uint_as_float(h[1]);
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// One 32-position group against this lane's query column, in three parts, so that callers can request the next
// group's keys and values as soon as this one's are used.
//   scores: S^T = K q^T, the lo parts of the query (q[4..7]) first.
__device__ __forceinline__ void group_scores(const Frag (&k)[2][4], const Frag (&q)[8], f32x4& s0, f32x4& s1) {
  s0 = f32x4{0.f, 0.f, 0.f, 0.f};
  s1 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    s0 = MFMA16(k[0][i & 3].v, q[(i + 4) & 7].v, s0);
    s1 = MFMA16(k[1][i & 3].v, q[(i + 4) & 7].v, s1);
  }
}
//   softmax: probabilities as hi + lo half-precision parts.  limit = last visible position of the column; m = the
//   column's maximum in log2 units less P_SCALE_LOG2; l = this lane's share of the column's sum (column_sum at the end);
//   o = unnormalised output^T fragments, rescaled only where the maximum of a column has moved.
//   m carries the scale of the probabilities because what is subtracted from the scores has to be the very number that
//   the sums and partial results go by: its own rounding then cancels, and a probability's exponent is rounded once.
//   The exponentials are bare instructions, which return 0 for results below 2^-126.  Nothing is lost by that: as a
//   half-precision operand such a probability is 0 anyway, and beside the maximum's own 2^10 neither it nor a sum
//   that is rescaled by so little (at most 2^27 terms of 2^10 before) reaches the last bit.
__device__ __forceinline__ void group_softmax(f32x4 s0, f32x4 s1, int tok0, int limit, float scale_log2, float& m,
                                              float& l, f32x4 (&o)[8], Frag& hi, Frag& lo, int lane) {
  if (!__all(tok0 + 31 <= limit)) {
    const int seen = limit - tok0 - 4 * (lane >> 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s0[i] = i <= seen ? s0[i] : -INFINITY;
      s1[i] = 16 + i <= seen ? s1[i] : -INFINITY;
    }
  }
  float mx = fmaxf(fmaxf(fmaxf(s0[0], s0[1]), fmaxf(s0[2], s0[3])), fmaxf(fmaxf(s1[0], s1[1]), fmaxf(s1[2], s1[3])));
  mx = fmaf(column_max(mx), scale_log2, -P_SCALE_LOG2);
  if (__any(mx > m)) {
    const float m_new = fmaxf(m, mx);
    const float alpha = __builtin_amdgcn_exp2f(m - (m_new == -INFINITY ? 0.f : m_new));
    m = m_new;
    l *= alpha;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      o[j][0] *= alpha;
      o[j][1] *= alpha;
      o[j][2] *= alpha;
      o[j][3] *= alpha;
    }
  }
  const float shift = m == -INFINITY ? 0.f : -m;
  float p[8];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    p[i] = __builtin_amdgcn_exp2f(fmaf(s0[i], scale_log2, shift));
    p[4 + i] = __builtin_amdgcn_exp2f(fmaf(s1[i], scale_log2, shift));
  }
  l += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
#pragma unroll
  for (int i = 0; i < 4; ++i) split2_f16(p[2 * i], p[2 * i + 1], hi.w[i], lo.w[i]);
}
//   values: O^T += V^T P^T
__device__ __forceinline__ void group_values(const Frag (&v)[8], const Frag& hi, const Frag& lo, f32x4 (&o)[8]) {
#pragma unroll
  for (int j = 0; j < 8; ++j) o[j] = MFMA16(v[j].v, lo.v, o[j]);
#pragma unroll
  for (int j = 0; j < 8; ++j) o[j] = MFMA16(v[j].v, hi.v, o[j]);
}
// The three together, fragments already in registers.
__device__ __forceinline__ void attend_frags(const Frag (&k)[2][4], const Frag (&v)[8], const Frag (&q)[8], int tok0,
                                             int limit, float scale_log2, float& m, float& l, f32x4 (&o)[8], int lane) {
  f32x4 s0, s1;
  Frag hi, lo;
  group_scores(k, q, s0, s1);
  group_softmax(s0, s1, tok0, limit, scale_log2, m, l, o, hi, lo, lane);
  group_values(v, hi, lo, o);
}

// key and value fragments of one 32-position group from its KV page
__device__ __forceinline__ void load_keys(const uint4* __restrict__ kblk, Frag (&k)[2][4], int lane) {
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) k[t][ks].u = kblk[(t * 4 + ks) * 64 + lane];
}
__device__ __forceinline__ void load_values(const uint4* __restrict__ vblk, Frag (&v)[8], int lane) {
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j].u = vblk[j * 64 + lane];
}
__device__ __forceinline__ void load_group(const uint4* __restrict__ kblk, const uint4* __restrict__ vblk,
                                           Frag (&k)[2][4], Frag (&v)[8], int lane) {
  load_keys(kblk, k, lane);
  load_values(vblk, v, lane);
}

// The same, with the group's key and value fragments streamed from a KV page.
__device__ inline void attend_group(const uint4* __restrict__ kblk, const uint4* __restrict__ vblk,
                                    const Frag (&q)[8], int tok0, int limit, float scale_log2, float& m,
                                    float& l, f32x4 (&o)[8], int lane) {
  Frag k[2][4], v[8];
  load_group(kblk, vblk, k, v, lane);
  attend_frags(k, v, q, tok0, limit, scale_log2, m, l, o, lane);
}

// the 32-position group that starts at position tok0, inside page `page`
__device__ inline const uint4* page_block(const AttnArgs& a, int page, int kv_head, int tok0, int is_v) {
  const int gip = (tok0 % a.geom.page_tokens) >> 5;
  return (const uint4*)(a.kv_pool + kv_block_base(a.geom, a.layer, page, kv_head, is_v)) + gip * GROUP_U4;
}
__device__ inline const uint4* group_block(const AttnArgs& a, int slot, int kv_head, int tok0, int is_v) {
  return page_block(a, a.page_table[(long long)slot * a.max_pages + tok0 / a.geom.page_tokens], kv_head, tok0, is_v);
}

// four consecutive values as hi + lo bf16 parts into an activation buffer
__device__ inline void store4_split(uint16_t* dst, long long lo_offset, float a, float b, float c, float d) {
  uint2 hi, lo;
  split4_bf16(a, b, c, d, hi, lo);
  *(uint2*)dst = hi;
  *(uint2*)(dst + lo_offset) = lo;
}
__device__ inline void store1_split(uint16_t* dst, long long lo_offset, float a) {
  uint32_t hi, lo;
  split2_bf16(a, a, hi, lo);
  dst[0] = (uint16_t)hi;
  dst[lo_offset] = (uint16_t)lo;
}

// element (row b, column k) of the decode result
__device__ inline long long out_offset(const AttnArgs& a, int b, int k) {
  const int q_dim = a.n_q_heads * DH;
  return a.out_frag ? frag_offset(b, k, q_dim >> 5) : plane_offset(b, k, q_dim);
}

// ------------------------------------------------------------------------------ fused decode
// One launch per layer for a decode step: sums nothing and stores nothing in between.
// Prologue: rotary embedding of this sample's G query rows (kept in LDS as hi + lo half-precision parts) and, in the
// workgroup whose split holds the new position, of the new key; that key and the new value
// are written to the sample's page and also kept in LDS.  Main loop: the cached positions
// t0..pos-1 from the pages (t0 = 0 unless the sample's prompt is attended by its group, below).
// The new position itself is attended from LDS as a one-token group, so nothing written in
// this launch is read back from memory.  With several partial results per (sample, KV head)
// the split that finishes last joins them (with shared prompts attn_merge_fused_kernel does).
// EXTRA: the model adds a bias to q, k, v and / or normalises q and k heads (a.extra).
struct DecodeSmem {
  uint16_t* q;   // [2][q_cols][Q_LD] hi parts, lo parts
  int q_cols;
  uint16_t* kv;  // [2][DH]
  float* m;      // [NW][ml_cols], NW = wavefronts of the workgroup
  float* l;      // [NW][ml_cols]
  int ml_cols;
  float* o;      // [NW][16][O_LD]
};
// Row pitches in LDS of the queries and of the wavefronts' outputs: 16 bytes past a multiple of the 64 banks, so that the
// 16 columns' 16-byte reads and stores go to different banks.
constexpr int Q_LD = DH + 8, O_LD = DH + 4;

// elements p[0] and p[64] summed over the split-K planes in ascending order, eight planes'
// loads in flight together
__device__ __forceinline__ void sum_planes(const AttnArgs& a, const float* p, float& x0, float& x1) {
  x0 = 0.f;
  x1 = 0.f;
  constexpr int ZR = 8;
  for (int z = 0; z < a.qkv_planes; z += ZR) {
    const long long st = a.qkv_plane_stride;
    const float* q = p + (long long)z * st;
    const int left = a.qkv_planes - z;
    float u[ZR], w[ZR];
#pragma unroll
    for (int i = 0; i < ZR; ++i) {
      u[i] = i < left ? q[i * st] : 0.f;
      w[i] = i < left ? q[i * st + 64] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < ZR; ++i) {
      x0 += u[i];
      x1 += w[i];
    }
  }
}

// Sum over the split-K planes of this thread's N query elements (x0 = element i, x1 = element
// i + 64 of each column's head), planes in ascending order.  The loads of up to eight planes (four
// with more than four columns) of all columns are in flight together: under load a round trip to memory costs more than
// anything else this kernel does before its main loop.
template <int N>
__device__ __forceinline__ void sum_query_planes(const AttnArgs& a, const float* const (&src)[N], float (&x0)[N],
                                                 float (&x1)[N]) {
  if (a.qkv_planes == 1) {
#pragma unroll
    for (int n = 0; n < N; ++n) {
      x0[n] = 0.f + src[n][0];
      x1[n] = 0.f + src[n][64];
    }
    return;
  }
#pragma unroll
  for (int n = 0; n < N; ++n) x0[n] = x1[n] = 0.f;
  constexpr int ZR = N <= 4 ? 8 : 4;  // planes per round: 64 values in flight per thread
  for (int z = 0; z < a.qkv_planes; z += ZR) {
    float u0[ZR][N], u1[ZR][N];
#pragma unroll
    for (int q = 0; q < ZR; ++q) {
      const bool on = z + q < a.qkv_planes;
      const long long o = (long long)(on ? z + q : z) * a.qkv_plane_stride;
#pragma unroll
      for (int n = 0; n < N; ++n) {
        u0[q][n] = on ? src[n][o] : 0.f;
        u1[q][n] = on ? src[n][o + 64] : 0.f;
      }
    }
#pragma unroll
    for (int q = 0; q < ZR; ++q)
#pragma unroll
      for (int n = 0; n < N; ++n) {
        x0[n] += u0[q][n];
        x1[n] += u1[q][n];
      }
  }
}

// Query staging.  Thread t of the workgroup owns the rotary pairs idx = t + 64 NW n, n < N:
// column idx / 64 (the same in all 64 lanes), pair idx % 64.  rows[n] / heads[n] name the
// sample row and the query head inside its KV group that column holds (row < 0: the column
// is empty).  x0 / x1: the projection's elements, planes summed; cs: cos, sin of the row's position.
// Bias / head norm, the rotary embedding, and the hi + lo half-precision parts into sm.q.
template <bool EXTRA, int N, int NW>
__device__ __forceinline__ void rotate_and_stage(const AttnArgs& a, const DecodeSmem& sm, int kvh, int G,
                                                 const int (&rows)[N], const int (&heads)[N], float (&x0)[N],
                                                 float (&x1)[N], const float2 (&cs)[N]) {
  const int tid = threadIdx.x, i = tid & 63;
#pragma unroll
  for (int n = 0; n < N; ++n) {
    const int col = (tid >> 6) + NW * n;
    float u = 0.f, w = 0.f;
    if (rows[n] >= 0) {  // uniform over the wavefront
      if (EXTRA) qkv_extras(a.extra, (kvh * G + heads[n]) * DH, i, a.extra.q_gain, x0[n], x1[n]);
      const float cc = cs[n].x, sn = cs[n].y;
      u = x0[n] * cc - x1[n] * sn;
      w = x1[n] * cc + x0[n] * sn;
    }
    uint16_t* hi = sm.q + col * Q_LD;
    uint16_t* lo = hi + sm.q_cols * Q_LD;
    split_f16(u, hi[i], lo[i]);
    split_f16(w, hi[i + 64], lo[i + 64]);
  }
}
// the two together, positions read from row_pos (columns of several rows)
template <bool EXTRA, int N>
__device__ __forceinline__ void stage_queries(const AttnArgs& a, const DecodeSmem& sm, int kvh, int G,
                                              const int (&rows)[N], const int (&heads)[N]) {
  const int i = threadIdx.x & 63;
  const int q_dim = a.n_q_heads * DH, kv_dim = a.geom.n_kv_heads * DH;
  const float* src[N];
  float x0[N], x1[N];
  float2 cs[N];  // requested with the planes
#pragma unroll
  for (int n = 0; n < N; ++n) {
    const int b = max(rows[n], 0);  // empty columns read row 0 and are zeroed below
    src[n] = a.qkv_raw + (long long)b * (q_dim + 2 * kv_dim) + (kvh * G + heads[n]) * DH + i;
    cs[n] = *(const float2*)(a.cos_sin + (long long)a.row_pos[b] * DH + 2 * i);
  }
  sum_query_planes<N>(a, src, x0, x1);
  rotate_and_stage<EXTRA, N, 4>(a, sm, kvh, G, rows, heads, x0, x1, cs);
}

// the NW wavefronts' results of 16 columns -> one (max, sum, unnormalised output) per column in
// sm.o[0..NW-1], sm.m, sm.l (columns ml0 ..); every thread of the workgroup calls it
template <int NW>
__device__ __forceinline__ float merged_max(const DecodeSmem& sm, int col) {
  float m = sm.m[col];
#pragma unroll
  for (int w = 1; w < NW; ++w) m = fmaxf(m, sm.m[w * sm.ml_cols + col]);
  return m;
}
template <int NW>
__device__ __forceinline__ float merged_sum(const DecodeSmem& sm, int col) {
  float l = sm.l[col];
#pragma unroll
  for (int w = 1; w < NW; ++w) l += sm.l[w * sm.ml_cols + col];
  return l;
}
template <int NW>
__device__ __forceinline__ void merge_wavefronts(const DecodeSmem& sm, int ml0, float m, float l, const f32x4 (&o)[8],
                                                 int wave, int c, int g, int cols) {
  l = column_sum(l);
  if (g == 0) sm.m[wave * sm.ml_cols + ml0 + c] = m;
  __syncthreads();
  const float M = merged_max<NW>(sm, ml0 + c);
  const float M_use = (M == -INFINITY) ? 0.f : M;
  const float w = exp2f(m - M_use);
  if (g == 0) sm.l[wave * sm.ml_cols + ml0 + c] = l * w;
  if (c < cols) {  // the columns in use
#pragma unroll
    for (int j = 0; j < 8; ++j)
      *(float4*)&sm.o[(wave * 16 + c) * O_LD + 16 * j + 4 * g] = make_float4(o[j][0] * w, o[j][1] * w, o[j][2] * w, o[j][3] * w);
  }
  __syncthreads();
}
// elements e .. e + 3 (e = column * DH + k) of the merged, unnormalised output: the wavefronts' parts in ascending order
template <int NW>
__device__ __forceinline__ float4 merged_out(const DecodeSmem& sm, int e) {
  const float4* at = (const float4*)&sm.o[(e >> 7) * O_LD + (e & 127)];
  float4 v = *at;
#pragma unroll
  for (int w = 1; w < NW; ++w) {
    const float4 u = at[w * (16 * O_LD / 4)];
    v.x += u.x;
    v.y += u.y;
    v.z += u.z;
    v.w += u.w;
  }
  return v;
}

// one workgroup = (own-range split, KV head, sample); wavefront w takes the groups w, w + NW, ...
// of the split.  What the workgroup needs before its main loop comes in three sets of loads:
// (1) the row's position and page-table row, and - they depend on neither - every split-K plane
// of its query columns and of the new key and value; (2) what depends on the position: cos and
// sin, the page of the new position and the page of the wavefront's first group; (3) that
// group's keys and values, in flight while the queries are rotated and staged.
template <bool EXTRA, int NW>
__device__ __forceinline__ void decode_own_range(const AttnArgs& a, const DecodeSmem& sm, int split, int kvh, int b) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, g = lane >> 4, i = lane;
  const int n_kv = a.geom.n_kv_heads;
  const int G = a.n_q_heads / n_kv;
  const int T = a.geom.page_tokens;
  const int pos = a.row_pos[b];
  const int t0 = a.row_t0 ? a.row_t0[b] : 0;
  const int slot = a.row_slot[b];
  const int q_dim = a.n_q_heads * DH, kv_dim = n_kv * DH;
  const float* row = a.qkv_raw + (long long)b * (q_dim + 2 * kv_dim);
  // ---- first set of loads (does not wait for the position)
  constexpr int N = 16 / NW;  // columns of this wavefront
  int rows[N], heads[N];
  const float* src[N];
  float x0[N], x1[N];
#pragma unroll
  for (int n = 0; n < N; ++n) {
    heads[n] = wave + NW * n;  // column = head inside the KV group
    rows[n] = heads[n] < G ? b : -1;
    heads[n] = min(heads[n], G - 1);
    src[n] = row + (kvh * G + heads[n]) * DH + i;
  }
  // the new key (even wavefronts) or value (odd ones); wavefronts 0 and 1 of the split that owns
  // the new position use theirs
  const bool is_v = wave & 1;
  float n0, n1;
  sum_planes(a, row + q_dim + (is_v ? kv_dim : 0) + kvh * DH + i, n0, n1);
  sum_query_planes<N>(a, src, x0, x1);
  const int used = (pos - t0) / a.split_tokens + 1;  // splits that hold at least the new position
  if (split >= used) return;
  const bool owner = split == used - 1;
  const bool direct = used == 1 && t0 == 0;          // the only partial result of this (sample, KV head)
  const bool writer = owner && wave < 2;
  const int t_begin = t0 + split * a.split_tokens;
  const int t_end = min(pos, t_begin + a.split_tokens);  // cached positions only
  int tok0 = t_begin + wave * 32;
  // ---- second set: what depends on the position
  const int* pt = a.page_table + (long long)slot * a.max_pages;
  const float2 rot = *(const float2*)(a.cos_sin + (long long)pos * DH + 2 * i);
  const int new_page = writer ? pt[pos / T] : 0;
  const int first_page = tok0 < t_end ? pt[tok0 / T] : 0;
  // ---- third set: the first group's keys and values
  Frag k[2][4], v[8];
  if (tok0 < t_end)
    load_group(page_block(a, first_page, kvh, tok0, 0), page_block(a, first_page, kvh, tok0, 1), k, v, lane);
  const float scale_log2 = 1.4426950408889634f / sqrtf((float)DH);
  float2 cs[N];
#pragma unroll
  for (int n = 0; n < N; ++n) cs[n] = rot;
  rotate_and_stage<EXTRA, N, NW>(a, sm, kvh, G, rows, heads, x0, x1, cs);
  if (writer) {
    const int tok = pos % T;
    if (!is_v) {
      if (EXTRA) qkv_extras(a.extra, q_dim + kvh * DH, i, a.extra.k_gain, n0, n1);  // wavefront 0
      const uint16_t k0 = f32_to_f16(n0 * rot.x - n1 * rot.y).bits, k1 = f32_to_f16(n1 * rot.x + n0 * rot.y).bits;
      sm.kv[i] = k0;
      sm.kv[i + 64] = k1;
      uint16_t* dst = a.kv_pool_w + kv_block_base(a.geom, a.layer, new_page, kvh, 0);
      dst[kv_k_offset(a.geom, tok, i)] = k0;
      dst[kv_k_offset(a.geom, tok, i + 64)] = k1;
    } else {
      if (EXTRA) qkv_extras(a.extra, q_dim + kv_dim + kvh * DH, i, nullptr, n0, n1);  // wavefront 1: bias only
      const uint16_t v0 = f32_to_f16(n0).bits, v1 = f32_to_f16(n1).bits;
      sm.kv[DH + i] = v0;
      sm.kv[DH + i + 64] = v1;
      uint16_t* dst = a.kv_pool_w + kv_block_base(a.geom, a.layer, new_page, kvh, 1);
      dst[kv_v_offset(a.geom, tok, i)] = v0;
      dst[kv_v_offset(a.geom, tok, i + 64)] = v1;
    }
  }
  __syncthreads();

  Frag q[8];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    q[ks].u = *(const uint4*)&sm.q[c * Q_LD + ks * 32 + g * 8];
    q[4 + ks].u = *(const uint4*)&sm.q[(sm.q_cols + c) * Q_LD + ks * 32 + g * 8];
  }
  float m = -INFINITY, l = 0.f;
  f32x4 o[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) o[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (tok0 < t_end) {  // the first group is in registers already
    // keys of the next group are requested as soon as this one's are used, its values likewise; the page number after
    // that ahead of both (loads return in order)
    int page = pt[min(tok0 + 32 * NW, t_end - 1) / T];
    for (; tok0 + 32 * NW < t_end; tok0 += 32 * NW) {
      const int next = tok0 + 32 * NW, after = pt[min(next + 32 * NW, t_end - 1) / T];
      f32x4 s0, s1;
      Frag hi, lo;
      group_scores(k, q, s0, s1);
      load_keys(page_block(a, page, kvh, next, 0), k, lane);
      group_softmax(s0, s1, tok0, pos - 1, scale_log2, m, l, o, hi, lo, lane);
      group_values(v, hi, lo, o);
      load_values(page_block(a, page, kvh, next, 1), v, lane);
      page = after;
    }
    attend_frags(k, v, q, tok0, pos - 1, scale_log2, m, l, o, lane);
  }
  if (owner && wave == NW - 1) {  // the new position, from LDS: token 0 of a group that starts at pos
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      k[0][ks].u = make_uint4(0, 0, 0, 0);
      k[1][ks].u = make_uint4(0, 0, 0, 0);
      if (c == 0) k[0][ks].u = *(const uint4*)&sm.kv[ks * 32 + g * 8];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      v[j].u = make_uint4(0, 0, 0, 0);
      if (g == 0) v[j].h[0] = sm.kv[DH + 16 * j + c];
    }
    attend_frags(k, v, q, pos, pos, scale_log2, m, l, o, lane);
  }

  merge_wavefronts<NW>(sm, 0, m, l, o, wave, c, g, G);
  const int n_slots = a.n_slots ? a.n_slots : a.n_splits;
  const long long slots0 = ((long long)b * n_kv + kvh) * n_slots;
  // the slots of this (sample, KV head); stored and loaded at the scope of the device where they meet in this launch
  const __amdgpu_buffer_rsrc_t part_o = __builtin_amdgcn_make_buffer_rsrc(a.part_o + slots0 * (16 * DH), 0, n_slots * 16 * DH * 4, 0x00027000);
  const __amdgpu_buffer_rsrc_t part_ml = __builtin_amdgcn_make_buffer_rsrc(a.part_ml + slots0 * 32, 0, n_slots * 32 * 4, 0x00027000);
  const int slot_here = a.slot0 + split;
  for (int e = 4 * tid; e < G * DH; e += 256 * NW) {
    const float4 acc = merged_out<NW>(sm, e);
    if (direct) {
      const float sum = merged_sum<NW>(sm, e >> 7), r = __builtin_amdgcn_rcpf(sum);
      store4_split(a.out + out_offset(a, b, kvh * G * DH + e), a.out_lo_offset, quotient(acc.x, sum, r),
                   quotient(acc.y, sum, r), quotient(acc.z, sum, r), quotient(acc.w, sum, r));
    } else {
      __builtin_amdgcn_raw_buffer_store_b128(u32x4{__float_as_uint(acc.x), __float_as_uint(acc.y), __float_as_uint(acc.z), __float_as_uint(acc.w)},
                                             part_o, e * 4, slot_here * (16 * DH * 4), kDeviceScope);
    }
  }
  if (direct) return;
  if (tid < 16) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(merged_max<NW>(sm, tid)), part_ml, tid * 4, slot_here * 128, kDeviceScope);
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(merged_sum<NW>(sm, tid)), part_ml, 64 + tid * 4, slot_here * 128, kDeviceScope);
  }
  if (!a.tickets) return;  // (uniform) a second launch joins the slots
  // The split that draws the last ticket joins the slots, in their order; as the joined projections do (join_splits):
  // the parts are there when their ticket is drawn, and no fence is needed.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) {
    unsigned* ticket = a.tickets + (b * n_kv + kvh) * kTicketStride;
    const unsigned drawn = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool last = (int)drawn == used - 1;
    if (last) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    sm.m[0] = last ? 1.f : 0.f;
  }
  __syncthreads();
  if (sm.m[0] == 0.f) return;
  for (int e = 4 * tid; e < G * DH; e += 256 * NW) {
    const int col = e >> 7;
    float ms[16], ls[16];
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      const int at = min(s, used - 1) * 128;
      ms[s] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(part_ml, col * 4, at, kDeviceScope));
      ls[s] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(part_ml, 64 + col * 4, at, kDeviceScope));
    }
    u32x4 v[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) v[s] = __builtin_amdgcn_raw_buffer_load_b128(part_o, e * 4, min(s, used - 1) * (16 * DH * 4), kDeviceScope);
    float M = -INFINITY, L = 0.f;
#pragma unroll
    for (int s = 0; s < 16; ++s) M = s < used ? fmaxf(M, ms[s]) : M;
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      ms[s] = s < used ? exp2f(ms[s] - M) : 0.f;
      L += s < used ? ls[s] * ms[s] : 0.f;
    }
    f32x4 acc{0.f, 0.f, 0.f, 0.f};
    auto add = [&](const u32x4& u, float w) {
      const f32x4 f = __builtin_bit_cast(f32x4, u);
      acc[0] += f[0] * w;
      acc[1] += f[1] * w;
      acc[2] += f[2] * w;
      acc[3] += f[3] * w;
    };
#pragma unroll
    for (int s = 0; s < 8; ++s)
      if (s < used) add(v[s], ms[s] / L);
    if (used > 8) {
#pragma unroll
      for (int s = 0; s < 8; ++s) v[s] = __builtin_amdgcn_raw_buffer_load_b128(part_o, e * 4, min(8 + s, used - 1) * (16 * DH * 4), kDeviceScope);
#pragma unroll
      for (int s = 0; s < 8; ++s)
        if (8 + s < used) add(v[s], ms[8 + s] / L);
    }
    store4_split(a.out + out_offset(a, b, kvh * G * DH + e), a.out_lo_offset, acc[0], acc[1], acc[2], acc[3]);
  }
}

// NW = 4: three workgroups per CU (registers capped at 168), for launches that fill the chip.  NW = 8: a
// workgroup has a CU to itself and covers 256 positions per round, for the steps whose (sample, KV head)
// pairs are fewer than the CUs.
template <bool EXTRA, int NW>
__global__ __launch_bounds__(64 * NW, NW == 4 ? 3 : 2) void attn_decode_fused_kernel(
    const float* qkv_raw, const int* row_pos, const int* row_slot, const int* page_table, int n_q_heads, int n_kv_heads,
    int qkv_planes, int max_pages, int page_tokens, int split_tokens, AttnArgs a) {
  a.qkv_raw = qkv_raw;
  a.row_pos = row_pos;
  a.row_slot = row_slot;
  a.page_table = page_table;
  a.n_q_heads = n_q_heads;
  a.geom.n_kv_heads = n_kv_heads;
  a.qkv_planes = qkv_planes;
  a.max_pages = max_pages;
  a.geom.page_tokens = page_tokens;
  a.split_tokens = split_tokens;
  a.row_t0 = nullptr;  // no prompt is attended by its group here
  a.slot0 = 0;
  a.n_slots = 0;
  __shared__ __attribute__((aligned(16))) uint16_t q_s[2 * 16 * Q_LD];
  __shared__ __attribute__((aligned(16))) uint16_t kv_s[2 * DH];
  __shared__ float m_s[NW * 16], l_s[NW * 16];
  __shared__ __attribute__((aligned(16))) float o_s[NW * 16 * O_LD];
  decode_own_range<EXTRA, NW>(a, DecodeSmem{q_s, 16, kv_s, m_s, l_s, 16, o_s}, blockIdx.x, blockIdx.y, blockIdx.z);
}

// ------------------------------------------------------------------------------ shared prompts
// The n samples of a prompt share the prompt's full pages.  A group workgroup = (split of the
// shared positions, KV head, up to 4 samples of one prompt): the members' query heads are the
// columns - 4 G of them in NCT tiles of 16 - so one pass over the shared keys and values serves
// all members, and each member's partial result lands in its own partial slot [0, slot0).
// The same launch holds the own-range workgroups of every sample (decode_own_range from
// row_t0 on); attn_merge_fused_kernel joins the slots.  Every shared position is visible to
// every member (it precedes their prompts' ends), so no causal limit applies here.
template <int NCT, bool EXTRA>
__device__ __forceinline__ void decode_shared_range(const AttnArgs& a, const DecodeSmem& sm, int split, int kvh,
                                                    int grp) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane & 15, g = lane >> 4;
  const int n_kv = a.geom.n_kv_heads;
  const int G = a.n_q_heads / n_kv;
  const int len = a.grp_len[grp];
  const int t_begin = split * a.split_tokens_a;
  if (t_begin >= len) return;
  const int t_end = min(len, t_begin + a.split_tokens_a);
  const int slot = a.grp_slot[grp];
  const int* members = a.grp_rows + grp * GROUP_MEMBERS;
  const float scale_log2 = 1.4426950408889634f / sqrtf((float)DH);

  {
    int rows[4 * NCT], heads[4 * NCT];
#pragma unroll
    for (int n = 0; n < 4 * NCT; ++n) {
      const int col = (tid >> 6) + 4 * n, j = col / G;
      rows[n] = j < GROUP_MEMBERS ? members[j] : -1;
      heads[n] = col % G;
    }
    stage_queries<EXTRA, 4 * NCT>(a, sm, kvh, G, rows, heads);
  }
  __syncthreads();

  // one pass over the range per column tile: the second pass finds the fragments in L2, and the
  // registers stay those of a single tile (three workgroups per CU)
  const int n_slots = a.n_slots ? a.n_slots : a.n_splits;
#pragma unroll 1
  for (int ct = 0; ct < NCT; ++ct) {
    Frag q[8];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      q[ks].u = *(const uint4*)&sm.q[(ct * 16 + c) * Q_LD + ks * 32 + g * 8];
      q[4 + ks].u = *(const uint4*)&sm.q[(sm.q_cols + ct * 16 + c) * Q_LD + ks * 32 + g * 8];
    }
    float m = -INFINITY, l = 0.f;
    f32x4 o[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) o[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int tok0 = t_begin + wave * 32; tok0 < t_end; tok0 += 128)
      attend_group(group_block(a, slot, kvh, tok0, 0), group_block(a, slot, kvh, tok0, 1), q, tok0, 0x7fffffff,
                   scale_log2, m, l, o, lane);
    merge_wavefronts<4>(sm, ct * 16, m, l, o, wave, c, g, 16);
    for (int e = 4 * tid; e < 16 * DH; e += 4 * 256) {
      const int col = ct * 16 + (e >> 7);
      const int j = col / G, hc = col % G;
      const int b = j < GROUP_MEMBERS ? members[j] : -1;
      if (b < 0) continue;
      const long long part = ((long long)b * n_kv + kvh) * n_slots + split;
      *(float4*)(a.part_o + part * (16 * DH) + hc * DH + (e & 127)) = merged_out<4>(sm, e);
    }
    if (tid < 16) {
      const int col = ct * 16 + tid;
      const int j = col / G, hc = col % G;
      const int b = j < GROUP_MEMBERS ? members[j] : -1;
      if (b >= 0) {
        const long long part = ((long long)b * n_kv + kvh) * n_slots + split;
        a.part_ml[part * 32 + hc] = merged_max<4>(sm, col);
        a.part_ml[part * 32 + 16 + hc] = merged_sum<4>(sm, col);
      }
    }
    __syncthreads();  // sm.o is reused by the next tile
  }
}

// workgroups [0, n_groups * n_kv * n_splits_a) take the shared ranges, the rest the own ranges
template <int NCT, bool EXTRA>
__global__ __launch_bounds__(256, 3) void attn_decode_grouped_kernel(AttnArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t q_s[2 * NCT * 16 * Q_LD];
  __shared__ __attribute__((aligned(16))) uint16_t kv_s[2 * DH];
  __shared__ float m_s[4 * NCT * 16], l_s[4 * NCT * 16];
  __shared__ __attribute__((aligned(16))) float o_s[4 * 16 * O_LD];
  const DecodeSmem sm{q_s, NCT * 16, kv_s, m_s, l_s, NCT * 16, o_s};
  const int n_kv = a.geom.n_kv_heads;
  const int n_shared = a.n_groups * n_kv * a.n_splits_a;
  int w = blockIdx.x;
  if (w < n_shared) {
    decode_shared_range<NCT, EXTRA>(a, sm, w % a.n_splits_a, (w / a.n_splits_a) % n_kv, w / (a.n_splits_a * n_kv));
  } else {
    w -= n_shared;
    decode_own_range<EXTRA, 4>(a, sm, w % a.n_splits, (w / a.n_splits) % n_kv, w / (a.n_splits * n_kv));
  }
}

// Merge of the partial results of one (sample, KV head), at most 16 slots, where samples of a prompt have
// attended to its shared pages together.
__global__ __launch_bounds__(256) void attn_merge_fused_kernel(AttnArgs a) {
  __shared__ float w_s[16][16];  // [slot][column] weight 2^(m_s - M) / L
  const int tid = threadIdx.x, kvh = blockIdx.x, b = blockIdx.y;
  const int n_kv = a.geom.n_kv_heads;
  const int G = a.n_q_heads / n_kv;
  const int n_slots = a.n_slots ? a.n_slots : a.n_splits;
  const long long part0 = ((long long)b * n_kv + kvh) * n_slots;
  // Every load is requested at once - the row's position, which tells the slots in use, and all
  // 16 slots' maxima, sums and outputs (up to 4 x 16 values per thread for 8 query heads; slots
  // past the last one read the last one) - and what an unused slot held is dropped afterwards:
  // one round trip to memory instead of three.
  const int t0 = a.row_t0 ? a.row_t0[b] : 0;
  const int pos = a.row_pos[b];
  const int ms = min(tid >> 4, n_slots - 1), mcol = tid & 15;
  const float m_ld = a.part_ml[(part0 + ms) * 32 + mcol];
  const float l_ld = a.part_ml[(part0 + ms) * 32 + 16 + mcol];
  constexpr int E_MAX = 4;  // the first 1024 of the G * DH outputs; more than 8 query heads: the rest below
  float v[E_MAX][16];
#pragma unroll
  for (int i = 0; i < E_MAX; ++i) {
    const int e = tid + 256 * i;
#pragma unroll
    for (int s = 0; s < 16; ++s)
      v[i][s] = e < G * DH ? a.part_o[(part0 + min(s, n_slots - 1)) * (16 * DH) + e] : 0.f;
  }
  const int used_shared = t0 ? (t0 + a.split_tokens_a - 1) / a.split_tokens_a : 0;
  const int used_own = (pos - t0) / a.split_tokens + 1;
  if (used_shared == 0 && used_own == 1) return;  // the attention kernel wrote the result itself
  const unsigned valid = ((1u << used_shared) - 1u) | (((1u << used_own) - 1u) << a.slot0);
#pragma unroll
  for (int i = 0; i < E_MAX; ++i)
#pragma unroll
    for (int s = 0; s < 16; ++s)
      if (!((valid >> s) & 1u)) v[i][s] = 0.f;
  {
    const int s = tid >> 4, col = tid & 15;  // 256 threads = 16 slots x 16 columns
    const bool on = (valid >> s) & 1u;
    const float m = on ? m_ld : -INFINITY;
    const float l = on ? l_ld : 0.f;
    w_s[s][col] = m;
    __syncthreads();
    float M = -INFINITY;
#pragma unroll
    for (int q = 0; q < 16; ++q) M = fmaxf(M, w_s[q][col]);
    const float w = exp2f(m - M);  // 0 for unused slots
    __syncthreads();
    w_s[s][col] = w;
    // total weight of the column, same order in every thread
    __shared__ float lw_s[16][16];
    lw_s[s][col] = l * w;
    __syncthreads();
    float L = 0.f;
#pragma unroll
    for (int q = 0; q < 16; ++q) L += lw_s[q][col];
    __syncthreads();
    w_s[s][col] = w / L;
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < E_MAX; ++i) {
    const int e = tid + 256 * i;
    if (e >= G * DH) break;
    const int col = e >> 7;
    float acc = 0.f;
#pragma unroll
    for (int s = 0; s < 16; ++s) acc += v[i][s] * w_s[s][col];
    store1_split(a.out + out_offset(a, b, kvh * G * DH + e), a.out_lo_offset, acc);
  }
  for (int e = tid + 256 * E_MAX; e < G * DH; e += 256) {
    const int col = e >> 7;
    float u[16];
#pragma unroll
    for (int s = 0; s < 16; ++s) u[s] = ((valid >> s) & 1u) ? a.part_o[(part0 + s) * (16 * DH) + e] : 0.f;
    float acc = 0.f;
#pragma unroll
    for (int s = 0; s < 16; ++s) acc += u[s] * w_s[s][col];
    store1_split(a.out + out_offset(a, b, kvh * G * DH + e), a.out_lo_offset, acc);
  }
}

#define DECODE_ARGS a.qkv_raw, a.row_pos, a.row_slot, a.page_table, a.n_q_heads, a.geom.n_kv_heads, a.qkv_planes, a.max_pages, \
                    a.geom.page_tokens, a.split_tokens, a
void launch_attention_decode_fused(const AttnArgs& a, hipStream_t s) {
  if (!a.rows) return;
  // the kernel takes no prompt's shared part (it would attend to it twice, or leave it out) and joins at most 16 splits, by ticket
  if (a.row_t0 || a.slot0 || a.n_slots || a.n_groups || a.n_splits > 16 || (a.n_splits > 1 && !a.tickets))
    throw HipError(hipErrorInvalidValue, "plain decode attention", __FILE__, __LINE__);
  const dim3 grid(a.n_splits, a.geom.n_kv_heads, a.rows);
  const bool extra = a.extra.bias || a.extra.q_gain;
  if (a.wide) {
    if (extra) attn_decode_fused_kernel<true, 8><<<grid, 512, 0, s>>>(DECODE_ARGS);
    else attn_decode_fused_kernel<false, 8><<<grid, 512, 0, s>>>(DECODE_ARGS);
  } else {
    if (extra) attn_decode_fused_kernel<true, 4><<<grid, 256, 0, s>>>(DECODE_ARGS);
    else attn_decode_fused_kernel<false, 4><<<grid, 256, 0, s>>>(DECODE_ARGS);
  }
}
void launch_attention_merge(const AttnArgs& a, hipStream_t s) {
  if (a.rows) attn_merge_fused_kernel<<<dim3(a.geom.n_kv_heads, a.rows), 256, 0, s>>>(a);
}

template <int NCT>
static void launch_grouped(const AttnArgs& a, unsigned grid, hipStream_t s) {
  if (a.extra.bias || a.extra.q_gain) attn_decode_grouped_kernel<NCT, true><<<grid, 256, 0, s>>>(a);
  else attn_decode_grouped_kernel<NCT, false><<<grid, 256, 0, s>>>(a);
}
void launch_attention_decode_grouped(const AttnArgs& a, hipStream_t s) {
  if (!a.rows) return;
  // slots are joined by launch_attention_merge: a ticket's holder would join them before the shared parts are there
  if (a.tickets) throw HipError(hipErrorInvalidValue, "grouped decode attention", __FILE__, __LINE__);
  const int n_kv = a.geom.n_kv_heads, G = a.n_q_heads / n_kv;
  const unsigned grid = (unsigned)(a.n_groups * n_kv * a.n_splits_a + a.rows * n_kv * a.n_splits);
  if (GROUP_MEMBERS * G <= 16) launch_grouped<1>(a, grid, s);
  else launch_grouped<2>(a, grid, s);
}

// ------------------------------------------------------------------------------ prefill
// A workgroup is one wavefront: CT tiles of 16 positions of one query head, which share every key and value fragment it
// loads.  The next group's keys and values are requested as soon as this one's are used, and the wavefronts with the last,
// longest rows start first.
// What bounds it: the fragments' way from L2 (16 KB per 32 positions and wavefront, about 14 TB/s with two tiles), then
// the products of hi and lo parts.  Per layer, against 16-position wavefronts in workgroups of four that exchanged by
// way of LDS: 7B shape, 10568 rows in 4 sequences 777 -> 522 us; 1.5B shape, 6000 rows in 2 sequences 211 -> 160,
// 187 rows 12.4 -> 7.5.  Two or four wavefronts to a workgroup (ragged sequences leave them unevenly filled): 548, 572.
template <int CT>
__global__ __launch_bounds__(64, 2) void attn_prefill_kernel(AttnArgs a) {
  const int lane = threadIdx.x;
  const int c = lane & 15, g = lane >> 4;
  const int seq = blockIdx.z, head = blockIdx.y;
  const int len = a.seq_len[seq];
  const int q0 = (gridDim.x - 1 - blockIdx.x) * 16 * CT;
  if (q0 >= len) return;
  const int row0 = a.seq_row0[seq];
  const int p0 = a.seq_pos0 ? a.seq_pos0[seq] : 0;  // cached positions before the sequence's first row
  const int kvh = head / (a.n_q_heads / a.geom.n_kv_heads);
  const int* pt = a.page_table + (long long)a.seq_slot[seq] * a.max_pages;
  const int T = a.geom.page_tokens;
  const float scale_log2 = 1.4426950408889634f / sqrtf((float)DH);
  const int last = p0 + min(q0 + 16 * CT, len) - 1;  // last position any row of the wavefront attends to
  Frag k[2][4], v[8];
  load_group(page_block(a, pt[0], kvh, 0, 0), page_block(a, pt[0], kvh, 0, 1), k, v, lane);
  int page = pt[min(32, last) / T];
  Frag q[CT][8];
#pragma unroll
  for (int t = 0; t < CT; ++t) {
    const int qi = min(q0 + 16 * t + c, len - 1);  // rows past the end repeat the last one and are not stored
    const uint16_t* src = a.q + ((long long)(row0 + qi) * a.n_q_heads + head) * DH + g * 8;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      q[t][ks].u = *(const uint4*)(src + ks * 32);
      q[t][4 + ks].u = *(const uint4*)(src + a.q_lo_offset + ks * 32);
    }
  }
  float m[CT], l[CT];
  f32x4 o[CT][8];
#pragma unroll
  for (int t = 0; t < CT; ++t) {
    m[t] = -INFINITY;
    l[t] = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) o[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  f32x4 s0[CT], s1[CT];
  Frag hi[CT], lo[CT];
  auto scores = [&]() {
#pragma unroll
    for (int t = 0; t < CT; ++t) group_scores(k, q[t], s0[t], s1[t]);
  };
  auto rest = [&](int tok0) {
#pragma unroll
    for (int t = 0; t < CT; ++t)
      group_softmax(s0[t], s1[t], tok0, p0 + q0 + 16 * t + c, scale_log2, m[t], l[t], o[t], hi[t], lo[t], lane);
#pragma unroll
    for (int t = 0; t < CT; ++t) group_values(v, hi[t], lo[t], o[t]);
  };
  int tok0 = 0;
  for (; tok0 + 32 <= last; tok0 += 32) {
    const int after = pt[min(tok0 + 64, last) / T];
    scores();
    load_keys(page_block(a, page, kvh, tok0 + 32, 0), k, lane);
    rest(tok0);
    load_values(page_block(a, page, kvh, tok0 + 32, 1), v, lane);
    page = after;
  }
  scores();
  rest(tok0);
#pragma unroll
  for (int t = 0; t < CT; ++t) {
    const int qi = q0 + 16 * t + c;
    const float inv = 1.0f / column_sum(l[t]);
    if (qi >= len) continue;
    uint16_t* dst = a.out + plane_offset(row0 + qi, head * DH + 4 * g, a.n_q_heads * DH);
#pragma unroll
    for (int j = 0; j < 8; ++j)
      store4_split(dst + plane_offset(0, 16 * j, 0), a.out_lo_offset, o[t][j][0] * inv, o[t][j][1] * inv, o[t][j][2] * inv,
                   o[t][j][3] * inv);
  }
}

// Two tiles to a wavefront from 2048 wavefronts (two per SIMD) on; with fewer, CUs would idle.  One tile / two: 72
// wavefronts of two tiles 7.5 / 11.2 us, 1224 14.8 / 16.0, 3840 30.7 / 30.7, 6144 73 / 66.
static bool prefill_pairs(const AttnArgs& a) {
  return (long long)ceil_div(a.max_seq_len, 32) * a.n_q_heads * a.n_seqs >= 2048;
}
const char* attention_prefill_name(const AttnArgs& a) {
  return prefill_pairs(a) ? "attn_prefill_kernel<2>" : "attn_prefill_kernel<1>";
}
void launch_attention_prefill(const AttnArgs& a, hipStream_t s) {
  if (!a.n_seqs) return;
  if (prefill_pairs(a)) attn_prefill_kernel<2><<<dim3(ceil_div(a.max_seq_len, 32), a.n_q_heads, a.n_seqs), 64, 0, s>>>(a);
  else attn_prefill_kernel<1><<<dim3(ceil_div(a.max_seq_len, 16), a.n_q_heads, a.n_seqs), 64, 0, s>>>(a);
}
