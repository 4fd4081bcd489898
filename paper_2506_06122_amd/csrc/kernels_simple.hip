// Plain one-operator-per-kernel path: fp32 activations, weights and KV cache in any
// storage type.  It serves fp32 models and cross-checks the matrix-core path.  What bounds it at the
// sizes it is used at (a few layers, a few rows) is latency and the number of launches, so a layer
// is five kernels in a decode step - projections take the norm before them and the SwiGLU behind
// them, attention the rotary embedding and the cache write - and each asks for all it reads at once.
// Operators: paper section 2.1 names the phases (prefill, decoding); the
// operator definitions are the standard ones of the model families in section 5.1.
#include "kernels.h"

// ---------------------------------------------------------------- embedding
// tokens NULL: a decode step, whose rows are gathered on the way (two launches of 3.4 and 2.1 us before; a step of 14
// launches 80 -> 78 us)
template <typename T>
__global__ void embed_kernel(const T* __restrict__ table, const int* __restrict__ tokens,
                             float* __restrict__ x, int hidden, GatherRows gather) {
  int r = blockIdx.x;
  const T* src = table + (long long)(tokens ? tokens[r] : gather_row(gather, r, threadIdx.x == 0)) * hidden;
  for (int i = threadIdx.x; i < hidden; i += blockDim.x) x[(long long)r * hidden + i] = to_f32(src[i]);
}
template <typename T>
void launch_embed(const T* table, const int* tokens, const GatherRows* gather, float* x, int rows, int hidden, hipStream_t s) {
  if (rows) embed_kernel<T><<<rows, 256, 0, s>>>(table, gather ? nullptr : tokens, x, hidden, gather ? *gather : GatherRows{});
}
template void launch_embed<float>(const float*, const int*, const GatherRows*, float*, int, int, hipStream_t);
template void launch_embed<bf16_t>(const bf16_t*, const int*, const GatherRows*, float*, int, int, hipStream_t);

// ---------------------------------------------------------------- RMSNorm
__global__ void rmsnorm_f32_kernel(const float* __restrict__ x, const float* __restrict__ gain,
                                   float* __restrict__ out, int hidden, float eps) {
  __shared__ float partial[4];
  int r = blockIdx.x;
  const float* src = x + (long long)r * hidden;
  float ss = 0.f;
  for (int i = threadIdx.x; i < hidden; i += blockDim.x) ss += src[i] * src[i];
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) partial[threadIdx.x >> 6] = ss;
  __syncthreads();
  float total = partial[0] + partial[1] + partial[2] + partial[3];
  float rinv = 1.0f / sqrtf(total / (float)hidden + eps);
  for (int i = threadIdx.x; i < hidden; i += blockDim.x)
    out[(long long)r * hidden + i] = src[i] * gain[i] * rinv;
}
void launch_rmsnorm_f32(const float* x, const float* gain, float* out, int rows, int hidden, float eps,
                        hipStream_t s) {
  if (rows) rmsnorm_f32_kernel<<<rows, 256, 0, s>>>(x, gain, out, hidden, eps);
}

// ---------------------------------------------------------------- linear
// One wavefront per output column (GLU: per gate column and its up column) and tile of LIN_ROWS rows:
// a lane takes four consecutive k of every 256.  With a gain the rows are RMS-normalised on the way: the
// gain multiplies the operand, the row's sum of squares is gathered beside the products, and
// 1 / rms the result.  The eight row sums of a wavefront are folded, half of the rows to each half
// of the lanes at each step: 10 exchanges in place of 48.
// 8 rows x 512..1376 columns x 256: 3.7 us with norm (4.8 us with the SwiGLU), where one value per lane and row
// at a time took 16 us, behind a norm of 4.2 us and before a SwiGLU of 4.6 us.
#define LIN_ROWS 8
template <typename T, bool VEC>
__device__ inline float4 load_quad_f32(const T* p, int k, int K) {  // values k .. k + 3, zero from K on
  float v[4] = {0.f, 0.f, 0.f, 0.f};
  if (VEC) {  // K is a multiple of four: all or nothing
    const T* q = p + (k < K ? k : 0);
    if (sizeof(T) == 4) {
      const float4 w = *(const float4*)q;
      v[0] = w.x, v[1] = w.y, v[2] = w.z, v[3] = w.w;
    } else {
      T w[4];
      *(uint2*)w = *(const uint2*)q;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = to_f32(w[e]);
    }
    if (k >= K) v[0] = v[1] = v[2] = v[3] = 0.f;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (k + e < K) v[e] = to_f32(p[k + e]);
  }
  return make_float4(v[0], v[1], v[2], v[3]);
}
__device__ inline float dot4(const float4& a, const float4& b, float acc) {
  return fmaf(a.w, b.w, fmaf(a.z, b.z, fmaf(a.y, b.y, fmaf(a.x, b.x, acc))));
}
// sums v[i] over the wavefront; lane l holds the sum of row l >> 3
__device__ inline float fold_rows(const float (&v)[LIN_ROWS], int lane) {
  float a[4], b[2], c;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    a[i] = (lane & 32 ? v[i + 4] : v[i]) + __shfl_xor(lane & 32 ? v[i] : v[i + 4], 32, WAVE);
#pragma unroll
  for (int i = 0; i < 2; ++i)
    b[i] = (lane & 16 ? a[i + 2] : a[i]) + __shfl_xor(lane & 16 ? a[i] : a[i + 2], 16, WAVE);
  c = (lane & 8 ? b[1] : b[0]) + __shfl_xor(lane & 8 ? b[0] : b[1], 8, WAVE);
#pragma unroll
  for (int o = 4; o > 0; o >>= 1) c += __shfl_xor(c, o, WAVE);
  return c;
}

template <typename T, bool NORM, bool GLU, bool VEC>
__global__ __launch_bounds__(256) void linear_simple_kernel(const T* __restrict__ w, const float* a, const float* gain, const int* rows_index,
                                                            int lda, int M, int N, int K, LinearArgs p) {
  p.a = a;
  p.gain = gain;
  p.rows_index = rows_index;
  p.lda = lda;
  p.M = M;
  p.N = N;
  p.K = K;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int n = blockIdx.x * 4 + wave, m0 = blockIdx.y * LIN_ROWS;
  if (n >= p.N) return;
  const float* row[LIN_ROWS];  // rows past the last repeat it, their results are dropped
#pragma unroll
  for (int i = 0; i < LIN_ROWS; ++i) {
    const int m = min(m0 + i, p.M - 1);
    row[i] = p.a + (long long)(p.rows_index ? p.rows_index[m] : m) * p.lda;
  }
  const T *wr = w + (long long)n * p.K, *wu = w + (long long)(n + p.N) * p.K;
  float acc[LIN_ROWS] = {}, up[LIN_ROWS] = {}, ss[LIN_ROWS] = {};
#pragma unroll 2
  for (int k = 4 * lane; k - 4 * lane < p.K; k += 4 * WAVE) {
    float4 wv = load_quad_f32<T, VEC>(wr, k, p.K), uv, gv;
    if (GLU) uv = load_quad_f32<T, VEC>(wu, k, p.K);
    if (NORM) gv = load_quad_f32<float, VEC>(p.gain, k, p.K);
    float4 av[LIN_ROWS];
#pragma unroll
    for (int i = 0; i < LIN_ROWS; ++i) av[i] = load_quad_f32<float, VEC>(row[i], k, p.K);
#pragma unroll
    for (int i = 0; i < LIN_ROWS; ++i) {
      if (NORM) {
        ss[i] = dot4(av[i], av[i], ss[i]);
        av[i] = make_float4(av[i].x * gv.x, av[i].y * gv.y, av[i].z * gv.z, av[i].w * gv.w);
      }
      acc[i] = dot4(av[i], wv, acc[i]);
      if (GLU) up[i] = dot4(av[i], uv, up[i]);
    }
  }
  float v = fold_rows(acc, lane);
  const int m = m0 + (lane >> 3);
  float rinv = 1.f;
  if (NORM) rinv = 1.0f / sqrtf(fold_rows(ss, lane) / (float)p.K + p.eps);
  v *= rinv;
  if (GLU) v = v / (1.0f + expf(-v)) * (fold_rows(up, lane) * rinv);
  if ((lane & 7) == 0 && m < p.M) {
    if (p.residual) v += p.residual[(long long)m * p.ldo + n];
    p.out[(long long)m * p.ldo + n] = v;
  }
}
template <typename T>
void launch_linear_simple(const LinearArgs& p, const T* w, bool glu, hipStream_t s) {
  if (!p.M || !p.N) return;
  const dim3 grid(ceil_div(p.N, 4), ceil_div(p.M, LIN_ROWS));
  const bool vec = p.K % 4 == 0 && p.lda % 4 == 0;  // 16-byte quads: every row of either operand starts on one
  const auto kernel =
      glu      ? (vec ? linear_simple_kernel<T, true, true, true> : linear_simple_kernel<T, true, true, false>)
      : p.gain ? (vec ? linear_simple_kernel<T, true, false, true> : linear_simple_kernel<T, true, false, false>)
               : (vec ? linear_simple_kernel<T, false, false, true> : linear_simple_kernel<T, false, false, false>);
  kernel<<<grid, 256, 0, s>>>(w, p.a, p.gain, p.rows_index, p.lda, p.M, p.N, p.K, p);
}
template void launch_linear_simple<float>(const LinearArgs&, const float*, bool, hipStream_t);
template void launch_linear_simple<bf16_t>(const LinearArgs&, const bf16_t*, bool, hipStream_t);

// ---------------------------------------------------------------- q/k/v bias and per-head norm
// One wavefront per (row, head) of the fused [q | k | v] rows, in place: adds the bias, then
// normalises q and k heads over head_dim with their gains (either part may be absent).
__global__ void qkv_bias_norm_kernel(float* __restrict__ qkv, const float* __restrict__ bias,
                                     const float* __restrict__ q_gain, const float* __restrict__ k_gain, float eps,
                                     int n_q_heads, int n_kv_heads, int dh) {
  const int r = blockIdx.x, head = blockIdx.y * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int n_heads = n_q_heads + 2 * n_kv_heads;
  if (head >= n_heads) return;
  float* x = qkv + ((long long)r * n_heads + head) * dh;
  float ss = 0.f;
  for (int i = lane; i < dh; i += 64) {
    const float v = x[i] + (bias ? bias[head * dh + i] : 0.f);
    x[i] = v;
    ss += v * v;
  }
  const float* gain = head < n_q_heads ? q_gain : head < n_q_heads + n_kv_heads ? k_gain : nullptr;
  if (!gain) return;
  const float rinv = 1.0f / sqrtf(wave_sum(ss) / (float)dh + eps);
  for (int i = lane; i < dh; i += 64) x[i] *= rinv * gain[i];
}
void launch_qkv_bias_norm(float* qkv, const float* bias, const float* q_gain, const float* k_gain, float eps,
                          int rows, int n_q_heads, int n_kv_heads, int dh, hipStream_t s) {
  if (rows && (bias || q_gain))
    qkv_bias_norm_kernel<<<dim3(rows, ceil_div(n_q_heads + 2 * n_kv_heads, 4)), 256, 0, s>>>(
        qkv, bias, q_gain, k_gain, eps, n_q_heads, n_kv_heads, dh);
}

// ---------------------------------------------------------------- RoPE + KV write
// qkv row = [q heads | k heads | v heads] x head_dim.  Half-split pairing: (u_i, u_{i+dh/2})
// rotates by pos * theta^(-2i/dh); cos_sin[pos][i] = (cos, sin) interleaved.
template <typename KT>
__global__ void rope_kvwrite_kernel(float* __restrict__ qkv, const float* __restrict__ cos_sin,
                                    const int* __restrict__ row_pos, const int* __restrict__ row_slot,
                                    const int* __restrict__ page_table, int max_pages, KT* __restrict__ kv_pool,
                                    KvGeom g, int layer, int n_q_heads) {
  int r = blockIdx.x;
  int dh = g.head_dim, half = dh >> 1;
  int pos = row_pos[r];
  int n_heads = n_q_heads + 2 * g.n_kv_heads;
  float* row = qkv + (long long)r * n_heads * dh;
  int page = page_table[(long long)row_slot[r] * max_pages + pos / g.page_tokens];
  int tok = pos % g.page_tokens;
  const float* cs = cos_sin + (long long)pos * dh;  // half pairs of (cos, sin)
  for (int idx = threadIdx.x; idx < n_heads * half; idx += blockDim.x) {
    int head = idx / half, i = idx % half;
    float a = row[head * dh + i], b = row[head * dh + i + half];
    if (head < n_q_heads + g.n_kv_heads) {
      float c = cs[2 * i], sn = cs[2 * i + 1];
      float ra = a * c - b * sn, rb = b * c + a * sn;
      a = ra;
      b = rb;
    }
    if (head < n_q_heads) {
      row[head * dh + i] = a;
      row[head * dh + i + half] = b;
    } else if (head < n_q_heads + g.n_kv_heads) {
      int kvh = head - n_q_heads;
      KT* dst = kv_pool + kv_block_base(g, layer, page, kvh, 0);
      dst[kv_k_offset(g, tok, i)] = from_f32<KT>(a);
      dst[kv_k_offset(g, tok, i + half)] = from_f32<KT>(b);
    } else {
      int kvh = head - n_q_heads - g.n_kv_heads;
      KT* dst = kv_pool + kv_block_base(g, layer, page, kvh, 1);
      dst[kv_v_offset(g, tok, i)] = from_f32<KT>(a);
      dst[kv_v_offset(g, tok, i + half)] = from_f32<KT>(b);
    }
  }
}
template <typename KT>
void launch_rope_kvwrite(float* qkv, const float* cos_sin, const int* row_pos, const int* row_slot,
                         const int* page_table, int max_pages, KT* kv_pool, KvGeom geom, int layer, int rows,
                         int n_q_heads, hipStream_t s) {
  if (rows)
    rope_kvwrite_kernel<KT><<<rows, 256, 0, s>>>(qkv, cos_sin, row_pos, row_slot, page_table, max_pages,
                                                   kv_pool, geom, layer, n_q_heads);
}
template void launch_rope_kvwrite<float>(float*, const float*, const int*, const int*, const int*, int, float*,
                                         KvGeom, int, int, int, hipStream_t);
template void launch_rope_kvwrite<f16_t>(float*, const float*, const int*, const int*, const int*, int, f16_t*,
                                         KvGeom, int, int, int, hipStream_t);

// ---------------------------------------------------------------- attention
// One block of ATT_T threads per (row, query head).  Cached positions are taken ATT_T at a
// time: thread t scores position base + t, the block updates the running max and sum
// (online softmax), then groups of threads, one thread per output dimension, share the positions
// of the weighted sum, eight values in flight each.
// DECODE: every row is another slot's next position.  The block rotates the query and the row's own
// key itself and takes the own position from LDS; the first block of each KV head's query heads
// writes key and value to the cache.  Otherwise rope_kvwrite_kernel has done all this before.
// 8 rows x 4 heads, 32..64 positions of 64: 6.6 us, rotation and cache write included; with one thread walking a
// key or all positions of a dimension value by value 18.8 us, and 4.4 us before it for those two.
#define ATT_T 256
template <typename KT, bool DECODE>
__global__ __launch_bounds__(ATT_T) void attention_simple_kernel(
    const float* __restrict__ qkv, const float* __restrict__ cos_sin, float* __restrict__ out,
    const int* __restrict__ row_pos, const int* __restrict__ row_slot, const int* __restrict__ page_table,
    int max_pages, KT* __restrict__ kv_pool, KvGeom g, int layer, int n_q_heads) {
  __shared__ __align__(16) float q_s[256], k_s[256];
  __shared__ float v_s[256], p_s[ATT_T], acc_s[ATT_T];
  __shared__ long long v_at[ATT_T];
  __shared__ float red[4];
  const int r = blockIdx.x, head = blockIdx.y, t = threadIdx.x;
  const int dh = g.head_dim, group = n_q_heads / g.n_kv_heads, kvh = head / group;
  const int n_heads = n_q_heads + 2 * g.n_kv_heads;
  const int pos = row_pos[r], ctx = pos + 1;
  const int* pages = page_table + (long long)row_slot[r] * max_pages;
  const float scale = 1.0f / sqrtf((float)dh);
  const float* row = qkv + (long long)r * n_heads * dh;
  if (DECODE) {
    const int half = dh >> 1;
    if (t < 2 * half) {  // threads 0 .. half - 1 rotate the query, the next half the key
      const int i = t < half ? t : t - half;
      const float* u = row + (t < half ? head : n_q_heads + kvh) * dh;
      const float cs = cos_sin[(long long)pos * dh + 2 * i], sn = cos_sin[(long long)pos * dh + 2 * i + 1];
      const float a = u[i], b = u[i + half], ra = a * cs - b * sn, rb = b * cs + a * sn;
      if (t < half) {
        q_s[i] = ra;
        q_s[i + half] = rb;
      } else {  // what the cache holds of it
        k_s[i] = to_f32(from_f32<KT>(ra));
        k_s[i + half] = to_f32(from_f32<KT>(rb));
      }
    }
    if (t < dh) v_s[t] = to_f32(from_f32<KT>(row[(n_q_heads + g.n_kv_heads + kvh) * dh + t]));
  } else {
    if (t < dh) q_s[t] = row[head * dh + t];
  }
  __syncthreads();
  if (DECODE && head % group == 0 && t < dh) {
    const int page = pages[pos / g.page_tokens], tok = pos % g.page_tokens;
    kv_pool[kv_block_base(g, layer, page, kvh, 0) + kv_k_offset(g, tok, t)] = from_f32<KT>(k_s[t]);
    kv_pool[kv_block_base(g, layer, page, kvh, 1) + kv_v_offset(g, tok, t)] = from_f32<KT>(v_s[t]);
  }
  const int cached = DECODE ? pos : ctx;  // positions read from the cache
  const int dh2 = dh <= 64 ? 64 : dh <= 128 ? 128 : 256, n_groups = ATT_T / dh2, grp = t / dh2, dim = t % dh2;
  float m = -INFINITY, l = 0.f, acc = 0.f;
  for (int base = 0; base < ctx; base += ATT_T) {
    const int u = base + t;
    float sc = -INFINITY;
    if (u < cached) {
      const int tok = u % g.page_tokens;
      const long long blk = kv_block_base(g, layer, pages[u / g.page_tokens], kvh, 0);
      v_at[t] = blk + (long long)g.page_tokens * dh + kv_v_offset(g, tok, 0);
      const KT* kb = kv_pool + blk + kv_k_offset(g, tok, 0);  // a position's values are contiguous here
      constexpr int V = 16 / sizeof(KT);
      float d[4] = {};
#pragma unroll 8
      for (int i = 0; i < dh; i += V) {
        KT x[V];
        *(uint4*)x = *(const uint4*)(kb + i);
#pragma unroll
        for (int e = 0; e < V; ++e) d[e & 3] = fmaf(q_s[i + e], to_f32(x[e]), d[e & 3]);
      }
      sc = ((d[0] + d[1]) + (d[2] + d[3])) * scale;
    } else if (u < ctx) {
      float d[4] = {};
      for (int i = 0; i < dh; i += 4) {
#pragma unroll
        for (int e = 0; e < 4; ++e) d[e] = fmaf(q_s[i + e], k_s[i + e], d[e]);
      }
      sc = ((d[0] + d[1]) + (d[2] + d[3])) * scale;
    }
    const float cm = wave_max(sc);
    if ((t & 63) == 0) red[t >> 6] = cm;
    __syncthreads();
    const float m_new = fmaxf(m, fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3])));
    __syncthreads();
    const float p = (u < ctx) ? expf(sc - m_new) : 0.f;
    p_s[t] = p;
    const float ps = wave_sum(p);
    if ((t & 63) == 0) red[t >> 6] = ps;
    __syncthreads();
    const float alpha = expf(m - m_new);  // m = -inf on the first chunk gives 0
    l = l * alpha + ((red[0] + red[1]) + (red[2] + red[3]));
    acc *= alpha;
    if (dim < dh) {
      const int n_here = min(ATT_T, cached - base);
      for (int j0 = grp; j0 < n_here; j0 += 8 * n_groups) {
        float v[8], pj[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int j = j0 + e * n_groups, jj = min(j, n_here - 1);
          v[e] = to_f32(kv_pool[v_at[jj] + dim]);
          pj[e] = j < n_here ? p_s[jj] : 0.f;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) acc = fmaf(pj[e], v[e], acc);
      }
      if (DECODE && base + ATT_T >= ctx && grp == 0) acc = fmaf(p_s[pos - base], v_s[dim], acc);
    }
    m = m_new;
    __syncthreads();
  }
  acc_s[t] = acc;
  __syncthreads();
  if (t < dh) {
    for (int k = 1; k < n_groups; ++k) acc += acc_s[k * dh2 + t];
    out[((long long)r * n_q_heads + head) * dh + t] = acc / l;
  }
}
template <typename KT>
void launch_attention_simple(const float* qkv, const float* cos_sin, float* out, const int* row_pos,
                             const int* row_slot, const int* page_table, int max_pages, KT* kv_pool, KvGeom geom,
                             int layer, int rows, int n_q_heads, bool decode, hipStream_t s) {
  if (!rows) return;
  const auto kernel = decode ? attention_simple_kernel<KT, true> : attention_simple_kernel<KT, false>;
  kernel<<<dim3(rows, n_q_heads), ATT_T, 0, s>>>(qkv, cos_sin, out, row_pos, row_slot, page_table, max_pages, kv_pool,
                                                 geom, layer, n_q_heads);
}
template void launch_attention_simple<float>(const float*, const float*, float*, const int*, const int*, const int*, int,
                                             float*, KvGeom, int, int, int, bool, hipStream_t);
template void launch_attention_simple<f16_t>(const float*, const float*, float*, const int*, const int*, const int*, int,
                                             f16_t*, KvGeom, int, int, int, bool, hipStream_t);

// ---------------------------------------------------------------- mixture of experts
// One wavefront per row: k rounds of arg-max over the experts (ties to the lower index),
// then a softmax over the k selected logits.
__global__ void moe_route_kernel(const float* __restrict__ logits, int* __restrict__ idx,
                                 float* __restrict__ wt, int n_experts, int top_k) {
  int r = blockIdx.x, lane = threadIdx.x;
  const float* row = logits + (long long)r * n_experts;
  unsigned taken = 0;  // bit c: this lane's expert lane + 64 c is already selected
  float first = 0.f, denom = 0.f, my_w = 0.f;
  int my_e = 0;
  for (int j = 0; j < top_k; ++j) {
    float best = -INFINITY;
    int best_e = 0x7fffffff;
    for (int e = lane, c = 0; e < n_experts; e += WAVE, ++c) {
      float v = row[e];
      if (!((taken >> c) & 1u) && (v > best || (v == best && e < best_e))) {
        best = v;
        best_e = e;
      }
    }
    for (int o = 32; o > 0; o >>= 1) {
      float ov = __shfl_xor(best, o, WAVE);
      int oe = __shfl_xor(best_e, o, WAVE);
      if (ov > best || (ov == best && oe < best_e)) {
        best = ov;
        best_e = oe;
      }
    }
    if ((best_e & 63) == lane) taken |= 1u << (best_e >> 6);
    if (j == 0) first = best;  // the largest selected logit
    float e_w = expf(best - first);
    denom += e_w;
    if (lane == j) {
      my_e = best_e;
      my_w = e_w;
    }
  }
  if (lane < top_k) {
    idx[(long long)r * top_k + lane] = my_e;
    wt[(long long)r * top_k + lane] = my_w / denom;
  }
}
void launch_moe_route(const float* router_logits, int* idx, float* wt, int rows, int n_experts, int top_k,
                      hipStream_t s) {
  if (rows) moe_route_kernel<<<rows, WAVE, 0, s>>>(router_logits, idx, wt, n_experts, top_k);
}

template <typename T>
__global__ void moe_gate_up_simple_kernel(const float* __restrict__ h, const T* __restrict__ w_gate_up,
                                          const int* __restrict__ idx, float* __restrict__ act, int hidden,
                                          int fe, int top_k) {
  int slot = blockIdx.y;  // (row, j)
  int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int f = blockIdx.x * 4 + wave;
  if (f >= fe) return;
  int e = idx[slot];
  const float* hv = h + (long long)(slot / top_k) * hidden;
  const T* wg = w_gate_up + ((long long)e * 2 * fe + f) * hidden;
  const T* wu = wg + (long long)fe * hidden;
  float ag = 0.f, au = 0.f;
  for (int k = lane; k < hidden; k += WAVE) {
    float x = hv[k];
    ag += x * to_f32(wg[k]);
    au += x * to_f32(wu[k]);
  }
  ag = wave_sum(ag);
  au = wave_sum(au);
  if (lane == 0) act[(long long)slot * fe + f] = ag / (1.0f + expf(-ag)) * au;
}
template <typename T>
void launch_moe_gate_up_simple(const float* h, const T* w_gate_up, const int* idx, float* act, int rows,
                               int top_k, int hidden, int expert_ffn, hipStream_t s) {
  if (rows)
    moe_gate_up_simple_kernel<T><<<dim3(ceil_div(expert_ffn, 4), rows * top_k), 256, 0, s>>>(
        h, w_gate_up, idx, act, hidden, expert_ffn, top_k);
}
template void launch_moe_gate_up_simple<float>(const float*, const float*, const int*, float*, int, int, int,
                                               int, hipStream_t);
template void launch_moe_gate_up_simple<bf16_t>(const float*, const bf16_t*, const int*, float*, int, int, int,
                                                int, hipStream_t);

template <typename T>
__global__ void moe_down_simple_kernel(const float* __restrict__ act, const T* __restrict__ w_down,
                                       const int* __restrict__ idx, const float* __restrict__ wt,
                                       float* __restrict__ x, int hidden, int fe, int top_k) {
  int r = blockIdx.y;
  int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int n = blockIdx.x * 4 + wave;
  if (n >= hidden) return;
  float total = 0.f;
  for (int j = 0; j < top_k; ++j) {
    int e = idx[(long long)r * top_k + j];
    const T* wd = w_down + ((long long)e * hidden + n) * fe;
    const float* a = act + ((long long)r * top_k + j) * fe;
    float acc = 0.f;
    for (int k = lane; k < fe; k += WAVE) acc += a[k] * to_f32(wd[k]);
    total += wt[(long long)r * top_k + j] * wave_sum(acc);
  }
  if (lane == 0) x[(long long)r * hidden + n] += total;
}
template <typename T>
void launch_moe_down_simple(const float* act, const T* w_down, const int* idx, const float* wt, float* x,
                            int rows, int top_k, int hidden, int expert_ffn, hipStream_t s) {
  if (rows)
    moe_down_simple_kernel<T><<<dim3(ceil_div(hidden, 4), rows), 256, 0, s>>>(act, w_down, idx, wt, x, hidden,
                                                                                expert_ffn, top_k);
}
template void launch_moe_down_simple<float>(const float*, const float*, const int*, const float*, float*, int,
                                            int, int, int, hipStream_t);
template void launch_moe_down_simple<bf16_t>(const float*, const bf16_t*, const int*, const float*, float*, int,
                                             int, int, int, hipStream_t);

// ---------------------------------------------------------------- page copy, conversions
__global__ void copy_pages_kernel(char* __restrict__ pool, const int* __restrict__ pairs,
                                  long long layer_stride, long long page_stride) {
  int pair = blockIdx.x, layer = blockIdx.y;
  const uint4* src = (const uint4*)(pool + layer * layer_stride + (long long)pairs[2 * pair] * page_stride);
  uint4* dst = (uint4*)(pool + layer * layer_stride + (long long)pairs[2 * pair + 1] * page_stride);
  for (long long i = threadIdx.x; i < page_stride / 16; i += blockDim.x) dst[i] = src[i];
}
void launch_copy_pages(void* kv_pool, const int* pairs, int n_pairs, int n_layers, long long layer_stride_bytes,
                       long long page_stride_bytes, hipStream_t s) {
  if (n_pairs)
    copy_pages_kernel<<<dim3(n_pairs, n_layers), 256, 0, s>>>((char*)kv_pool, pairs, layer_stride_bytes,
                                                               page_stride_bytes);
}

__global__ void convert_to_f32_kernel(const void* __restrict__ src, int is_bf16, float* __restrict__ dst,
                                      long long n) {
  long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = is_bf16 ? bf16_to_f32(((const bf16_t*)src)[i]) : ((const float*)src)[i];
}
void launch_convert_to_f32(const void* src, int dtype, float* dst, long long n, hipStream_t s) {
  if (n) convert_to_f32_kernel<<<ceil_div(n, 256), 256, 0, s>>>(src, dtype == 1, dst, n);
}

// ---------------------------------------------------------------- decode row plumbing
__global__ void gather_decode_rows_kernel(GatherRows a) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r < a.rows) gather_row(a, r, true);
}
void launch_gather_decode_rows(const GatherRows& a, hipStream_t s) {
  if (a.rows) gather_decode_rows_kernel<<<ceil_div(a.rows, 256), 256, 0, s>>>(a);
}

// ---------------------------------------------------------------- uploads
// One launch in place of a copy per array, each of which costs the stream 3 us and the host more; a
// call's arrays are a few kilobytes, and every word crosses the bus once, 64 of them to a read.
__global__ __launch_bounds__(256) void host_copies_kernel(HostCopies a) {
  const int* src = a.src[blockIdx.y];
  int* dst = a.dst[blockIdx.y];
  const int n = a.words[blockIdx.y];
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) dst[i] = src[i];
}
void launch_host_copies(const HostCopies& a, hipStream_t s) {
  if (!a.n) return;
  int most = 0;
  for (int i = 0; i < a.n; ++i) most = a.words[i] > most ? a.words[i] : most;
  host_copies_kernel<<<dim3(ceil_div(most, 256) < 64 ? ceil_div(most, 256) : 64, a.n), 256, 0, s>>>(a);
}
__global__ __launch_bounds__(64) void upload_page_rows_kernel(int* __restrict__ page_table, int max_pages,
                                                              const int* __restrict__ list,
                                                              const int* __restrict__ packed) {
  const int k = blockIdx.x;
  int* dst = page_table + (long long)list[2 * k] * max_pages;
  const int* src = packed + (long long)k * max_pages;
  for (int i = threadIdx.x, n = list[2 * k + 1]; i < n; i += 64) dst[i] = src[i];
}
void launch_upload_page_rows(int* page_table, int max_pages, const int* list, const int* packed, int n, hipStream_t s) {
  if (n) upload_page_rows_kernel<<<n, 64, 0, s>>>(page_table, max_pages, list, packed);
}

// ---------------------------------------------------------------- page-table patches
__global__ void patch_page_table_kernel(int* __restrict__ page_table, int max_pages, const int* __restrict__ triples,
                                        int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) page_table[(long long)triples[3 * i] * max_pages + triples[3 * i + 1]] = triples[3 * i + 2];
}
void launch_patch_page_table(int* page_table, int max_pages, const int* triples, int n, hipStream_t s) {
  if (n) patch_page_table_kernel<<<ceil_div(n, 256), 256, 0, s>>>(page_table, max_pages, triples, n);
}
