// Fused per-row kernels of the matrix-core path: residual add + RMSNorm + bf16 cast (with
// optional embedding gather), and split-K reduction + rotary embedding + KV-page write.
// The residual stream stays fp32; only projection inputs and the KV cache are bf16.
#include <type_traits>

#include "kernels_fast.h"

// One workgroup of ROW_T threads per row; thread t holds the row's float4 chunks t, t + ROW_T, ... (V of them) in
// registers, so every load of the row is in flight before the first use (hidden <= 4 ROW_T V).
// What bounds it in a decode step: latency.  A launch has as many workgroups as rows, each makes a few round trips to
// memory, so as many threads as the row has chunks, and up to 16 split planes requested together (64 rows x 1536, 8 and 10
// planes: 5.5 -> 4.8 us; 64 x 3584, 8 planes 6.9 -> 5.8; both with 2 us of launch).  With more rows than the chip
// holds at once it is the bytes, and small workgroups that come and go keep more of them in flight.
template <int ROW_T, int V>
__global__ __launch_bounds__(ROW_T) void row_norm_kernel(float* x_rows, const float* partial_rows, const float* gain, long long split_stride,
                                                         const int* tokens, int hidden, int splits, int moe_k, RowNormArgs a) {
  a.x = x_rows;
  a.partial = partial_rows;
  a.gain = gain;
  a.split_stride = split_stride;
  a.tokens = tokens;
  a.hidden = hidden;
  a.splits = splits;
  a.moe_k = moe_k;
  __shared__ float partial[ROW_T / WAVE];
  const int r = blockIdx.x, t = threadIdx.x;
  const int n4 = a.hidden >> 2;
  const long long src_row = a.rows_index ? a.rows_index[r] : r;
  float4 x[V];
  if (a.tokens) {
    const uint2* e = (const uint2*)(a.embed + (long long)(a.gather.rows ? gather_row(a.gather, r, t == 0) : a.tokens[r]) * a.hidden);
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const int c = t + ROW_T * v;
      uint2 u = make_uint2(0, 0);
      if (c < n4) u = e[c];
      x[v] = make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16),
                         __uint_as_float(u.y & 0xffff0000u));
    }
  } else {
    const float4* xs = (const float4*)(a.x + src_row * a.hidden);
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const int c = t + ROW_T * v;
      x[v] = c < n4 ? xs[c] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
  // the gain is not needed before the end: requested now, it arrives with the row
  float4 gn[V];
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const int c = t + ROW_T * v;
    gn[v] = c < n4 ? ((const float4*)a.gain)[c] : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  // split planes, added in ascending order; the loads of a batch of planes are issued together (a projection with a
  // deep K leaves up to 16 planes)
  auto add_planes = [&](auto batch) {
    constexpr int Z = decltype(batch)::value;
    for (int z = 0; z < a.splits; z += Z) {
      float4 u[Z][V];
#pragma unroll
      for (int q = 0; q < Z; ++q) {
        const float4* pz = (const float4*)(a.partial + (long long)(z + q) * a.split_stride + (long long)r * a.hidden);
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const int c = t + ROW_T * v;
          u[q][v] = (z + q < a.splits && c < n4) ? pz[c] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
      }
#pragma unroll
      for (int q = 0; q < Z; ++q)
#pragma unroll
        for (int v = 0; v < V; ++v) {
          x[v].x += u[q][v].x;
          x[v].y += u[q][v].y;
          x[v].z += u[q][v].z;
          x[v].w += u[q][v].w;
        }
    }
  };
  constexpr int MOST = V == 1 ? 16 : 4;
  if (a.splits <= 4) add_planes(std::integral_constant<int, 4>{});
  else if (a.splits <= 8) add_planes(std::integral_constant<int, MOST < 8 ? MOST : 8>{});
  else add_planes(std::integral_constant<int, MOST>{});
  // the row's expert picks, in pick order: slots and weights of a batch first, then all its rows at once
  constexpr int MB = V <= 2 ? 8 : 4;
  for (int j0 = 0; j0 < a.moe_k; j0 += MB) {
    int slot[MB];
    float wt[MB];
#pragma unroll
    for (int j = 0; j < MB; ++j) {
      const long long at = (long long)r * a.moe_k + min(j0 + j, a.moe_k - 1);
      slot[j] = a.moe_slot[at];
      wt[j] = a.moe_wt[at];
    }
    float4 y[MB][V];
#pragma unroll
    for (int j = 0; j < MB; ++j)
#pragma unroll
      for (int v = 0; v < V; ++v)
        y[j][v] = ((const float4*)(a.moe_y + (long long)slot[j] * a.hidden))[min(t + ROW_T * v, n4 - 1)];
#pragma unroll
    for (int j = 0; j < MB; ++j) {
      if (j0 + j >= a.moe_k) break;
#pragma unroll
      for (int v = 0; v < V; ++v) {
        if (t + ROW_T * v >= n4) continue;
        x[v].x += wt[j] * y[j][v].x;
        x[v].y += wt[j] * y[j][v].y;
        x[v].z += wt[j] * y[j][v].z;
        x[v].w += wt[j] * y[j][v].w;
      }
    }
  }
  float ss = 0.f;
#pragma unroll
  for (int v = 0; v < V; ++v) ss += x[v].x * x[v].x + x[v].y * x[v].y + x[v].z * x[v].z + x[v].w * x[v].w;
  ss = wave_sum(ss);
  if ((t & 63) == 0) partial[t >> 6] = ss;
  __syncthreads();
  float total = 0.f;
#pragma unroll
  for (int w = 0; w < ROW_T / WAVE; ++w) total += partial[w];
  const float rinv = a.ssq_out ? 1.0f : 1.0f / sqrtf(total / (float)a.hidden + a.eps);
  if (a.ssq_out && t == 0) a.ssq_out[r] = total;
  const bool write_x = !a.rows_index && (a.splits || a.tokens || a.moe_k);
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const int c = t + ROW_T * v;
    if (c >= n4) continue;
    if (write_x) ((float4*)(a.x + (long long)r * a.hidden))[c] = x[v];
    uint2 hi, lo;
    split4_bf16(x[v].x * gn[v].x * rinv, x[v].y * gn[v].y * rinv, x[v].z * gn[v].z * rinv, x[v].w * gn[v].w * rinv, hi, lo);
    uint16_t* hp = a.h + (a.h_frag ? frag_offset(r, 4 * c, a.hidden >> 5) : plane_offset(r, 4 * c, a.hidden));
    *(uint2*)hp = hi;
    *(uint2*)(hp + a.h_lo_offset) = lo;
  }
}
#define ROW_ARGS a.x, a.partial, a.gain, a.split_stride, a.tokens, a.hidden, a.splits, a.moe_k, a
void launch_row_norm(const RowNormArgs& a, hipStream_t s) {
  if (!a.rows) return;
  const int n4 = a.hidden >> 2;  // hidden is a multiple of 32 and at most 8192
  // A thread per chunk where the chip's 512 Ki threads hold all rows at once; 256 threads beyond that (10568 rows x
  // 3584: 134 us with 1024 threads to a row, 94 with 256) and where a row has no more chunks.
  const bool at_once = (long long)a.rows * n4 <= 512 * 1024;
  if (n4 <= 256) row_norm_kernel<256, 1><<<a.rows, 256, 0, s>>>(ROW_ARGS);
  else if (n4 <= 512 && at_once) row_norm_kernel<512, 1><<<a.rows, 512, 0, s>>>(ROW_ARGS);
  else if (n4 <= 512) row_norm_kernel<256, 2><<<a.rows, 256, 0, s>>>(ROW_ARGS);
  else if (n4 <= 1024 && at_once) row_norm_kernel<1024, 1><<<a.rows, 1024, 0, s>>>(ROW_ARGS);
  else if (n4 <= 1024) row_norm_kernel<256, 4><<<a.rows, 256, 0, s>>>(ROW_ARGS);
  else row_norm_kernel<256, 8><<<a.rows, 256, 0, s>>>(ROW_ARGS);
}

// One thread per rotary pair (head, i): grid (rows, heads / 4), 4 heads of 64 pairs per block.
__global__ __launch_bounds__(256) void qkv_post_kernel(QkvPostArgs a) {
  const int r = blockIdx.x;
  const KvGeom& g = a.geom;
  const int dh = g.head_dim, half = dh >> 1;
  const int n_heads = a.n_q_heads + 2 * g.n_kv_heads;
  const int per_block = 256 / half;  // heads per block
  const int head = blockIdx.y * per_block + threadIdx.x / half, i = threadIdx.x % half;
  if (head >= n_heads) return;
  const int pos = a.row_pos[r];
  const long long row_off = (long long)r * n_heads * dh + head * dh;
  const float* p = a.partial + row_off;
  float u = 0.f, w = 0.f;
  for (int z = 0; z < a.splits; z += 4) {  // four planes at a time, loads issued together
    const float* q = p + (long long)z * a.split_stride;
    float u0 = q[i], w0 = q[i + half], u1 = 0.f, u2 = 0.f, u3 = 0.f, w1 = 0.f, w2 = 0.f, w3 = 0.f;
    if (z + 1 < a.splits) { u1 = q[a.split_stride + i]; w1 = q[a.split_stride + i + half]; }
    if (z + 2 < a.splits) { u2 = q[2 * a.split_stride + i]; w2 = q[2 * a.split_stride + i + half]; }
    if (z + 3 < a.splits) { u3 = q[3 * a.split_stride + i]; w3 = q[3 * a.split_stride + i + half]; }
    u = (((u + u0) + u1) + u2) + u3;
    w = (((w + w0) + w1) + w2) + w3;
  }
  // bias and per-head norm: this launch runs with head_dim 128, a wavefront per head
  if (a.extra.bias || a.extra.q_gain)
    qkv_extras(a.extra, head * dh, i,
               head < a.n_q_heads ? a.extra.q_gain : head < a.n_q_heads + g.n_kv_heads ? a.extra.k_gain : nullptr, u, w);
  if (head < a.n_q_heads + g.n_kv_heads) {
    const float* cs = a.cos_sin + (long long)pos * dh;
    float c = cs[2 * i], sn = cs[2 * i + 1];
    float ru = u * c - w * sn, rw = w * c + u * sn;
    u = ru;
    w = rw;
  }
  if (head < a.n_q_heads) {
    long long o = ((long long)r * a.n_q_heads + head) * dh;
    uint16_t hi, lo;  // the attention kernels multiply q with half-precision keys
    split_f16(u, hi, lo);
    a.q_bf16[o + i] = hi;
    a.q_bf16[a.q_lo_offset + o + i] = lo;
    split_f16(w, hi, lo);
    a.q_bf16[o + i + half] = hi;
    a.q_bf16[a.q_lo_offset + o + i + half] = lo;
    if (a.q_f32) {
      a.q_f32[(long long)r * a.q_f32_ld + head * dh + i] = u;
      a.q_f32[(long long)r * a.q_f32_ld + head * dh + i + half] = w;
    }
  } else {
    const int page = a.page_table[(long long)a.row_slot[r] * a.max_pages + pos / g.page_tokens];
    const int tok = pos % g.page_tokens;
    int is_v = head >= a.n_q_heads + g.n_kv_heads;
    int kvh = head - a.n_q_heads - (is_v ? g.n_kv_heads : 0);
    uint16_t* dst = a.kv_pool + kv_block_base(g, a.layer, page, kvh, is_v);
    if (is_v) {
      dst[kv_v_offset(g, tok, i)] = f32_to_f16(u).bits;
      dst[kv_v_offset(g, tok, i + half)] = f32_to_f16(w).bits;
    } else {
      dst[kv_k_offset(g, tok, i)] = f32_to_f16(u).bits;
      dst[kv_k_offset(g, tok, i + half)] = f32_to_f16(w).bits;
    }
  }
}
void launch_qkv_post(const QkvPostArgs& a, hipStream_t s) {
  if (!a.rows) return;
  const int per_block = 256 / (a.geom.head_dim / 2);
  const int n_heads = a.n_q_heads + 2 * a.geom.n_kv_heads;
  qkv_post_kernel<<<dim3(a.rows, ceil_div(n_heads, per_block)), 256, 0, s>>>(a);
}
