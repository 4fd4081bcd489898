// Mixture-of-experts block of the matrix-core path: routing and the plan of the grouped
// expert projections.  The projections themselves are gemm_tile_kernel launches whose row
// blocks each belong to one expert (kernels_gemm.hip); the weighted sum of the experts'
// results rides in row_norm_kernel (kernels_rows.hip).
//
// Routing follows the usual top-k definition: the k largest router logits of a row, ties to
// the lower expert index; mixing weights are the softmax over those k logits.  Each pick gets
// a position inside its expert's list from an integer atomic counter: which pick gets which
// position depends on timing, but no result depends on the position - a slot's projection
// rows are computed independently and a row's picks are summed in pick order.
#include "kernels_fast.h"

#define MOE_MAX_PER_LANE 4  // n_experts <= 256

// order-preserving image of a float
__device__ inline unsigned float_order(float v) {
  const unsigned b = __float_as_uint(v);
  return b & 0x80000000u ? ~b : b | 0x80000000u;
}
// largest value of the wavefront, in every lane: lane shifts inside the rows of 16 and two row
// broadcasts, a few cycles each, where exchanges through LDS cost tens
template <int CTRL>
__device__ inline unsigned dpp_max(unsigned v) {
  return max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false));
}
__device__ inline unsigned wave_max_u32(unsigned v) {
  v = dpp_max<0x111>(v);  // row_shr:1, 2, 4, 8
  v = dpp_max<0x112>(v);
  v = dpp_max<0x114>(v);
  v = dpp_max<0x118>(v);
  v = dpp_max<0x142>(v);  // row_bcast:15, 31
  v = dpp_max<0x143>(v);
  return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}

// One wavefront per row.  The row's split planes are requested four at a time, for all of a lane's
// experts together; a pick is a maximum over the wavefront and a vote on who holds it.
// Up to 128 rows, 128 experts, 8 picks: 7.7 us, where planes added one by one and exchanges through LDS took 13.6.
__global__ __launch_bounds__(256) void moe_route_topk_kernel(MoeRouteArgs a) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= a.rows) return;
  float v[MOE_MAX_PER_LANE] = {};
  for (int z0 = 0; z0 < a.splits; z0 += 4) {  // planes added in ascending order
    float u[4][MOE_MAX_PER_LANE];
#pragma unroll
    for (int z = 0; z < 4; ++z)
#pragma unroll
      for (int q = 0; q < MOE_MAX_PER_LANE; ++q)
        u[z][q] = a.partial[(long long)min(z0 + z, a.splits - 1) * a.split_stride + (long long)r * a.n_experts +
                            min(lane + 64 * q, a.n_experts - 1)];
#pragma unroll
    for (int z = 0; z < 4; ++z)
#pragma unroll
      for (int q = 0; q < MOE_MAX_PER_LANE; ++q) v[q] += z0 + z < a.splits ? u[z][q] : 0.f;
  }
  unsigned key[MOE_MAX_PER_LANE];
  bool free_[MOE_MAX_PER_LANE];
#pragma unroll
  for (int q = 0; q < MOE_MAX_PER_LANE; ++q) {
    key[q] = float_order(v[q]);
    free_[q] = lane + 64 * q < a.n_experts;
  }
  float top = 0.f, denom = 0.f, my_w = 0.f;
  int my_e = 0;
  for (int j = 0; j < a.top_k; ++j) {
    unsigned best = 0;
#pragma unroll
    for (int q = 0; q < MOE_MAX_PER_LANE; ++q) best = max(best, free_[q] ? key[q] : 0u);
    best = wave_max_u32(best);
    int be = -1;  // the lowest index among those that hold it
#pragma unroll
    for (int q = 0; q < MOE_MAX_PER_LANE; ++q) {
      const unsigned long long holds = __ballot(free_[q] && key[q] == best);
      if (be < 0 && holds) be = __ffsll((long long)holds) - 1 + 64 * q;
    }
    const float bv = __uint_as_float(best & 0x80000000u ? best & 0x7fffffffu : ~best);
    if (j == 0) top = bv;
    const float w = expf(bv - top);
    denom += w;
#pragma unroll
    for (int q = 0; q < MOE_MAX_PER_LANE; ++q)
      if (be == lane + 64 * q) free_[q] = false;
    if (lane == j) {  // lane j keeps pick j (top_k <= 64)
      my_e = be;
      my_w = w;
    }
  }
  if (lane < a.top_k) {
    const long long o = (long long)r * a.top_k + lane;
    a.idx[o] = my_e;
    a.wt[o] = my_w / denom;
    a.pos[o] = atomicAdd(a.count + my_e, 1);
    if (a.route_log) a.route_log[o] = my_e;
  }
}
void launch_moe_route_topk(const MoeRouteArgs& a, hipStream_t s) {
  if (a.rows) moe_route_topk_kernel<<<ceil_div(a.rows, 4), 256, 0, s>>>(a);
}

// One workgroup: exclusive prefix of the expert counts and of the experts' row blocks (a wavefront's
// lanes hold four experts each), the row blocks of every expert, then the slot of every pick.  The
// picks of the first round are requested before all that.  Up to 1024 picks, 128 experts: 5.1 us, before 9.1 us with every thread
// adding up the counts before its own.
__global__ __launch_bounds__(1024) void moe_plan_kernel(MoePlanArgs a) {
  __shared__ int start[256], block0[257];
  const int t = threadIdx.x, picks = a.rows * a.top_k;
  const int shift = __ffs(a.block_rows) - 1;  // a power of two
  const int e_first = t < picks ? a.idx[t] : 0, p_first = t < picks ? a.pos[t] : 0;
  if (t < WAVE) {
    int n[4], s = 0, b = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c = a.count[min(4 * t + q, a.n_experts - 1)];
      n[q] = 4 * t + q < a.n_experts ? c : 0;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      s += n[q];
      b += (n[q] + a.block_rows - 1) >> shift;
    }
    int s_in = s, b_in = b;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
      const int us = __shfl_up(s_in, o, WAVE), ub = __shfl_up(b_in, o, WAVE);
      if (t >= o) s_in += us, b_in += ub;
    }
    if (t == WAVE - 1) block0[256] = b_in;  // experts past the last add nothing
    s_in -= s, b_in -= b;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      start[4 * t + q] = s_in;
      block0[4 * t + q] = b_in;
      for (int r0 = 0; r0 < n[q]; r0 += a.block_rows, ++b_in) {
        a.group_of_block[b_in] = 4 * t + q;
        a.block_row_begin[b_in] = s_in + r0;
        a.block_row_end[b_in] = s_in + min(n[q], r0 + a.block_rows);
      }
      s_in += n[q];
    }
  }
  __syncthreads();
  for (int b = block0[256] + t; b < a.max_blocks; b += 1024) {
    a.group_of_block[b] = 0;
    a.block_row_begin[b] = 0;
    a.block_row_end[b] = 0;
  }
  for (int i = t; i < picks; i += 1024) {
    const int slot = start[i == t ? e_first : a.idx[i]] + (i == t ? p_first : a.pos[i]);
    a.row_map[slot] = i / a.top_k;
    a.slot_of[i] = slot;
  }
}
void launch_moe_plan(const MoePlanArgs& a, hipStream_t s) {
  if (a.rows) moe_plan_kernel<<<1, 1024, 0, s>>>(a);
}
