// Policy-gradient objective over packed rollouts: the training stage's consumer of the
// log-probs (paper sections 5.1 and 5.2: PPO loss on REINFORCE returns, rewards clipped at 20,
// advantages at 10; section 2.1: KL penalty from the reference model).  Definitions, token by
// token, in include/rollout.h.
//
// Two launches.  policy_count_kernel counts the tokens that count, N, over the packed mask (up to
// 512 integer partials), so that the second can write the gradient final, without a sweep to scale
// it.  policy_loss_kernel takes one sequence per workgroup.  The return G_j = rho_j + gamma G_{j+1}
// over the counted tokens is a first-order linear recurrence, so a chunk of the sequence, taken from
// its end, is a scan of affine maps y -> a y + b (a = gamma, b = rho for a counted token; the
// identity for any other): four tokens in a thread's registers, Hillis-Steele over a span of the
// wavefront's threads (all 64, see launch_policy_loss), the spans' totals composed through LDS, the
// chunk's last value carried to the next chunk.  Sums for the loss leave as one partial per sequence and are added in sequence order by
// the host, so the result does not depend on scheduling.
//
// What bounds it: memory latency of few, short chunks (a sequence's chunks are serial), so a chunk
// is 4096 tokens, loaded as 16-byte quads cut at multiples of four of the packed index, and only
// batches of short sequences take 256 threads.  512 sequences: see launch_policy_loss.
#include "kernels_fast.h"

struct Affine {
  float a, b;  // y -> a y + b
};
// apply `first`, then `second`
__device__ inline Affine then(const Affine& first, const Affine& second) {
  return Affine{second.a * first.a, second.a * first.b + second.b};
}

__device__ inline int nonzero_bytes(unsigned v) {
  return __popc((((v & 0x7f7f7f7fu) + 0x7f7f7f7fu) | v) & 0x80808080u);
}

// counted tokens of the workgroup's share of the mask; the call's cu_seqlens and rewards, which the
// host left in its own memory, are copied beside it for the second launch
__global__ __launch_bounds__(256) void policy_count_kernel(PolicyLossArgs p) {
  __shared__ int count_s[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const long long id = (long long)blockIdx.x * 256 + tid, n_threads = (long long)gridDim.x * 256;
  for (long long i = id; i <= p.n_seqs; i += n_threads) p.cu_seqlens[i] = p.host_cu[i];
  for (long long i = id; i < p.n_seqs; i += n_threads) p.rewards[i] = p.host_rewards[i];
  // 16-byte words between the first and the last aligned address; the edges byte by byte
  const long long head = min((long long)((16 - ((size_t)p.mask & 15)) & 15), p.total);
  const long long words = (p.total - head) >> 4, tail = head + (words << 4);
  const uint4* m = (const uint4*)(p.mask + head);
  int n = 0;
  for (long long w = id; w < words; w += n_threads) {
    const uint4 v = m[w];
    n += nonzero_bytes(v.x) + nonzero_bytes(v.y) + nonzero_bytes(v.z) + nonzero_bytes(v.w);
  }
  if (id < head) n += p.mask[id] != 0;
  if (id < p.total - tail) n += p.mask[tail + id] != 0;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o, WAVE);
  if (lane == 0) count_s[wave] = n;
  __syncthreads();
  if (tid == 0) p.part_count[blockIdx.x] = (count_s[0] + count_s[1]) + (count_s[2] + count_s[3]);
}

// four consecutive values from index t, a multiple of four when VEC (then base is 16-byte aligned); only
// those in [lo, hi) mean anything
template <bool VEC>
__device__ inline float4 load_quad(const float* base, long long t, long long lo, long long hi, long long total) {
  if (VEC && t >= 0 && t + 4 <= total) return *(const float4*)(base + t);
  float v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = t + e >= lo && t + e < hi ? base[t + e] : 0.f;
  return make_float4(v[0], v[1], v[2], v[3]);
}
template <bool VEC>
__device__ inline void store_quad(float* base, long long t, long long lo, long long hi, const float* v) {
  if (VEC && t >= lo && t + 4 <= hi) {
    *(float4*)(base + t) = make_float4(v[0], v[1], v[2], v[3]);
    return;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (t + e >= lo && t + e < hi) base[t + e] = v[e];
}

template <int T, bool VEC, int SPAN>
__global__ __launch_bounds__(T) void policy_loss_kernel(PolicyLossArgs p) {
  constexpr int NW = T / WAVE, NS = T / SPAN;
  __shared__ int count_s[NW], last_s[NW];
  __shared__ Affine total_s[NS];
  __shared__ float sum_s[NW];
  const int seq = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int span = tid / SPAN, at = tid % SPAN;
  const long long lo = p.cu_seqlens[seq], hi = p.cu_seqlens[seq + 1];
  const float reward = fminf(fmaxf(p.rewards[seq], -p.reward_clip), p.reward_clip);
  int n = 0;
  for (int i = tid; i < p.n_parts; i += T) n += p.part_count[i];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o, WAVE);
  if (lane == 0) count_s[wave] = n;
  float inv_n = 0.f, carry = 0.f, s_sum = 0.f;
  bool rewarded = false;  // the sequence's last counted token, met first, takes the clipped reward
  const long long end = VEC ? (hi + 3) & ~3ll : hi;
  for (long long top = end; top > lo; top -= 4 * T) {  // chunks from the end; thread 0 takes the latest tokens
    const long long t = top - 4 - 4ll * tid;
    float nw[4] = {}, old[4] = {}, ref[4] = {};
    unsigned counted = 0;  // bit e: token t + e
    if (t + 4 > lo) {
      const float4 a = load_quad<VEC>(p.logp_new, t, lo, hi, p.total), b = load_quad<VEC>(p.logp_old, t, lo, hi, p.total);
      nw[0] = a.x, nw[1] = a.y, nw[2] = a.z, nw[3] = a.w;
      old[0] = b.x, old[1] = b.y, old[2] = b.z, old[3] = b.w;
      if (p.logp_ref) {
        const float4 c = load_quad<VEC>(p.logp_ref, t, lo, hi, p.total);
        ref[0] = c.x, ref[1] = c.y, ref[2] = c.z, ref[3] = c.w;
      }
      unsigned char c4[4];
      if (VEC && t >= 0 && t + 4 <= p.total) {
        *(unsigned*)c4 = *(const unsigned*)(p.mask + t);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) c4[e] = t + e >= lo && t + e < hi ? p.mask[t + e] : 0;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (t + e >= lo && t + e < hi && c4[e]) counted |= 1u << e;
    }
    // position of the chunk's last counted token, and N from its partials in the first round
    int last = counted ? 4 * tid + __clz(counted) - 28 : 4 * T;
    if (!rewarded) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) last = min(last, __shfl_xor(last, o, WAVE));
      if (lane == 0) last_s[wave] = last;
      __syncthreads();
      last = last_s[0];
#pragma unroll 4
      for (int w = 1; w < NW; ++w) last = min(last, last_s[w]);
    }
    if (top == end) {
      n = 0;
#pragma unroll 4
      for (int w = 0; w < NW; ++w) n += count_s[w];
      inv_n = n > 0 ? (float)(1.0 / (double)n) : 0.f;
    }
    Affine m[4];  // of the tokens in walking order, the latest first
    Affine f{1.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = 3 - i;
      m[i] = Affine{1.f, 0.f};
      if (counted >> e & 1) {
        m[i].a = p.gamma;
        m[i].b = (p.logp_ref ? -p.kl_coef * (old[e] - ref[e]) : 0.f) + (!rewarded && 4 * tid + i == last ? reward : 0.f);
      }
      f = then(f, m[i]);
    }
    rewarded = rewarded || last < 4 * T;
    // inclusive scan over the threads: f becomes "everything from the span's first thread up to this one"
#pragma unroll
    for (int o = 1; o < SPAN; o <<= 1) {
      Affine prev{__shfl_up(f.a, o, WAVE), __shfl_up(f.b, o, WAVE)};
      if (at >= o) f = then(prev, f);
    }
    if (at == SPAN - 1) total_s[span] = f;
    __syncthreads();
    float y = carry;  // the value entering this span, then this thread; carry the one that leaves the chunk
#pragma unroll 4
    for (int w = 0; w < NS; ++w) {
      if (w == span) y = carry;
      carry = total_s[w].a * carry + total_s[w].b;
    }
    const float fa = __shfl_up(f.a, 1, WAVE), fb = __shfl_up(f.b, 1, WAVE);
    if (at > 0) y = fa * y + fb;
    if (t + 4 > lo) {
      float adv[4], grad[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int e = 3 - i;
        y = m[i].a * y + m[i].b;
        adv[e] = grad[e] = 0.f;
        if (counted >> e & 1) {
          adv[e] = fminf(fmaxf(y, -p.adv_clip), p.adv_clip);
          const float r = expf(nw[e] - old[e]);
          const float plain = r * adv[e], clipped = fminf(fmaxf(r, 1.f - p.eps_low), 1.f + p.eps_high) * adv[e];
          s_sum += fminf(plain, clipped);
          if (plain <= clipped) grad[e] = -plain * inv_n;
        }
      }
      if (p.advantages) store_quad<VEC>(p.advantages, t, lo, hi, adv);
      store_quad<VEC>(p.grad, t, lo, hi, grad);
    }
    __syncthreads();  // total_s and last_s are free again
  }
  s_sum = wave_sum(s_sum);
  if (lane == 0) sum_s[wave] = s_sum;
  __syncthreads();
  if (tid == 0) {
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) sum += sum_s[w];
    p.part_sum[seq] = sum;
    if (seq == 0) {
      n = 0;
#pragma unroll 4
      for (int w = 0; w < NW; ++w) n += count_s[w];
      *p.count = n;
    }
  }
}

// 256 threads where every sequence fits one of their chunks twice over; the quads need arrays
// aligned to 16 bytes (the mask to 4), any others are taken value by value.
// Spans of 64 threads hold 256 tokens.  With gamma above 1 the powers of gamma in a span's maps grow, and one that
// leaves fp32 makes inf x 0 of a return that is 0 (gamma 1.5 from 219 tokens on), so spans of 16
// threads, 64 tokens, then: finite up to gamma 4, and a longer walk over the spans' totals.
// 512 sequences of 512..8192 tokens, KL on: 5.2 us to count + 16.0 us (2.9 TB/s of the 47 MB it moves) where
// 256-token chunks, a reduction and a scaling pass took 60 us; the call 43 us, before 94 us.
template <int T, bool VEC>
static void launch_loss(const PolicyLossArgs& p, hipStream_t s) {
  if (p.gamma > 1.f) policy_loss_kernel<T, VEC, 16><<<p.n_seqs, T, 0, s>>>(p);
  else policy_loss_kernel<T, VEC, 64><<<p.n_seqs, T, 0, s>>>(p);
}
void launch_policy_loss(const PolicyLossArgs& p, int longest, hipStream_t s) {
  if (p.n_seqs == 0) return;
  policy_count_kernel<<<p.n_parts, 256, 0, s>>>(p);
  const size_t any = (size_t)p.logp_new | (size_t)p.logp_old | (size_t)p.logp_ref | (size_t)p.grad | (size_t)p.advantages;
  const bool vec = (any & 15) == 0 && ((size_t)p.mask & 3) == 0, small = longest <= 2048;
  if (vec) small ? launch_loss<256, true>(p, s) : launch_loss<1024, true>(p, s);
  else small ? launch_loss<256, false>(p, s) : launch_loss<1024, false>(p, s);
}
