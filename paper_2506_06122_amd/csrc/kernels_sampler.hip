// Temperature / top-p sampling over the full vocabulary on integer weights, the
// Philox4x32-10 generator that drives it, and the log-prob gather of the teacher-forced
// pass.  The paper leaves the sampler to its serving engines (section 2.1: the actor
// generates tokens until the termination criteria are met); the integer procedure below
// exists so that a drawn token id is one exact function of (logits row, temperature,
// top-p, 32-bit word) whatever the reduction order:
//   z = logit * inv_T; d = z - max z; w = floor(P(frac(t)) * 2^(40 + floor(t))), t = d*log2(e),
//   w = 0 for t < -40; S = sum w; nucleus = shortest prefix in (w desc, id asc) order whose
//   weight reaches theta = max(1, floor(S * floor(top_p 2^24) / 2^24)); R = floor(S_N x / 2^32);
//   token = first id of the nucleus, ascending, whose running weight exceeds R.
// Every floating-point step is a single rounded fp32 operation: no contraction allowed.
//
// Where the nucleus ends (top_p < 1): the smallest weight tau it holds is found by three histograms
// of weight over the vocabulary instead of one sweep per bit of the weight.  A weight has at most 24
// significant bits, so as a float it is exact and its bits order like its value: 6 bits of
// exponent and 23 of mantissa.  Histogram 0 bins by exponent and 4 mantissa bits (656 bins), the next
// two by the following 10 and the last 9 bits among the ids of the bin found before; a bin is
// found from the top by a prefix sum.  A fifth sweep leaves, per segment of 256 ids, the weight
// above tau and the number of ids at tau, from which the draw needs no further sweep.  What bounds it:
// the arithmetic of the weights (about 60 instructions per id and sweep), so the sweeps of a row
// run on several workgroups, like the first two.  64 rows x 151936 ids, top_p 0.9: see launch_sample.
#include <algorithm>

#include "kernels.h"

#pragma clang fp contract(off)

#define SAMP_T 1024

// P(frac(t)) of t = d * log2(e), as bits; n = floor(t).  false: the weight is 0.
__device__ inline bool fixexp_bits(float d, unsigned& bits, int& n_out) {
#pragma clang fp contract(off)
  const float log2e = 0x1.715476p+0f;
  float t = d * log2e;
  if (!(t >= -40.0f)) return false;
  float n = floorf(t);
  float f = t - n;
  float y = 0x1.5bd2aep-16f;
  y = y * f;
  y = y + 0x1.3262dep-13f;
  y = y * f;
  y = y + 0x1.5efc6ap-10f;
  y = y * f;
  y = y + 0x1.3b1a32p-7f;
  y = y * f;
  y = y + 0x1.c6b140p-5f;
  y = y * f;
  y = y + 0x1.ebfbdep-3f;
  y = y * f;
  y = y + 0x1.62e430p-1f;
  y = y * f;
  y = y + 0x1.000000p+0f;
  bits = __float_as_uint(y);
  n_out = (int)n;
  return true;
}
// The weight as the bits of a float, exact (24 significant bits at most); 0 for weight 0.
__device__ inline unsigned fixexp_key(float d) {
  unsigned bits;
  int n;
  if (!fixexp_bits(d, bits, n)) return 0u;
  // floor(y * 2^(40 + n)): the exponent grows by 40 + n, mantissa bits worth less than 1 go
  const int e = (int)((bits >> 23) & 0xffu) - 127 + 40 + n;
  if (e < 0) return 0u;
  const unsigned below_one = e < 23 ? (1u << (23 - e)) - 1u : 0u;
  return (((unsigned)(e + 127) << 23) | (bits & 0x7fffffu)) & ~below_one;
}
__device__ inline unsigned long long key_weight(unsigned key) {
  if (!key) return 0ull;
  const int e = (int)(key >> 23) - 127;
  const unsigned mant = (key & 0x7fffffu) | 0x800000u;
  return e >= 23 ? (unsigned long long)mant << (e - 23) : (unsigned long long)(mant >> (23 - e));
}

// The weight itself, for the sweeps that only add weights up.
__device__ inline unsigned long long fixexp_weight(float d) {
  unsigned bits;
  int n;
  if (!fixexp_bits(d, bits, n)) return 0ull;
  // y's 24 bits times 2^(e + 40 + n - 23), at most 2^17 (d <= 0): one 64-bit shift, to the right
  const int e = (int)((bits >> 23) & 0xffu) - 127;
  return ((unsigned long long)((bits & 0x7fffffu) | 0x800000u) << 17) >> (-e - n);
}

__device__ inline float scaled_logit(float logit, float inv_t) {
#pragma clang fp contract(off)
  return logit * inv_t;
}
__device__ inline float shifted(float z, float m) {
#pragma clang fp contract(off)
  return z - m;
}

// Inclusive prefix sum over a wavefront whose lanes are all active, in registers: DPP row shifts by 1, 2,
// 4, 8, then lane 15 of a row into rows 1 and 3 and lane 31 into rows 2 and 3.
template <int CTRL, int ROWS>
__device__ inline unsigned long long dpp_add_u64(unsigned long long v) {
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)v, CTRL, ROWS, 0xf, false);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(v >> 32), CTRL, ROWS, 0xf, false);
  return v + (((unsigned long long)hi << 32) | lo);
}
__device__ inline unsigned long long wave_scan_u64(unsigned long long v) {
  v = dpp_add_u64<0x111, 0xf>(v);
  v = dpp_add_u64<0x112, 0xf>(v);
  v = dpp_add_u64<0x114, 0xf>(v);
  v = dpp_add_u64<0x118, 0xf>(v);
  v = dpp_add_u64<0x142, 0xa>(v);
  return dpp_add_u64<0x143, 0xc>(v);
}
__device__ inline unsigned long long wave_total_u64(unsigned long long v) {
  v = wave_scan_u64(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, 63);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), 63);
  return ((unsigned long long)hi << 32) | lo;
}

// Sum over the wavefront of values below 2^43 (the weights of four ids), in every lane: as two sums of 32 bits,
// whose steps are one instruction each.
__device__ inline unsigned wave_total_u32(unsigned v) {
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);
  return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ inline unsigned long long wave_total_weights(unsigned long long v) {
  const unsigned lo = wave_total_u32((unsigned)v & 0x3fffffu), hi = wave_total_u32((unsigned)(v >> 22));
  return ((unsigned long long)hi << 22) + lo;
}

struct SampShared {
  unsigned long long vals[SAMP_T];   // one value per segment
  unsigned long long hist[SAMP_T];   // a histogram, or the nucleus' weight above tau per segment
  unsigned ties[SAMP_T];             // ids at tau per segment
  unsigned long long wave_part[SAMP_T / WAVE];
  unsigned long long bcast[2];
  float fwave[SAMP_T / WAVE];
};

__device__ inline float block_max(float v, SampShared& sh) {
  v = wave_max(v);
  if ((threadIdx.x & 63) == 0) sh.fwave[threadIdx.x >> 6] = v;
  __syncthreads();
  float m = sh.fwave[0];
  for (int i = 1; i < SAMP_T / WAVE; ++i) m = fmaxf(m, sh.fwave[i]);
  __syncthreads();
  return m;
}

__device__ inline unsigned long long block_sum_u64(unsigned long long v, SampShared& sh) {
  v = wave_total_u64(v);
  if ((threadIdx.x & 63) == 0) sh.wave_part[threadIdx.x >> 6] = v;
  __syncthreads();
  unsigned long long s = 0;
  for (int i = 0; i < SAMP_T / WAVE; ++i) s += sh.wave_part[i];
  __syncthreads();
  return s;
}

// Inclusive prefix sum over the threads of the workgroup.
__device__ inline unsigned long long block_scan_u64(unsigned long long v, SampShared& sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  v = wave_scan_u64(v);
  if (lane == 63) sh.wave_part[wave] = v;
  __syncthreads();
  for (int w = 0; w < wave; ++w) v += sh.wave_part[w];
  __syncthreads();
  return v;
}

__device__ inline void philox_round(unsigned& c0, unsigned& c1, unsigned& c2, unsigned& c3, unsigned k0,
                                    unsigned k1) {
  const unsigned MA = 0xD2511F53u, MB = 0xCD9E8D57u;
  unsigned hi0 = __umulhi(MA, c0), lo0 = MA * c0;
  unsigned hi1 = __umulhi(MB, c2), lo1 = MB * c2;
  unsigned n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
  c0 = n0;
  c1 = lo1;
  c2 = n2;
  c3 = lo0;
}
// Philox4x32-10 (Salmon et al., SC'11), output word 0.
__device__ inline unsigned philox_word0(unsigned long long seed, unsigned long long sample_id, unsigned step) {
  unsigned k0 = (unsigned)seed, k1 = (unsigned)(seed >> 32);
  unsigned c0 = (unsigned)sample_id, c1 = (unsigned)(sample_id >> 32), c2 = step, c3 = 0u;
  for (int r = 0; r < 10; ++r) {
    philox_round(c0, c1, c2, c3, k0, k1);
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return c0;
}

__global__ void philox_words_kernel(unsigned long long seed, const long long* __restrict__ ids,
                                    const unsigned* __restrict__ steps, unsigned* __restrict__ out, int n) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = philox_word0(seed, (unsigned long long)ids[i], steps[i]);
}
void launch_philox_words(unsigned long long seed, const long long* ids, const unsigned* steps, unsigned* out,
                         int n, hipStream_t s) {
  if (n) philox_words_kernel<<<ceil_div(n, 256), 256, 0, s>>>(seed, ids, steps, out, n);
}

// The vocabulary is walked in segments of 256 consecutive ids: one wavefront, 4 ids per lane,
// 16 segments per 4096-id tile of the block.  Every pass is a coalesced sweep that leaves one
// value per segment in LDS; a prefix search over at most 1024 segment values then names the
// segment that holds the id in question, and one wavefront resolves it inside the segment.
struct Seg4 {
  unsigned long long w[4];
};
struct Key4 {
  unsigned k[4];
};

struct Logit4 {
  float v[4];
};

// logits of ids i0 .. i0 + 3, -inf past the end
__device__ inline Logit4 load_logits4(const float* __restrict__ row, int i0, int vocab, bool vec_ok) {
  Logit4 out = {{-INFINITY, -INFINITY, -INFINITY, -INFINITY}};
  float(&v)[4] = out.v;
  if (vec_ok && i0 + 3 < vocab) {
    const float4 t = *(const float4*)(row + i0);
    v[0] = t.x;
    v[1] = t.y;
    v[2] = t.z;
    v[3] = t.w;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (i0 + e < vocab) v[e] = row[i0 + e];
  }
  return out;
}
__device__ inline Key4 load_keys4(const float* __restrict__ row, int i0, int vocab, bool vec_ok, float inv_t, float m) {
  const Logit4 z = load_logits4(row, i0, vocab, vec_ok);
  Key4 out;
#pragma unroll
  for (int e = 0; e < 4; ++e) out.k[e] = i0 + e < vocab ? fixexp_key(shifted(scaled_logit(z.v[e], inv_t), m)) : 0u;
  return out;
}
__device__ inline Seg4 load_weights4(const float* __restrict__ row, int i0, int vocab, bool vec_ok, float inv_t,
                                     float m) {
  const Logit4 z = load_logits4(row, i0, vocab, vec_ok);
  Seg4 out;
#pragma unroll
  for (int e = 0; e < 4; ++e) out.w[e] = i0 + e < vocab ? fixexp_weight(shifted(scaled_logit(z.v[e], inv_t), m)) : 0ull;
  return out;
}

__device__ inline float row_inv_temp(const SampleRows& a, int r) { return a.inv_temp ? a.inv_temp[r] : a.inv_temp_all; }
__device__ inline float row_top_p(const SampleRows& a, int r) { return a.top_p ? a.top_p[r] : a.top_p_all; }

// ---- the end of the nucleus
// Row r draws from a nucleus (a forced token or top_p >= 1 does not).
__device__ inline bool row_has_nucleus(const SampleRows& a, int r, int vocab) {
  return row_top_p(a, r) < 1.0f && !(a.forced && (unsigned)a.forced[r] < (unsigned)vocab);
}
// bin of a key in histogram `level`; the bits above it name the bins of the levels before
__device__ inline unsigned nucleus_prefix(unsigned key, int level) { return level == 0 ? 0u : key >> (level == 1 ? 19 : 9); }
__device__ inline unsigned nucleus_bin(unsigned key, int level) {
  return level == 0 ? (key >> 19) - (127u << 4) : level == 1 ? (key >> 9) & 1023u : key & 511u;
}
__device__ inline int nucleus_bins(int level) { return level == 0 ? kNucleusBins0 : level == 1 ? 1024 : 512; }

struct NucleusState {
  unsigned long long theta, above;  // weight to reach; weight of the bins above the ones found
  unsigned prefix;                  // key bits found so far (nucleus_prefix of the next level; the key of tau after level 2)
};
// One more level: hist (n bins) names the highest bin at which the weight from the top reaches theta.
__device__ inline void nucleus_descend(const unsigned long long* hist, int level, NucleusState& st, SampShared& sh) {
  const int n = nucleus_bins(level), t = threadIdx.x;
  if (t == 0) sh.bcast[0] = sh.bcast[1] = 0ull;  // a row without weights (no finite maximum) finds no bin
  const unsigned long long v = t < n ? hist[n - 1 - t] : 0ull;
  const unsigned long long inc = block_scan_u64(v, sh) + st.above;
  if (t < n && inc >= st.theta && inc - v < st.theta) {  // exactly one thread: the sums only grow, and all of them reach theta
    sh.bcast[0] = (unsigned long long)(n - 1 - t);
    sh.bcast[1] = inc - v;
  }
  __syncthreads();
  const unsigned bin = (unsigned)sh.bcast[0];
  st.above = sh.bcast[1];
  st.prefix = level == 0 ? bin + (127u << 4) : level == 1 ? (st.prefix << 10) | bin : (st.prefix << 9) | bin;
  __syncthreads();
}
__device__ inline unsigned long long nucleus_theta(unsigned long long S, float top_p) {
  const unsigned long long p24 = (unsigned long long)floorf(fmaxf(top_p, 0.f) * 16777216.0f);
  const unsigned long long theta = (S >> 24) * p24 + (((S & 0xffffffull) * p24) >> 24);
  return theta < 1 ? 1 : theta;
}
// State after the first `levels` histograms of row r (global scratch); S = sum of all weights.
__device__ inline NucleusState nucleus_from_scratch(const SampleRows& a, int r, int levels, unsigned long long& S,
                                                    SampShared& sh) {
  const unsigned long long* h = a.nucleus + (long long)r * kNucleusScratch;
  S = block_sum_u64(threadIdx.x < kNucleusBins0 ? h[threadIdx.x] : 0ull, sh);
  NucleusState st{nucleus_theta(S, row_top_p(a, r)), 0ull, 0u};
  nucleus_descend(h, 0, st, sh);
  if (levels > 1) nucleus_descend(h + kNucleusBins0, 1, st, sh);
  if (levels > 2) nucleus_descend(h + kNucleusBins0 + 1024, 2, st, sh);
  return st;
}
// Tiles t0, t0 + step, ... of the row into the LDS histogram of `level` (zeroed here).  From level 1 on only the ids
// of one narrow bin count, so an id whose exponent t lies outside the bin's range is passed over before its
// weight is computed: a weight w in the bin [lo, hi) comes from a value in [w, w + 1) that is 2^(40 + t) within
// a few 2^-23, so t + 40 lies between log2(lo) and log2(hi + 1), each widened by 0.01.
__device__ inline void nucleus_histogram(const float* row, int vocab, bool vec_ok, float inv_t, float m, int t0, int step,
                                         int level, unsigned prefix, SampShared& sh) {
  const int tid = threadIdx.x, n_tiles = (vocab + 4095) >> 12;
  sh.hist[tid] = 0ull;
  __syncthreads();
  float t_lo = 0.f, t_hi = 0.f;
  if (level > 0) {
    const int shift = level == 1 ? 19 : 9;
    t_lo = log2f(__uint_as_float(prefix << shift)) - 40.01f;
    t_hi = log2f(__uint_as_float((prefix + 1u) << shift) + 1.f) - 39.99f;
  }
  for (int t = t0; t < n_tiles; t += step) {
    if (level > 0) {
      const Logit4 z = load_logits4(row, t * 4096 + tid * 4, vocab, vec_ok);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float d = shifted(scaled_logit(z.v[e], inv_t), m), x = d * 0x1.715476p+0f;
        if (x >= t_lo && x <= t_hi) {  // (not so where d is no number)
          const unsigned key = fixexp_key(d);
          if (key && nucleus_prefix(key, level) == prefix) atomicAdd(&sh.hist[nucleus_bin(key, level)], key_weight(key));
        }
      }
      continue;
    }
    const Key4 q = load_keys4(row, t * 4096 + tid * 4, vocab, vec_ok, inv_t, m);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (q.k[e]) atomicAdd(&sh.hist[nucleus_bin(q.k[e], level)], key_weight(q.k[e]));
  }
  __syncthreads();
}
// Tiles t0, t0 + step, ...: per segment the weight above tau and the number of ids at tau
template <typename F>
__device__ inline void nucleus_segments(const float* row, int vocab, bool vec_ok, float inv_t, float m, int t0, int step,
                                        unsigned tau_key, F&& put) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n_tiles = (vocab + 4095) >> 12, n_seg = (vocab + 255) >> 8;
  for (int t = t0; t < n_tiles; t += step) {
    const Key4 q = load_keys4(row, t * 4096 + tid * 4, vocab, vec_ok, inv_t, m);
    unsigned long long v = 0;  // the weight (at most 256 x 2^40 per segment), the count from bit 52 on
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (q.k[e] > tau_key) v += key_weight(q.k[e]);
      if (q.k[e] == tau_key) v += 1ull << 52;
    }
    v = wave_total_u64(v);
    if (lane == 0 && t * 16 + wave < n_seg) put(t * 16 + wave, v & ((1ull << 52) - 1ull), (unsigned)(v >> 52));
  }
}

// Smallest segment whose inclusive prefix of sh.vals[0..n_seg) exceeds target, and the
// exclusive prefix before it.  Requires the total to exceed target.
__device__ inline void find_segment(SampShared& sh, int n_seg, unsigned long long target, int& seg,
                                    unsigned long long& before) {
  const int tid = threadIdx.x;
  if (tid == 0) {
    sh.bcast[0] = 0;
    sh.bcast[1] = 0;
  }
  __syncthreads();
  if (tid < WAVE) {
    const int per = SAMP_T / WAVE;
    unsigned long long mine = 0;
    for (int j = 0; j < per; ++j) mine += tid * per + j < n_seg ? sh.vals[tid * per + j] : 0ull;
    const unsigned long long inc = wave_scan_u64(mine);
    unsigned long long exc = inc - mine;
    if (exc <= target && target < inc) {
      unsigned long long acc = exc;
      int j = 0;
      for (; j < per - 1; ++j) {
        unsigned long long v = tid * per + j < n_seg ? sh.vals[tid * per + j] : 0ull;
        if (acc + v > target) break;
        acc += v;
      }
      sh.bcast[0] = (unsigned long long)(tid * per + j);
      sh.bcast[1] = acc;
    }
  }
  __syncthreads();
  seg = (int)sh.bcast[0];
  before = sh.bcast[1];
  __syncthreads();
}

// One wavefront: index of the element of its 4-per-lane values whose running sum first exceeds
// target (values in ascending id order: lane-major, element-minor).
__device__ inline int resolve_in_segment(const unsigned long long (&v)[4], unsigned long long target, int lane) {
  const unsigned long long mine = v[0] + v[1] + v[2] + v[3];
  const unsigned long long inc = wave_scan_u64(mine);
  const unsigned long long exc = inc - mine;
  int found = -1;
  if (exc <= target && target < inc) {
    unsigned long long acc = exc;
    found = lane * 4 + 3;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      acc += v[e];
      if (acc > target && found == lane * 4 + 3) found = lane * 4 + e;
    }
  }
  // exactly one lane found it
  for (int o = WAVE / 2; o > 0; o >>= 1) found = max(found, __shfl_xor(found, o, WAVE));
  return found;
}

// First sweep on `parts` workgroups per row: maximum of the scaled logits over tiles
// blockIdx.x, blockIdx.x + parts, ...
__global__ __launch_bounds__(SAMP_T) void sample_max_kernel(SampleRows a, int vocab, int parts) {
  __shared__ SampShared sh;
  const int tid = threadIdx.x, r = blockIdx.y;
  const float* row = a.logits + (long long)(a.logits_row ? a.logits_row[r] : r) * vocab;
  const float inv_t = row_inv_temp(a, r);
  const bool vec_ok = (vocab & 3) == 0 && (((unsigned long long)row) & 15ull) == 0;
  const int n_tiles = (vocab + 4095) >> 12;
  float m = -INFINITY;
  for (int t = blockIdx.x; t < n_tiles; t += parts) {
    const int i0 = t * 4096 + tid * 4;
    if (vec_ok && i0 + 3 < vocab) {
      const float4 v = *(const float4*)(row + i0);
      m = fmaxf(fmaxf(m, fmaxf(scaled_logit(v.x, inv_t), scaled_logit(v.y, inv_t))),
                fmaxf(scaled_logit(v.z, inv_t), scaled_logit(v.w, inv_t)));
    } else {
      for (int e = 0; e < 4; ++e)
        if (i0 + e < vocab) m = fmaxf(m, scaled_logit(row[i0 + e], inv_t));
    }
  }
  m = block_max(m, sh);
  if (tid == 0) a.part_max[(long long)r * kSampleParts + blockIdx.x] = m;
  if (a.nucleus && row_has_nucleus(a, r, vocab))
    for (int i = blockIdx.x * SAMP_T + tid; i < kNucleusHist; i += parts * SAMP_T)
      a.nucleus[(long long)r * kNucleusScratch + i] = 0ull;
}

// one part per lane: their loads go out together
__device__ inline float row_max(const SampleRows& a, int r, int parts) {
  static_assert(kSampleParts <= WAVE, "one part per lane");
  const int lane = threadIdx.x & 63;
  return wave_max(lane < parts ? a.part_max[(long long)r * kSampleParts + lane] : -INFINITY);
}

// Second sweep on `parts` workgroups per row: the weights of the same tiles, one sum per
// 256-id segment; rows with a nucleus: histogram 0.  Bound by the arithmetic: 256 rows x 151936 ids without a
// nucleus 40.0 us (64 rows 13.3), where weights by way of keys and 64-bit wavefront sums took 58.6 (18.0) and
// a weight from two 64-bit shifts with sums by exchanges through LDS 45.4 (16.0).
__global__ __launch_bounds__(SAMP_T) void sample_segments_kernel(SampleRows a, int vocab, int parts) {
  __shared__ SampShared sh;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r = blockIdx.y;
  const float* row = a.logits + (long long)(a.logits_row ? a.logits_row[r] : r) * vocab;
  const float inv_t = row_inv_temp(a, r);
  const bool vec_ok = (vocab & 3) == 0 && (((unsigned long long)row) & 15ull) == 0;
  const int n_seg = (vocab + 255) >> 8;
  const int n_tiles = (vocab + 4095) >> 12;
  const float m = row_max(a, r, parts);
  if (a.nucleus && row_has_nucleus(a, r, vocab)) {
    nucleus_histogram(row, vocab, vec_ok, inv_t, m, blockIdx.x, parts, 0, 0u, sh);
    if (tid < kNucleusBins0 && sh.hist[tid]) atomicAdd(a.nucleus + (long long)r * kNucleusScratch + tid, sh.hist[tid]);
    return;
  }
  for (int t = blockIdx.x; t < n_tiles; t += parts) {
    const Seg4 q = load_weights4(row, t * 4096 + tid * 4, vocab, vec_ok, inv_t, m);
    const unsigned long long ws = wave_total_weights(q.w[0] + q.w[1] + q.w[2] + q.w[3]);
    if (lane == 0 && t * 16 + wave < n_seg) a.seg_sums[(long long)r * kSampleSegments + t * 16 + wave] = ws;
  }
}

// The sweeps that only rows with a nucleus need, `parts` workgroups per row: histogram 1, histogram 2 (every
// workgroup finds the bins of the histograms before it again, from a few KiB), then the segments.
template <int LEVEL>
__global__ __launch_bounds__(SAMP_T) void sample_nucleus_kernel(SampleRows a, int vocab, int parts) {
  __shared__ SampShared sh;
  const int tid = threadIdx.x, r = blockIdx.y;
  if (!row_has_nucleus(a, r, vocab)) return;  // uniform
  const float* row = a.logits + (long long)(a.logits_row ? a.logits_row[r] : r) * vocab;
  const float inv_t = row_inv_temp(a, r);
  const bool vec_ok = (vocab & 3) == 0 && (((unsigned long long)row) & 15ull) == 0;
  const float m = row_max(a, r, parts);
  unsigned long long S;
  const NucleusState st = nucleus_from_scratch(a, r, LEVEL, S, sh);
  unsigned long long* scratch = a.nucleus + (long long)r * kNucleusScratch;
  if constexpr (LEVEL < 3) {
    nucleus_histogram(row, vocab, vec_ok, inv_t, m, blockIdx.x, parts, LEVEL, st.prefix, sh);
    unsigned long long* h = scratch + (LEVEL == 1 ? kNucleusBins0 : kNucleusBins0 + 1024);
    if (tid < nucleus_bins(LEVEL) && sh.hist[tid]) atomicAdd(h + tid, sh.hist[tid]);
  } else {
    unsigned* ties = (unsigned*)(scratch + kNucleusHist);
    if (blockIdx.x == 0 && tid == 0) {  // for the selection
      unsigned long long* found = scratch + kNucleusFound;
      found[0] = S;
      found[1] = st.theta;
      found[2] = st.above;
      found[3] = st.prefix;
    }
    nucleus_segments(row, vocab, vec_ok, inv_t, m, blockIdx.x, parts, st.prefix,
                     [&](int seg, unsigned long long above, unsigned n) {
                       a.seg_sums[(long long)r * kSampleSegments + seg] = above;
                       ties[seg] = n;
                     });
  }
}

// parts = 0: this kernel sweeps the row itself; else it starts from what the kernels above left
__global__ __launch_bounds__(SAMP_T) void sample_kernel(SampleRows a, int vocab, int parts) {
  __shared__ SampShared sh;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r = blockIdx.x;
  const float* row = a.logits + (long long)(a.logits_row ? a.logits_row[r] : r) * vocab;
  const float inv_t = row_inv_temp(a, r);
  const bool vec_ok = (vocab & 3) == 0 && (((unsigned long long)row) & 15ull) == 0;
  const int n_seg = (vocab + 255) >> 8;
  const int n_tiles = (vocab + 4095) >> 12;
  const bool nucleus = row_has_nucleus(a, r, vocab);

  float m = -INFINITY;
  unsigned long long S = 0;
  NucleusState st{0ull, 0ull, 0u};
  if (parts) {
    m = row_max(a, r, parts);
    if (nucleus) {
      const unsigned long long* scratch = a.nucleus + (long long)r * kNucleusScratch;
      S = scratch[kNucleusFound];
      st = NucleusState{scratch[kNucleusFound + 1], scratch[kNucleusFound + 2], (unsigned)scratch[kNucleusFound + 3]};
      const unsigned* ties = (const unsigned*)(scratch + kNucleusHist);
      if (tid < n_seg) {
        sh.hist[tid] = a.seg_sums[(long long)r * kSampleSegments + tid];
        sh.ties[tid] = ties[tid];
      }
    } else {
      unsigned long long local = 0;
      if (tid < n_seg) {
        local = a.seg_sums[(long long)r * kSampleSegments + tid];
        sh.vals[tid] = local;
      }
      S = block_sum_u64(local, sh);
    }
  } else {
    for (int t = 0; t < n_tiles; ++t) {
      const int i0 = t * 4096 + tid * 4;
      if (vec_ok && i0 + 3 < vocab) {
        const float4 v = *(const float4*)(row + i0);
        m = fmaxf(fmaxf(m, fmaxf(scaled_logit(v.x, inv_t), scaled_logit(v.y, inv_t))),
                  fmaxf(scaled_logit(v.z, inv_t), scaled_logit(v.w, inv_t)));
      } else {
        for (int e = 0; e < 4; ++e)
          if (i0 + e < vocab) m = fmaxf(m, scaled_logit(row[i0 + e], inv_t));
      }
    }
    m = block_max(m, sh);
    if (nucleus) {
      nucleus_histogram(row, vocab, vec_ok, inv_t, m, 0, 1, 0, 0u, sh);
      S = block_sum_u64(sh.hist[tid], sh);
      st.theta = nucleus_theta(S, row_top_p(a, r));
      nucleus_descend(sh.hist, 0, st, sh);
      for (int level = 1; level < 3; ++level) {
        nucleus_histogram(row, vocab, vec_ok, inv_t, m, 0, 1, level, st.prefix, sh);
        nucleus_descend(sh.hist, level, st, sh);
      }
      nucleus_segments(row, vocab, vec_ok, inv_t, m, 0, 1, st.prefix,
                       [&](int seg, unsigned long long above, unsigned n) {
                         sh.hist[seg] = above;
                         sh.ties[seg] = n;
                       });
    } else {
      // all weights, one sum per segment
      unsigned long long local = 0;
      for (int t = 0; t < n_tiles; ++t) {
        const Seg4 q = load_weights4(row, t * 4096 + tid * 4, vocab, vec_ok, inv_t, m);
        const unsigned long long mine = q.w[0] + q.w[1] + q.w[2] + q.w[3];
        local += mine;
        const unsigned long long ws = wave_total_weights(mine);
        if (lane == 0 && t * 16 + wave < n_seg) sh.vals[t * 16 + wave] = ws;
      }
      S = block_sum_u64(local, sh);  // also orders the writes to sh.vals
    }
  }

  int token = a.forced ? a.forced[r] : -1;
  if ((unsigned)token >= (unsigned)vocab) {  // nothing forced (an id outside the vocabulary forces nothing)
    // nucleus membership: key above tau's, or at tau among the first k_ties ids there
    const unsigned tau_key = st.prefix;
    unsigned long long s_n = S;
    unsigned k_ties = 0;
    if (nucleus) {
      __syncthreads();
      const unsigned long long tau = key_weight(tau_key);
      k_ties = tau ? (unsigned)((st.theta - st.above + tau - 1) / tau) : 0u;  // theta > above: tau's bin was needed to reach it
      s_n = st.above + k_ties * tau;
      const unsigned mine = tid < n_seg ? sh.ties[tid] : 0u;
      const unsigned before = (unsigned)block_scan_u64(mine, sh) - mine;
      const unsigned in = before < k_ties ? min(mine, k_ties - before) : 0u;
      if (tid < n_seg) {
        sh.vals[tid] = sh.hist[tid] + in * tau;
        sh.ties[tid] = in;  // ids at tau that are in, per segment
      }
      __syncthreads();
    }
    // inverse CDF in ascending id order over the nucleus
    const unsigned x = a.uniforms ? a.uniforms[r]
                                  : philox_word0(a.seed, (unsigned long long)a.sample_id[r], (unsigned)a.step[r]);
    const unsigned long long R = (s_n >> 32) * x + (((s_n & 0xffffffffull) * x) >> 32);
    int seg;
    unsigned long long before;
    find_segment(sh, n_seg, R, seg, before);
    if (wave == 0) {
      const Key4 q = load_keys4(row, seg * 256 + lane * 4, vocab, vec_ok, inv_t, m);
      unsigned long long v[4];
      if (nucleus) {
        unsigned at_tau = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) at_tau += q.k[e] == tau_key ? 1u : 0u;
        unsigned rank = at_tau;
        for (int o = 1; o < WAVE; o <<= 1) {
          const unsigned up = __shfl_up(rank, o, WAVE);
          if (lane >= o) rank += up;
        }
        rank -= at_tau;  // ids at tau before this lane's
        const unsigned in = sh.ties[seg];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool tie = q.k[e] == tau_key;
          v[e] = q.k[e] > tau_key || (tie && rank < in) ? key_weight(q.k[e]) : 0ull;
          rank += tie ? 1u : 0u;
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = key_weight(q.k[e]);
      }
      const int idx = resolve_in_segment(v, R - before, lane);
      if (lane == 0) sh.bcast[0] = (unsigned long long)(seg * 256 + idx);
    }
    __syncthreads();
    token = min(max((int)sh.bcast[0], 0), vocab - 1);  // (no id is found in a row without weights)
  }
  if (tid == 0) {
    float d = shifted(scaled_logit(row[token], inv_t), m);
    a.tokens[r] = token;
    a.logprobs[r] = d - (float)(log((double)S) - 40.0 * 0.693147180559945309417);
    if (a.weight_sums) a.weight_sums[r] = S;
    if (a.host_tokens) {
      a.host_tokens[r] = token;
      a.host_logprobs[r] = a.logprobs[r];
    }
    const int sl = a.row_slot ? a.row_slot[r] : -1;
    if (sl >= 0) {
      a.slots.last_token[sl] = token;
      a.slots.pos[sl] = a.row_pos[r] + a.pos_step;
      a.slots.step[sl] = a.step[r] + 1;
      a.slots.sample_id[sl] = a.sample_id[r];
      a.slots.inv_temp[sl] = a.inv_temp[r];
      a.slots.top_p[sl] = a.top_p[r];
    }
  }
}

// Large vocabularies with scratch at hand: the sweeps of a row on several workgroups (about 512 in all),
// then the selection; else everything in one workgroup per row.
// 64 rows x 151936 ids, top_p 0.9: 8.1 + 16.3 us for maximum and histogram 0, 12.9 + 12.5 + 24.7 us for the other
// histograms and the segments above tau, 9.1 us for the selection: 95 us per call of rollout_sample, where
// one workgroup per row that searched tau bit by bit took 1809 us.  (111 us with the parts' maxima read one
// after the other, scans through LDS and every id's weight computed in histograms 1 and 2.)  The sweeps'
// arithmetic takes the time: 39 MB of logits pass in 8 us.
static void launch_sample_rows(const SampleRows& r, int rows, int vocab, hipStream_t s) {
  const int n_tiles = (vocab + 4095) >> 12;
  int parts = 0;
  if (r.part_max && r.seg_sums && (r.nucleus || !r.any_nucleus) && n_tiles >= 8 && vocab <= 256 * kSampleSegments)
    parts = std::max(2, std::min({n_tiles, kSampleParts, 512 / rows}));
  if (parts < 2) {
    sample_kernel<<<rows, SAMP_T, 0, s>>>(r, vocab, 0);
    return;
  }
  const dim3 grid(parts, rows);
  sample_max_kernel<<<grid, SAMP_T, 0, s>>>(r, vocab, parts);
  sample_segments_kernel<<<grid, SAMP_T, 0, s>>>(r, vocab, parts);
  if (r.any_nucleus) {
    sample_nucleus_kernel<1><<<grid, SAMP_T, 0, s>>>(r, vocab, parts);
    sample_nucleus_kernel<2><<<grid, SAMP_T, 0, s>>>(r, vocab, parts);
    sample_nucleus_kernel<3><<<grid, SAMP_T, 0, s>>>(r, vocab, parts);
  }
  sample_kernel<<<rows, SAMP_T, 0, s>>>(r, vocab, parts);
}

void launch_sample(SampleRows r, int rows, int vocab, hipStream_t s) {
  if (!r.any_nucleus) r.nucleus = nullptr;
  // the nucleus scratch holds nucleus_rows rows: more of them go batch by batch
  const int batch = r.any_nucleus && r.nucleus ? r.nucleus_rows : rows;
  for (int r0 = 0; r0 < rows; r0 += batch) {
    SampleRows b = r;
    if (r0) {
      if (b.logits_row) b.logits_row += r0;
      else b.logits += (long long)r0 * vocab;
      if (b.inv_temp) b.inv_temp += r0;
      if (b.top_p) b.top_p += r0;
      if (b.uniforms) b.uniforms += r0;
      if (b.sample_id) b.sample_id += r0;
      if (b.step) b.step += r0;
      if (b.forced) b.forced += r0;
      b.tokens += r0;
      b.logprobs += r0;
      if (b.weight_sums) b.weight_sums += r0;
      if (b.host_tokens) b.host_tokens += r0, b.host_logprobs += r0;
      if (b.row_slot) b.row_slot += r0, b.row_pos += r0;
    }
    launch_sample_rows(b, std::min(batch, rows - r0), vocab, s);
  }
}

// ---------------------------------------------------------------- teacher-forced gather
__global__ __launch_bounds__(SAMP_T) void logprob_gather_kernel(const float* __restrict__ logits,
                                                                const int* __restrict__ target, float inv_t,
                                                                float* __restrict__ out, int vocab) {
  __shared__ SampShared sh;
  const int tid = threadIdx.x, r = blockIdx.x;
  const int tgt = target[r];
  if (tgt < 0) {
    if (tid == 0) out[r] = 0.f;
    return;
  }
  const float* row = logits + (long long)r * vocab;
  float m = -INFINITY;
  for (int i = tid; i < vocab; i += SAMP_T) m = fmaxf(m, row[i] * inv_t);
  m = block_max(m, sh);
  float part = 0.f;
  for (int i = tid; i < vocab; i += SAMP_T) part += expf(row[i] * inv_t - m);
  part = wave_sum(part);
  if ((tid & 63) == 0) sh.fwave[tid >> 6] = part;
  __syncthreads();
  if (tid == 0) {
    float total = 0.f;
    for (int i = 0; i < SAMP_T / WAVE; ++i) total += sh.fwave[i];
    out[r] = row[tgt] * inv_t - m - logf(total);
  }
}
void launch_logprob_gather(const float* logits, const int* target, float inv_temp, float* out, int rows,
                           int vocab, hipStream_t s) {
  if (rows) logprob_gather_kernel<<<rows, SAMP_T, 0, s>>>(logits, target, inv_temp, out, vocab);
}
