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
// found from the top by a prefix sum.  The sweeps of a row run on several workgroups, and the sweep that fills
// histogram 1 is the last one as a rule: it leaves, per segment of 256 ids, the weight of the bins above the one found,
// and lists the ids of that bin (some 500 of 151936 where logits spread like N(0, 2.5)); the draw finds the
// rest from the list.  Rows so flat that the list would overflow (nucleus_is_flat) take full sweeps instead:
// histogram 1, histogram 2, then per segment the weight above tau and the number of ids at tau.  64 rows x 151936 ids,
// top_p 0.9: see launch_sample_rows.
#include <algorithm>

#include "kernel_timer.h"
#include "kernels.h"

#pragma clang fp contract(off)

#define SAMP_T 1024

// The weight as a float, exact (24 significant bits at most): P(frac(t)) with its exponent raised by 40 + floor(t),
// t = d * log2(e), less what is worth less than 1; 0 for t below -40.  No branch, so that the arithmetic of a
// thread's ids interleaves.  The coefficients carry the 2^40 (a power of two scales every product and sum exactly), and a t below -40,
// or one that is no number, becomes one whose weight is below 1.
__device__ inline float fixexp_value(float d) {
#pragma clang fp contract(off)
  const float log2e = 0x1.715476p+0f;
  float t = d * log2e;
  t = t >= -40.0f ? t : -50.0f;
  float n = floorf(t);
  float f = t - n;
  float y = 0x1.5bd2aep+24f;
  y = y * f;
  y = y + 0x1.3262dep+27f;
  y = y * f;
  y = y + 0x1.5efc6ap+30f;
  y = y * f;
  y = y + 0x1.3b1a32p+33f;
  y = y * f;
  y = y + 0x1.c6b140p+35f;
  y = y * f;
  y = y + 0x1.ebfbdep+37f;
  y = y * f;
  y = y + 0x1.62e430p+39f;
  y = y * f;
  y = y + 0x1.000000p+40f;
  // y is about 2^40 to 2^41, so nothing leaves the exponent's 8 bits
  return truncf(__uint_as_float(__float_as_uint(y) + ((unsigned)(int)n << 23)));
}
// its bits: they order like the weights
__device__ inline unsigned fixexp_key(float d) { return __float_as_uint(fixexp_value(d)); }
// A weight, at most 2^41, as hi 2^22 + lo, lo below 2^22: a few instructions where 64-bit shifts take several times as
// many cycles, and 256 ids' parts add up in 32 bits.
struct WeightParts {
  unsigned hi, lo;
};
__device__ inline WeightParts weight_parts(float v) {
  const unsigned hi = (unsigned)(v * 0x1p-22f);
  return WeightParts{hi, (unsigned)fmaf(-0x1p22f, (float)hi, v)};
}
__device__ inline unsigned long long parts_sum(const WeightParts& w) { return ((unsigned long long)w.hi << 22) + w.lo; }
__device__ inline unsigned long long key_weight(unsigned key) { return parts_sum(weight_parts(__uint_as_float(key))); }

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
__device__ inline unsigned long long row_scan_u64(unsigned long long v) {  // over each 16 lanes
  v = dpp_add_u64<0x111, 0xf>(v);
  v = dpp_add_u64<0x112, 0xf>(v);
  v = dpp_add_u64<0x114, 0xf>(v);
  return dpp_add_u64<0x118, 0xf>(v);
}
__device__ inline unsigned long long read_lane_u64(unsigned long long v, int lane) {  // lane: uniform
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), lane);
  return ((unsigned long long)hi << 32) | lo;
}
__device__ inline unsigned long long wave_scan_u64(unsigned long long v) {
  v = row_scan_u64(v);
  v = dpp_add_u64<0x142, 0xa>(v);
  return dpp_add_u64<0x143, 0xc>(v);
}
__device__ inline unsigned long long wave_total_u64(unsigned long long v) {
  return read_lane_u64(wave_scan_u64(v), 63);
}

// Sum over the wavefront, in every lane.
__device__ inline unsigned wave_total_u32(unsigned v) {
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);
  v += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);
  return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ inline unsigned long long wave_total_weights(const WeightParts& w) {
  return parts_sum(WeightParts{wave_total_u32(w.hi), wave_total_u32(w.lo)});
}

struct SampShared {
  unsigned long long vals[SAMP_T];   // one value per segment
  unsigned long long hist[SAMP_T];   // a histogram, or the nucleus' weight above tau per segment
  unsigned ties[SAMP_T];             // ids at tau per segment
  unsigned long long wave_part[SAMP_T / WAVE];
  unsigned long long bcast[3];
  float fwave[SAMP_T / WAVE];
  float log_sum, logit;
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

// Inclusive prefix sum over the threads of the workgroup, and the sum over all of them.
__device__ inline unsigned long long block_scan_u64(unsigned long long v, SampShared& sh, unsigned long long& total) {
  static_assert(SAMP_T / WAVE == 16, "a wavefront's sum to each lane of a row");
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  v = wave_scan_u64(v);
  if (lane == 63) sh.wave_part[wave] = v;
  __syncthreads();
  const unsigned long long waves = row_scan_u64(sh.wave_part[lane & 15]);
  total = read_lane_u64(waves, 15);
  if (wave > 0) v += read_lane_u64(waves, wave - 1);
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
struct Key4 {
  unsigned k[4];
};

struct Logit4 {
  float v[4];
};

// logits of ids i0 .. i0 + 3 for i0 <= vocab - 4, of the row's last four for more (logits4 puts those right).  One
// 16-byte load whatever the row's alignment (the chip asks for that of a dword), and no branch: a load behind one
// waits for the loads before it.
typedef float quad_any __attribute__((ext_vector_type(4), aligned(4)));
template <bool ANY_VOCAB>
__device__ inline Logit4 request4(const float* __restrict__ row, int i0, int vocab) {
  Logit4 out;
  if (!ANY_VOCAB || vocab >= 4) {
    const quad_any t = *(const quad_any*)(row + min(i0, vocab - 4));
#pragma unroll
    for (int e = 0; e < 4; ++e) out.v[e] = t[e];
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) out.v[e] = row[min(e, vocab - 1)];
  }
  return out;
}
// ids past the end hold one of the row's last logits, for the caller to leave out
__device__ inline Logit4 logits4(Logit4 z, int i0, int vocab) {
  if (i0 > vocab - 4 && vocab >= 4 && (vocab & 3)) {
    const int by = min(i0 - (vocab - 4), 3);
    if (by & 1) z = Logit4{{z.v[1], z.v[2], z.v[3], z.v[3]}};
    if (by & 2) z = Logit4{{z.v[2], z.v[3], z.v[3], z.v[3]}};
  }
  return z;
}
__device__ inline Key4 keys4(const Logit4& z, int i0, int vocab, float inv_t, float m) {
  Key4 out;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const unsigned key = fixexp_key(shifted(scaled_logit(z.v[e], inv_t), m));
    out.k[e] = i0 + e < vocab ? key : 0u;
  }
  return out;
}
__device__ inline WeightParts weight4(const Logit4& z, int i0, int vocab, float inv_t, float m) {  // of the four together
  const Key4 q = keys4(z, i0, vocab, inv_t, m);
  WeightParts sum{0u, 0u};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const WeightParts w = weight_parts(__uint_as_float(q.k[e]));
    sum.hi += w.hi;
    sum.lo += w.lo;
  }
  return sum;
}

// How `parts` workgroups share a row: whole rounds of tiles go round by tile, and what is left by segments, the same
// number to each, so that the last round does not leave some of them idle (38 tiles, 8 parts: 75 segments each instead of 64
// or 80).  The last round's segments of a part are one wavefront's each, as in a tile.
struct RowShares {
  int parts, rounds, per;  // whole rounds; ids of the rest per part
  __host__ __device__ RowShares(int vocab, int parts) : parts(parts), rounds((vocab >> 12) / parts) {
    per = (((vocab - rest0() + 255) >> 8) + parts - 1) / parts << 8;
  }
  __host__ __device__ inline int rest0() const { return rounds * parts << 12; }  // the first id behind the rounds
  __device__ inline int part_of_segment(int seg) const {
    const int rest = seg - (rest0() >> 8);
    return rest < 0 ? (seg >> 4) % parts : rest / (per >> 8);
  }
};

// This thread's four logits of a part's share of a row, round by round.  The first AHEAD rounds are requested where the object
// is made, so that they are under way while a sweep finds out what it needs to know of the sweeps before (those
// sweeps have vocabularies of several tiles).  One round ahead in the sweeps of a nucleus, each round the next: with four, the
// 64 registers that two workgroups to a CU leave to a thread overflowed into memory in every round (64 rows x 151936 48.1 -> 39.6 us
// a call, 96 x 65536 42.6 -> 33.6, 170 x 32001 38.3 -> 31.7); four in the sweeps without one, which have the registers.
template <int AHEAD>
struct RowTiles {
  const float* row;
  int vocab, part;
  RowShares in;
  Logit4 ahead[AHEAD > 0 ? AHEAD : 1];
  __device__ inline int first_id(int q) const {  // of round q
    const int i0 = (int)threadIdx.x * 4;
    if (q < in.rounds) return ((part + q * in.parts) << 12) + i0;
    const int at = (q - in.rounds) * 4096 + i0;  // (a rest of more than a tile per part is none: it would be a round)
    return at < in.per ? in.rest0() + part * in.per + at : 0x7ffffff0;
  }
  __device__ inline RowTiles(const float* row, int vocab, int part, const RowShares& in) : row(row), vocab(vocab), part(part), in(in) {
#pragma unroll
    for (int q = 0; q < AHEAD; ++q) ahead[q] = request4<false>(row, first_id(q), vocab);
    if (AHEAD > 0) __builtin_amdgcn_sched_barrier(0);
  }
  // f(first id, logits) of every round; a wavefront whose ids all lie past the end passes.  (With one workgroup per row a
  // small vocabulary leaves most wavefronts of its one tile without any, and their arithmetic took as long again as the
  // others': 1024 ids, top_p 1 / 0.9 6.0 -> 5.4, 13.3 -> 11.9 us a call.)
  template <typename F>
  __device__ inline void each(F&& f) const {
    if constexpr (AHEAD == 1) {  // every round's logits are requested ahead of the round before
      auto round = [&](int q, const Logit4& z) {
        const int i0 = first_id(q);
        if ((i0 & ~255) < vocab) f(i0, logits4(z, i0, vocab));  // (uniform: a wavefront's 256 ids are one segment)
      };
      Logit4 next = ahead[0];
      for (int q = 0; q < in.rounds; ++q) {
        const Logit4 z = next;
        next = request4<false>(row, first_id(q + 1), vocab);
        __builtin_amdgcn_sched_barrier(0);
        round(q, z);
      }
      round(in.rounds, next);
    } else {
#pragma unroll
      for (int q = 0; q < AHEAD; ++q) {
        const int i0 = first_id(q);
        if ((i0 & ~255) < vocab) f(i0, logits4(ahead[q], i0, vocab));
      }
      for (int q = AHEAD; q <= in.rounds; ++q) {
        const int i0 = first_id(q);
        if ((i0 & ~255) < vocab) f(i0, logits4(request4<AHEAD == 0>(row, i0, vocab), i0, vocab));
      }
    }
  }
};

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

__device__ inline unsigned long long nucleus_theta(unsigned long long S, float top_p) {
  const unsigned long long p24 = (unsigned long long)floorf(fmaxf(top_p, 0.f) * 16777216.0f);
  const unsigned long long theta = (S >> 24) * p24 + (((S & 0xffffffull) * p24) >> 24);
  return theta < 1 ? 1 : theta;
}
struct NucleusState {
  unsigned long long sum, theta, above;  // all weight; weight to reach; weight of the bins above the ones found
  unsigned prefix;                       // key bits found so far (nucleus_prefix of the next level; the key of tau after level 2)
  unsigned long long here;               // weight of the bin found last
};
// One more level.  The histogram's bins, counted from the top, lie one per thread (v); the first at which the weight
// from the top reaches theta is found.
__device__ inline void nucleus_descend(unsigned long long v, int level, float top_p, NucleusState& st, SampShared& sh) {
  const int n = nucleus_bins(level), t = threadIdx.x;
  if (t == 0) sh.bcast[0] = sh.bcast[1] = sh.bcast[2] = 0ull;  // a row without weights (no finite maximum) finds no bin
  unsigned long long total;
  const unsigned long long inc = block_scan_u64(v, sh, total) + st.above;
  if (level == 0) {
    st.sum = total;
    st.theta = nucleus_theta(total, top_p);
  }
  if (t < n && inc >= st.theta && inc - v < st.theta) {  // exactly one thread: the sums only grow, and all of them reach theta
    sh.bcast[0] = (unsigned long long)(n - 1 - t);
    sh.bcast[1] = inc - v;
    sh.bcast[2] = v;
  }
  __syncthreads();
  const unsigned bin = (unsigned)sh.bcast[0];
  st.above = sh.bcast[1];
  st.here = sh.bcast[2];
  st.prefix = level == 0 ? bin + (127u << 4) : level == 1 ? (st.prefix << 10) | bin : (st.prefix << 9) | bin;
  __syncthreads();
}
// Loads and stores at the scope of the device: what parts of a row, on different XCDs, leave for each other in one launch.
template <typename T>
__device__ inline T load_device(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ inline void store_device(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// this thread's bin of a histogram (in LDS, or DEVICE: in the scratch), counted from the top
template <bool DEVICE>
__device__ inline unsigned long long nucleus_bin_from_top(const unsigned long long* hist, int level) {
  const int at = nucleus_bins(level) - 1 - (int)threadIdx.x;
  if (at < 0) return 0ull;
  return DEVICE ? load_device(hist + at) : hist[at];
}
// The tiles into the LDS histogram of `level` (zeroed here).  From level 1 on only the ids
// of one narrow bin count, so an id whose exponent t lies outside the bin's range is passed over before its
// weight is computed: a weight w in the bin [lo, hi) comes from a value in [w, w + 1) that is 2^(40 + t) within
// a few 2^-23, so t + 40 lies between log2(lo) and log2(hi + 1), each widened by 0.01.
template <int AHEAD>
__device__ inline void nucleus_histogram(const RowTiles<AHEAD>& tiles, float inv_t, float m, int level, unsigned prefix,
                                         SampShared& sh) {
  sh.hist[threadIdx.x] = 0ull;
  __syncthreads();
  if (level > 0) {
    const int shift = level == 1 ? 19 : 9;
    const float t_lo = log2f(__uint_as_float(prefix << shift)) - 40.01f;
    const float t_hi = log2f(__uint_as_float((prefix + 1u) << shift) + 1.f) - 39.99f;
    tiles.each([&](int i0, const Logit4& z) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float d = shifted(scaled_logit(z.v[e], inv_t), m), x = d * 0x1.715476p+0f;
        if (x >= t_lo && x <= t_hi && i0 + e < tiles.vocab) {  // (not so where d is no number)
          const unsigned key = fixexp_key(d);
          if (key && nucleus_prefix(key, level) == prefix) atomicAdd(&sh.hist[nucleus_bin(key, level)], key_weight(key));
        }
      }
    });
  } else {
    tiles.each([&](int i0, const Logit4& z) {
      const Key4 q = keys4(z, i0, tiles.vocab, inv_t, m);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (q.k[e]) atomicAdd(&sh.hist[nucleus_bin(q.k[e], 0)], key_weight(q.k[e]));
    });
  }
  __syncthreads();
}
// Per segment the weight above tau and the number of ids at tau
template <int AHEAD, typename F>
__device__ inline void nucleus_segments(const RowTiles<AHEAD>& tiles, float inv_t, float m, unsigned tau_key, F&& put) {
  const int n_seg = (tiles.vocab + 255) >> 8;
  tiles.each([&](int i0, const Logit4& z) {
    const Key4 q = keys4(z, i0, tiles.vocab, inv_t, m);
    WeightParts above{0u, 0u};
    unsigned at = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const WeightParts w = weight_parts(__uint_as_float(q.k[e]));
      above.hi += q.k[e] > tau_key ? w.hi : 0u;
      above.lo += q.k[e] > tau_key ? w.lo : 0u;
      at += (unsigned)__popcll(__ballot(q.k[e] == tau_key));
    }
    const unsigned long long sum = wave_total_weights(above);
    const int seg = i0 >> 8;
    if ((threadIdx.x & 63) == 0 && seg < n_seg) put(seg, sum, at);
  });
}

// Smallest segment whose inclusive prefix of the segments' values (one per thread) exceeds target, and the
// exclusive prefix before it.  Requires the total to exceed target.
__device__ inline void find_segment(SampShared& sh, unsigned long long mine, unsigned long long target, int& seg,
                                    unsigned long long& before) {
  if (threadIdx.x == 0) sh.bcast[0] = sh.bcast[1] = 0ull;
  unsigned long long total;
  const unsigned long long inc = block_scan_u64(mine, sh, total);  // (its barriers stand between the two writes)
  if (inc > target && inc - mine <= target) {
    sh.bcast[0] = threadIdx.x;
    sh.bcast[1] = inc - mine;
  }
  __syncthreads();
  seg = (int)sh.bcast[0];
  before = sh.bcast[1];
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

// The parts' common words of a row (SampleRows::part_max)
__device__ inline unsigned* meeting_words(const SampleRows& a, int r) {
  return (unsigned*)a.part_max + (long long)r * kSampleHead + kSampleParts;
}

// First launch, `parts` workgroups per row: maximum of the scaled logits over a part's share (RowShares)
__global__ __launch_bounds__(SAMP_T, 8) void sample_max_kernel(SampleRows a, int vocab, RowShares in) {
  const int parts = in.parts;
  __shared__ SampShared sh;
  const int tid = threadIdx.x, r = blockIdx.y;
  const float* row = a.logits + (long long)(a.logits_row ? a.logits_row[r] : r) * vocab;
  const float inv_t = row_inv_temp(a, r);
  float m = -INFINITY;
  RowTiles<4>(row, vocab, blockIdx.x, in).each([&](int, const Logit4& z) {  // an id taken twice changes no maximum
#pragma unroll
    for (int e = 0; e < 4; ++e) m = fmaxf(m, scaled_logit(z.v[e], inv_t));
  });
  m = block_max(m, sh);
  if (tid == 0) a.part_max[(long long)r * kSampleHead + blockIdx.x] = m;
  // the words the parts meet at, and behind them the row's random word: from host memory it takes the draw 2 us
  if (blockIdx.x == 0 && tid < kSampleHead - kSampleParts) meeting_words(a, r)[tid] = tid < kMeetWords || !a.uniforms ? 0u : a.uniforms[r];
  if (a.nucleus && row_has_nucleus(a, r, vocab))
    for (int i = blockIdx.x * SAMP_T + tid; i < kNucleusHist; i += parts * SAMP_T)
      a.nucleus[(long long)r * kNucleusScratch + i] = 0ull;
}

// one part per lane: their loads go out together, and wave_max joins them
__device__ inline float row_part_max(const SampleRows& a, int r, int parts) {
  static_assert(kSampleParts <= WAVE, "one part per lane");
  return a.part_max[(long long)r * kSampleHead + min((int)threadIdx.x & 63, parts - 1)];
}

// What lanes of a wavefront wrote to LDS before it, others read after it.  (Its LDS accesses are carried out in order, so
// this is an order for the compiler and no instruction.)
__device__ inline void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ids a part can list
__device__ inline int nucleus_listed(int parts) { return min(2048, kNucleusListed / parts); }
// Did a part of row r find more ids in its bin than it could list?  Every lane takes a part's count.
__device__ inline bool nucleus_overflow(const unsigned long long* scratch, int parts) {
  const unsigned n = load_device((const unsigned*)(scratch + kNucleusCounts) + min((int)threadIdx.x & 63, parts - 1));
  return __any(n > (unsigned)nucleus_listed(parts));
}

// Will the ids of the bin that histogram 0 names overflow the list?  Its weight over the power of two below it is their number, or
// what it would be at the foot of that power of two, where bins are twice as wide as at its end: whatever the phase,
// rows of one spread decide alike.  (A call whose rows go both ways pays for both: 64 rows of N(0, 0.2) by the true
// number 99 us.)  They fall to the parts within some three standard deviations.  64 rows x 151936 ids of N(0, s), top_p
// 0.9, us a call with the list / with full sweeps throughout: s 0.05 99 / 86, 0.2 101 / 80 (some 7500 ids: the
// list overflows), 0.35 74 / 80, 0.7 65 / 79, 1.5 58 / 78; 256 rows: 0.2 261 / 208, 0.7 252 / 205 (2 x 2048 places),
// 1.0 168 / 205.  The same in every workgroup of a row.
__device__ inline bool nucleus_is_flat(const NucleusState& st, int parts) {
  const float room = __builtin_amdgcn_sqrtf((float)nucleus_listed(parts) + 2.25f) - 1.5f;  // x^2 + 3 x = places
  return (float)st.here > __uint_as_float((st.prefix << 19) & 0x7f800000u) * ((float)parts * room * room);
}

// Do the bin's ids fit one part's places, wherever they lie?  An id weighs at least the power of two below the bin.
__device__ inline bool nucleus_fits(const NucleusState& st, int parts) {
  return (float)st.here <= __uint_as_float((st.prefix << 19) & 0x7f800000u) * (float)nucleus_listed(parts);
}

// What the draw from a row starts with: weights, and with a nucleus its end (st) and, in sh.hist and sh.ties, per segment
// the weight above tau and the ids at tau; without one the segments' weights in sh.vals.  word: the row's random word.
// A chain of round trips and barriers: in a draw the logarithm of the sum is another wavefront's, and the token's logit comes
// from the one that resolves it.
__device__ inline void select_token(const SampleRows& a, int r, const float* row, int vocab, float inv_t, float m,
                                    unsigned long long S, const NucleusState& st, bool nucleus, const unsigned* word, SampShared& sh) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n_seg = (vocab + 255) >> 8;
  const unsigned x_given = word ? *word : 0u;
  int token = a.forced ? a.forced[r] : -1;
  const bool given = (unsigned)token < (unsigned)vocab;
  const int who = given ? 0 : SAMP_T - 1;
  float log_sum = 0.f, logit = 0.f;
  if (tid == who) {
    if (given) logit = row[token];
    log_sum = (float)(log((double)S) - 40.0 * 0.693147180559945309417);
    if (!given) sh.log_sum = log_sum;
  }
  if (!given) {  // nothing forced (an id outside the vocabulary forces nothing)
    // nucleus membership: key above tau's, or at tau among the first k_ties ids there
    const unsigned tau_key = st.prefix;
    unsigned long long s_n = S, of_segment;
    unsigned k_ties = 0;
    const bool few = n_seg <= WAVE;  // then the first wavefront, which draws, holds all segments and needs no other
    if (nucleus || !few) __syncthreads();
    if (nucleus) {
      const unsigned long long tau = key_weight(tau_key);
      k_ties = tau ? (unsigned)((st.theta - st.above + tau - 1) / tau) : 0u;  // theta > above: tau's bin was needed to reach it
      s_n = st.above + k_ties * tau;
      const unsigned mine = tid < n_seg ? sh.ties[tid] : 0u;
      unsigned long long all;
      const unsigned before = (few ? (unsigned)wave_scan_u64(mine) : (unsigned)block_scan_u64(mine, sh, all)) - mine;
      const unsigned in = before < k_ties ? min(mine, k_ties - before) : 0u;
      of_segment = tid < n_seg ? sh.hist[tid] + in * tau : 0ull;
      if (!few || wave == 0) sh.ties[tid] = in;  // ids at tau that are in, per segment
    } else {
      of_segment = tid < n_seg ? sh.vals[tid] : 0ull;
    }
    // inverse CDF in ascending id order over the nucleus
    const unsigned x = word ? x_given : philox_word0(a.seed, (unsigned long long)a.sample_id[r], (unsigned)a.step[r]);
    const unsigned long long R = (s_n >> 32) * x + (((s_n & 0xffffffffull) * x) >> 32);
    int seg;
    unsigned long long before;
    if (!few) find_segment(sh, of_segment, R, seg, before);
    if (wave == 0) {
      if (few) {
        const unsigned long long inc = wave_scan_u64(of_segment);
        const unsigned long long hit = __ballot(inc > R && inc - of_segment <= R);
        seg = hit ? __ffsll((long long)hit) - 1 : 0;
        before = hit ? read_lane_u64(inc - of_segment, seg) : 0ull;
      }
      const int i0 = seg * 256 + lane * 4;
      const Logit4 z = logits4(request4<true>(row, i0, vocab), i0, vocab);
      const Key4 q = keys4(z, i0, vocab, inv_t, m);
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
        if (few) wave_lds_fence();  // another lane's word (the other way has a barrier between)
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
      if (idx >= 0 && lane == idx >> 2) sh.logit = (idx & 3) == 0 ? z.v[0] : (idx & 3) == 1 ? z.v[1] : (idx & 3) == 2 ? z.v[2] : z.v[3];
      token = min(max(seg * 256 + idx, 0), vocab - 1);  // (no id is found in a row without weights)
      if (lane == 0 && idx < 0) sh.logit = row[token];
    }
    __syncthreads();
    logit = sh.logit;
    log_sum = sh.log_sum;
  }
  if (tid == 0) {
    const float d = shifted(scaled_logit(logit, inv_t), m);
    a.tokens[r] = token;
    const float logprob = d - log_sum;
    a.logprobs[r] = logprob;
    if (a.weight_sums) a.weight_sums[r] = S;
    if (a.host_tokens) {
      a.host_tokens[r] = token;
      a.host_logprobs[r] = logprob;
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


// Where the parts of a row meet between the phases of one launch: count (words 4 phase) and `left` (the 64 bits behind).
// Every part does its share and reports, and the one that reports last is `last`; the others look up to `patience` times whether
// all have reported (below 0: they end).  A part waits only so long: if the others have not reported by then - their workgroups may not even run, for all it
// knows - it leaves its share of the phases to come to the last one and ends.  So no wait needs another workgroup
// to make progress, and every share is done once: the last one closes `left` as it takes what is in it, and
// a part that finds it closed keeps its own.  What the parts leave for each other goes by load_device, store_device
// and atomics, and is there when they report.  Returns the shares to go on with; 0: this workgroup is done.
constexpr unsigned long long kLeftClosed = 1ull << 63;
__device__ inline unsigned long long meet(unsigned* words, int phase, int parts, unsigned long long shares, int patience, bool& last,
                                          SampShared& sh) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned* count = words + 4 * phase;
    unsigned long long* left = (unsigned long long*)(words + 4 * phase + 2);
    const int n = __popcll(shares);
    int seen = (int)__hip_atomic_fetch_add(count, (unsigned)n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + n;
    const bool is_last = seen == parts;
    if (is_last) {
      shares |= __hip_atomic_exchange(left, kLeftClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else if (patience >= 0) {
      for (int spin = 0; spin < patience && seen != parts; ++spin) {
        __builtin_amdgcn_s_sleep(1);
        seen = (int)load_device(count);
      }
      if (seen != parts && !(__hip_atomic_fetch_or(left, shares, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kLeftClosed)) shares = 0ull;
    } else {
      shares = 0ull;
    }
    sh.bcast[0] = shares;
    sh.bcast[1] = is_last;
  }
  __syncthreads();
  shares = read_lane_u64(sh.bcast[0], 0);
  last = sh.bcast[1] != 0ull;
  __syncthreads();
  return shares;
}

// One part's share of the sweep that lists: histogram 1, the segments' weights above the bin that histogram 0
// names, and the list of its ids; of flat rows histogram 1 alone, and the part says that its list overflowed.
// One id in eight or so can be at or above the bin: a wavefront queues those in LDS and computes their
// weights 64 at a time.  64 rows x 151936 ids: see launch_sample_rows.
struct ListShared {
  uint2 queue[SAMP_T / WAVE][256 + WAVE];  // (logit, id)
  uint2 list[2048];                        // (key, id)
  unsigned listed;
};
__device__ inline void list_share(const SampleRows& a, int r, const RowTiles<1>& tiles, int part, int parts, bool flat, float inv_t,
                                  float m, const NucleusState& st, unsigned long long* scratch, SampShared& sh, ListShared& ls) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, vocab = tiles.vocab;
  const unsigned room = (unsigned)nucleus_listed(parts);
  unsigned* counts = (unsigned*)(scratch + kNucleusCounts);
  if (flat) {
    nucleus_histogram(tiles, inv_t, m, 1, st.prefix, sh);
    if (sh.hist[tid]) atomicAdd(scratch + kNucleusBins0 + tid, sh.hist[tid]);
    if (tid == 0) store_device(counts + part, room + 1u);
    return;
  }
  sh.hist[tid] = sh.vals[tid] = 0ull;
  if (tid == 0) ls.listed = 0u;
  __syncthreads();
  const int n_seg = (vocab + 255) >> 8;
  // As in nucleus_histogram no weight of the bin is found below some t, and so below some logit: t's d + m over
  // 1 / T, lowered by more than the four roundings between a logit and its t add up to.  (No number where there is no
  // finite maximum: no id passes, and none has a weight.)
  const float d_lo = (log2f(__uint_as_float(st.prefix << 19)) - 40.02f) * 0.6931472f;
  const float z_lo = (m + d_lo - 0x1p-19f * (fabsf(m) + fabsf(d_lo))) / inv_t;
  const float lowest = z_lo - 0x1p-19f * fabsf(z_lo);
  uint2* mine = ls.queue[wave];
  int queued = 0;
  auto weigh = [&](const uint2& u, bool full) {
    const unsigned key = fixexp_key(shifted(scaled_logit(__uint_as_float(u.x), inv_t), m)), prefix = key >> 19, seg = u.y >> 8;
    const WeightParts w = weight_parts(__uint_as_float(key));
    const bool above = prefix > st.prefix;
    if (full && __all(seg == (unsigned)__builtin_amdgcn_readfirstlane((int)seg))) {
      // ids of one segment, as in flat rows: 64 atomics on one word are one after the other
      const unsigned long long sum = wave_total_weights(WeightParts{above ? w.hi : 0u, above ? w.lo : 0u});
      if (lane == 0) atomicAdd(&sh.vals[seg], sum);
    } else if (above) {
      atomicAdd(&sh.vals[seg], parts_sum(w));
    }
    if (prefix == st.prefix) {
      atomicAdd(&sh.hist[nucleus_bin(key, 1)], parts_sum(w));
      const unsigned to = atomicAdd(&ls.listed, 1u);
      if (to < room) ls.list[to] = make_uint2(key, u.y);
    }
  };
  tiles.each([&](int i0, const Logit4& z) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool in = z.v[e] >= lowest && i0 + e < vocab;
      const unsigned long long lanes = __ballot(in);
      const int to = queued + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(lanes >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)lanes, 0u));
      if (in) mine[to] = make_uint2(__float_as_uint(z.v[e]), (unsigned)(i0 + e));
      queued += __popcll(lanes);
    }
    wave_lds_fence();
    while (queued >= WAVE) {
      queued -= WAVE;
      weigh(mine[queued + lane], true);
    }
    wave_lds_fence();
  });
  if (lane < queued) weigh(mine[lane], false);
  __syncthreads();
  if (tid < n_seg && tiles.in.part_of_segment(tid) == part) store_device(a.seg_sums + (long long)r * kSampleSegments + tid, sh.vals[tid]);
  if (sh.hist[tid]) atomicAdd(scratch + kNucleusBins0 + tid, sh.hist[tid]);
  if (tid == 0) store_device(counts + part, ls.listed);
  unsigned long long* out = scratch + kNucleusList + part * room;
  for (unsigned q = tid; q < min(ls.listed, room); q += SAMP_T) store_device(out + q, (unsigned long long)ls.list[q].y << 32 | ls.list[q].x);
  __syncthreads();  // ls and sh are free again
}

// Second launch, `parts` workgroups per row: the sweeps behind the maximum and the draw, in phases between which the
// parts meet.  Without a nucleus one sum per 256-id segment, and the last part draws.  With one: histogram 0; the sweep that lists;
// then, unless a part found more ids than it could list, the last part draws, else histogram 2, the
// segments, and the last part draws.  (In flat rows every part says so: nucleus_is_flat.)
// What a phase takes: see launch_sample_rows.  A part's first tiles are requested before
// it knows what it needs to know of the phase before.  As launches of their own the phases cost 2 us each to start, two of
// them for nothing in ordinary rows, and their last workgroups' time: see launch_sample_rows.
// NUCLEUS: some rows may have one.
template <bool NUCLEUS>
__global__ __launch_bounds__(SAMP_T, 8) void sample_rest_kernel(SampleRows a, int vocab, RowShares in) {
  const int parts = in.parts;
  __shared__ SampShared sh;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r = blockIdx.y;
  const float* row = a.logits + (long long)(a.logits_row ? a.logits_row[r] : r) * vocab;
  const float inv_t = row_inv_temp(a, r);
  const int n_seg = (vocab + 255) >> 8;
  const float part_max = row_part_max(a, r, parts);
  unsigned long long shares = 1ull << blockIdx.x;
  unsigned* words = meeting_words(a, r);
  unsigned long long* seg_sums = a.seg_sums + (long long)r * kSampleSegments;
  bool last;
  float m;
  NucleusState st{};
  if (!NUCLEUS || !row_has_nucleus(a, r, vocab)) {  // uniform
    {
      const RowTiles<4> tiles(row, vocab, blockIdx.x, in);
      m = wave_max(part_max);
      tiles.each([&](int i0, const Logit4& z) {
        const unsigned long long ws = wave_total_weights(weight4(z, i0, vocab, inv_t, m));
        if (lane == 0 && i0 >> 8 < n_seg) store_device(seg_sums + (i0 >> 8), ws);
      });
    }
    if (!meet(words, 0, parts, shares, -1, last, sh)) return;
    unsigned long long local = 0;
    if (tid < n_seg) {
      local = load_device(seg_sums + tid);
      sh.vals[tid] = local;
    }
    select_token(a, r, row, vocab, inv_t, m, block_sum_u64(local, sh), st, false, a.uniforms ? words + kMeetWords : nullptr, sh);
    return;
  }
  if constexpr (NUCLEUS) {
    __shared__ ListShared ls;
    unsigned long long* scratch = a.nucleus + (long long)r * kNucleusScratch;
    {
      const RowTiles<1> tiles(row, vocab, blockIdx.x, in);
      m = wave_max(part_max);
      nucleus_histogram(tiles, inv_t, m, 0, 0u, sh);
      if (tid < kNucleusBins0 && sh.hist[tid]) atomicAdd(scratch + tid, sh.hist[tid]);
    }
    const float top_p = row_top_p(a, r);
    // f(part, its tiles) for every share; `before` while the first one's tiles are on their way
    auto each_share = [&](auto&& before, auto&& f) {
      int part = __ffsll((long long)shares) - 1;
      bool first = true;
      for (unsigned long long rest = shares; rest; rest &= rest - 1) {
        part = __ffsll((long long)rest) - 1;
        const RowTiles<1> tiles(row, vocab, part, in);
        if (first) before();
        first = false;
        f(part, tiles);
      }
    };
    shares = meet(words, 0, parts, shares, a.patience, last, sh);
    if (!shares) return;
    bool flat = false, fits = false;
    {
      const unsigned long long h0 = nucleus_bin_from_top<true>(scratch, 0);
      each_share(
          [&] {
            nucleus_descend(h0, 0, top_p, st, sh);
            flat = nucleus_is_flat(st, parts);
            fits = nucleus_fits(st, parts);
          },
          [&](int part, const RowTiles<1>& tiles) { list_share(a, r, tiles, part, parts, flat, inv_t, m, st, scratch, sh, ls); });
    }
    // only the last part goes on where all ids are listed, and the others need not wait to hear that
    shares = meet(words, 1, parts, shares, !flat && fits ? -1 : a.patience, last, sh);
    if (!shares) return;
    // all that is needed as a rule, requested at once: this wavefront's first 64 ids come before their number
    const unsigned long long h1 = nucleus_bin_from_top<true>(scratch + kNucleusBins0, 1);
    const bool overflow = nucleus_overflow(scratch, parts);
    if (!overflow && !last) return;
    if (!overflow) {
      const unsigned* counts = (const unsigned*)(scratch + kNucleusCounts);
      const unsigned long long* list = scratch + kNucleusList;
      const int room = nucleus_listed(parts);
      const unsigned long long sum = load_device(seg_sums + min(tid, n_seg - 1));
      // 16 wavefronts share the lists of up to 16 parts, 8, 4, 2 or one to a part
      const int share = parts > 8 ? 0 : parts > 4 ? 1 : parts > 2 ? 2 : 3, step = WAVE << share;
      const int q = min(wave >> share, parts - 1), i0 = (wave & ((1 << share) - 1)) * WAVE + lane;
      const int n_part = wave >> share < parts ? (int)load_device(counts + q) : 0;
      static_assert(kNucleusListed >= SAMP_T, "a part has room for 64 ids of each of its wavefronts");
      const unsigned long long first = load_device(list + q * room + i0);
      sh.hist[tid] = tid < n_seg ? sum : 0ull;
      sh.vals[tid] = 0ull;
      sh.ties[tid] = 0u;
      nucleus_descend(h1, 1, top_p, st, sh);
      auto each_listed = [&](auto&& f) {
        if (i0 < n_part) f((unsigned)first, (unsigned)(first >> 32));
        for (int i = i0 + step; i < n_part; i += step) {
          const unsigned long long u = load_device(list + q * room + i);
          f((unsigned)u, (unsigned)(u >> 32));
        }
      };
      each_listed([&](unsigned key, unsigned) {
        if (nucleus_prefix(key, 2) == st.prefix) atomicAdd(&sh.vals[nucleus_bin(key, 2)], key_weight(key));
      });
      __syncthreads();
      nucleus_descend(nucleus_bin_from_top<false>(sh.vals, 2), 2, top_p, st, sh);
      each_listed([&](unsigned key, unsigned id) {
        if (key > st.prefix) atomicAdd(&sh.hist[id >> 8], key_weight(key));
        else if (key == st.prefix) atomicAdd(&sh.ties[id >> 8], 1u);
      });
      select_token(a, r, row, vocab, inv_t, m, st.sum, st, true, a.uniforms ? words + kMeetWords : nullptr, sh);
      return;
    }
    // the ids did not fit
    {
      each_share([&] { nucleus_descend(h1, 1, top_p, st, sh); },
                 [&](int, const RowTiles<1>& tiles) {
                   nucleus_histogram(tiles, inv_t, m, 2, st.prefix, sh);
                   if (tid < nucleus_bins(2) && sh.hist[tid]) atomicAdd(scratch + kNucleusBins0 + 1024 + tid, sh.hist[tid]);
                   __syncthreads();
                 });
    }
    shares = meet(words, 2, parts, shares, a.patience, last, sh);
    if (!shares) return;
    unsigned* ties = (unsigned*)(scratch + kNucleusHist);
    {
      const unsigned long long h2 = nucleus_bin_from_top<true>(scratch + kNucleusBins0 + 1024, 2);
      each_share([&] { nucleus_descend(h2, 2, top_p, st, sh); },
                 [&](int, const RowTiles<1>& tiles) {
                   nucleus_segments(tiles, inv_t, m, st.prefix, [&](int seg, unsigned long long above, unsigned n) {
                     store_device(seg_sums + seg, above);
                     store_device(ties + seg, n);
                   });
                 });
    }
    if (!meet(words, 3, parts, shares, -1, last, sh)) return;
    if (tid < n_seg) {
      sh.hist[tid] = load_device(seg_sums + tid);
      sh.ties[tid] = load_device(ties + tid);
    }
    select_token(a, r, row, vocab, inv_t, m, st.sum, st, true, a.uniforms ? words + kMeetWords : nullptr, sh);
  }
}

// One workgroup per row: small vocabularies, or no scratch.
__global__ __launch_bounds__(SAMP_T) void sample_kernel(SampleRows a, int vocab) {
  __shared__ SampShared sh;
  const int lane = threadIdx.x & 63, r = blockIdx.x;
  const float* row = a.logits + (long long)(a.logits_row ? a.logits_row[r] : r) * vocab;
  const float inv_t = row_inv_temp(a, r);
  const int n_seg = (vocab + 255) >> 8;
  const bool nucleus = row_has_nucleus(a, r, vocab);
  const RowTiles<0> tiles(row, vocab, 0, RowShares(vocab, 1));
  float m = -INFINITY;
  tiles.each([&](int, const Logit4& z) {
#pragma unroll
    for (int e = 0; e < 4; ++e) m = fmaxf(m, scaled_logit(z.v[e], inv_t));
  });
  m = block_max(m, sh);
  unsigned long long S;
  NucleusState st{};
  if (nucleus) {
    const float top_p = row_top_p(a, r);
    for (int level = 0; level < 3; ++level) {
      nucleus_histogram(tiles, inv_t, m, level, st.prefix, sh);
      nucleus_descend(nucleus_bin_from_top<false>(sh.hist, level), level, top_p, st, sh);
    }
    S = st.sum;
    nucleus_segments(tiles, inv_t, m, st.prefix, [&](int seg, unsigned long long above, unsigned n) {
      sh.hist[seg] = above;
      sh.ties[seg] = n;
    });
  } else {
    // all weights, one sum per segment
    unsigned long long local = 0;
    tiles.each([&](int i0, const Logit4& z) {
      const WeightParts mine = weight4(z, i0, vocab, inv_t, m);
      local += parts_sum(mine);
      const unsigned long long ws = wave_total_weights(mine);
      if (lane == 0 && i0 >> 8 < n_seg) sh.vals[i0 >> 8] = ws;
    });
    S = block_sum_u64(local, sh);  // also orders the writes to sh.vals
  }
  select_token(a, r, row, vocab, inv_t, m, S, st, nucleus, a.uniforms ? a.uniforms + r : nullptr, sh);
}

// Parts of a row: as many as give every CU one workgroup, of a nucleus at most one to a wavefront of the last part.  A part waits
// for the slowest, and a CU that holds two while others hold one is the slowest.  Only where a part's share gets long - more than 5
// tiles, 7 of a nucleus, whose phases end in more waits - two workgroups to every CU, that fill each other's gaps.
// us a call, back to back on a stream, one / two to a CU:
//                   top_p 0.9                                                top_p 1
//   32001 ids       42 rows 23.0 / 26.6, 128 rows 27.9 / 30.0                42 rows 11.5 / 13.5, 128 rows 14.2 / 15.2
//   65536 ids       64 rows 27.8 / 30.0, 80 rows 30.1 / 31.2, 88 rows 36.7 / 32.7    50 rows 13.1 / 14.5, 80 rows 16.2 / 16.0
//   151936 ids      42 rows 32.6 / 33.4, 50 rows 35.1 / 34.7, 64 rows 40.0 / 39.6    16 rows 12.4 / 13.8, 42 rows 18.1 / 16.9,
//                   88 rows 58.1 / 51.0                                              64 rows 24.7 / 23.1, 88 rows 39.5 / 31.8
// (the draw of a nucleus counts on that: a wavefront to a part's list)
static int sample_parts(int rows, int n_tiles, bool nucleus) {
  const int most = std::min(n_tiles, nucleus ? SAMP_T / WAVE : kSampleParts - 1);
  const int one = std::min(most, 256 / rows);
  if (one >= 2 && n_tiles <= one * (nucleus ? 7 : 5)) return one;
  return std::max(2, std::min(most, 512 / rows));
}

// Large vocabularies with scratch at hand: the sweeps of a row on several workgroups and two launches,
// the maximum and the rest; else everything in one workgroup per row.
// 64 rows x 151936 ids, top_p 0.9, in us (clock readings of the parts, averages): the maximum 8.0, a launch of its own; then 8.7 for
// histogram 0 (all weights: 35 instructions an id), 2.1 to meet, 7.2 for the sweep that lists (one id in eight is weighed), 1.0 to report
// and 8 for the draw, a chain of round trips and barriers (1.2 to fetch, 0.8 + 1.3 to find tau, 4.6 from there to the token); 6.6 go
// by because a part waits for its row's slowest.  Launches 8.0 + 35.3, 39.6 a call back to back.  No one thing bounds it: 39 MB of logits
// are read three times, at 6 us each from memory.
// In six launches (9.5 + 14.2 + 15.3 + 2.9 + 2.7 + 13.7, where two found nothing to do) 50.9; one row 27.2 -> 23.2, 64 flat rows
// (N(0, 0.2)) 80.9 -> 59.5, 64 rows without a nucleus 25.5 -> 23.1; one workgroup per row that searched tau bit by bit 1809.
static void launch_sample_rows(const SampleRows& r, int rows, int vocab, hipStream_t s, KernelTimer* timer) {
  auto timed = [&](const char* name, auto&& launch) {  // each reads all logits
    if (timer) timer->begin(name, 4.0 * rows * vocab, 0, s);
    launch();
    if (timer) timer->end(s);
  };
  const int n_tiles = (vocab + 4095) >> 12;
  int parts = 0;
  if (r.part_max && r.seg_sums && (r.nucleus || !r.any_nucleus) && n_tiles >= 8 && vocab <= 256 * kSampleSegments)
    parts = sample_parts(rows, n_tiles, r.any_nucleus);
  if (parts < 2) {
    timed("sample_kernel", [&] { sample_kernel<<<rows, SAMP_T, 0, s>>>(r, vocab); });
    return;
  }
  const dim3 grid(parts, rows);
  const RowShares in(vocab, parts);
  timed("sample_max_kernel", [&] { sample_max_kernel<<<grid, SAMP_T, 0, s>>>(r, vocab, in); });
  if (r.any_nucleus) timed("sample_rest_kernel<true>", [&] { sample_rest_kernel<true><<<grid, SAMP_T, 0, s>>>(r, vocab, in); });
  else timed("sample_rest_kernel<false>", [&] { sample_rest_kernel<false><<<grid, SAMP_T, 0, s>>>(r, vocab, in); });
}

void launch_sample(SampleRows r, int rows, int vocab, hipStream_t s, KernelTimer* timer) {
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
    launch_sample_rows(b, std::min(batch, rows - r0), vocab, s, timer);
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
