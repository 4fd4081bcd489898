// bf16 projections on the matrix cores: out[m][n] = sum_k a[m][k] w[n][k], fp32 accumulate.
//
// The decoding phase is memory-bound (paper section 2.1): with few live rows every
// projection is a stream over the weight matrix.  Weights are therefore re-ordered once,
// at load time, into the fragment order of the 16x16x32 bf16 matrix instruction
//     packed[n_tile][k_tile][lane][8],  lane = (k % 32 / 8) * 16 + n % 16
// so that a wavefront reads each 16-column x 32-deep weight fragment as one contiguous
// 1 KiB load straight into registers, and a whole row of fragments [n_tile][*] is one
// contiguous stream.  The instruction computes D = W_frag . A_frag^T, i.e. a tile of
// out^T, so each lane ends up with four consecutive output columns of one row.
//
// Activations keep near-fp32 precision through the bf16 instruction: every activation value v
// travels as two bf16 numbers, hi = bf16(v) and lo = bf16(v - hi) - side by side in blocks of 32
// (plane_offset) or, where the weights are streamed, as two planes in fragment order (frag_offset,
// kernels_fast.h) - and each weight fragment is multiplied with both (the weights themselves are bf16
// exactly, so nothing else is rounded).  That doubles the matrix instructions, which the
// memory-bound decode step does not notice.
//
// Two kernels:
//   gemm_stream_kernel  (rows <= 16, of models up to a hidden size of 2048 rows <= 32, decoding): the NW
//       wavefronts of a workgroup share MT row and NT column tiles and interleave over the K range in chunks of KU fragments, so one
//       workgroup walks one contiguous weight stream with up to 2 NW x KU x NT KiB in flight; the
//       partial accumulators meet in LDS.  Activations come straight from L2, stored in
//       fragment order by their producers (frag_offset, kernels_fast.h) so that an operand
//       fragment, like a weight fragment, is whole cache lines.  Narrow outputs (few column
//       tiles) use wide workgroups (16 wavefronts) or, where K is deep, splits that join in the launch
//       (join_splits), so every output element is complete inside one wavefront and the epilogue can
//       carry the neighbouring element-wise work:
//         - RMSNorm is split in two.  The producer of the residual stream (EPI_RESID) adds
//           its result to x, stores x * gain as the next projection's operand and one
//           partial sum of squares per (workgroup, row); the consumer sums those partials
//           in a fixed order (all its wavefronts share the loads) and scales its output rows
//           by rsqrt(mean + eps) - a row scale commutes with the projection.  No workgroup
//           ever waits for another.
//         - SwiGLU on column tiles of 8 gates and their 8 ups (EPI_SWIGLU_BF16).
//   gemm_tile_kernel    (more rows: larger decode steps, prefill, the teacher-forced
//       pass, the experts' grouped projections): output tiles of 32 x 64 up to 192 x 256, both
//       operands copied straight from memory into a ring of LDS stages.
#include <cstdio>
#include <utility>

#include "kernels_fast.h"
#include "tile_plan.h"

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

// a / (1 + e^-a).  Over all 2^32 operands the bits are those of the IEEE division; only for a < -87.3, where the
// reciprocal of more than 2^126 is flushed, 0 stands for results below 6e-37.  div_fixup is for infinite operands.
__device__ inline float silu_f(float a) {
  const float d = 1.0f + __expf(-a);
  return __builtin_amdgcn_div_fixupf(quotient(a, d, __builtin_amdgcn_rcpf(d)), d, a);
}

// D[n][m] tile of fp32 results -> memory.  lane (r, g) holds rows n = 4g..4g+3 of the tile at column m = r.
__device__ inline void store_tile_f32(const GemmArgs& p, int m, int nt, const f32x4& t, int g, int z) {
  float* out = (float*)p.out + (long long)z * p.split_stride + (long long)m * p.ldo;
  *(float4*)(out + nt * 16 + g * 4) = make_float4(t[0], t[1], t[2], t[3]);
}
// SwiGLU of the tiles nt and nt + 1 (`two`; else t1 is not used): columns 0..7 of a tile are gates, 8..15 their
// ups; act[m][f] = silu(gate) * up.  Lanes g < 2 hold gates and take tile nt, the others hold ups and take tile nt + 1:
// swapping the halves of the wavefront brings every lane both operands of its four f's.  A second swap, between
// neighbouring rows of 16 lanes, gathers eight f's hi (even g) or lo parts (odd g) for 16-byte stores.  All lanes of the
// wavefront call it; `valid`: row m is stored.
// What bounds it: instructions of a wavefront that has its SIMD to itself.  With exchanges through LDS, an IEEE division
// and the rounding in integers the epilogue was 4.5 us of the 55 us that 33 rows x 37888 x 3584 take.
template <bool TILE>  // the tile kernel's results are never in fragment order
__device__ inline void store_swiglu(const GemmArgs& p, bool valid, int m, int nt, const f32x4& t0, const f32x4& t1,
                                    int g, bool two) {
  float v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const auto gu = __builtin_amdgcn_permlane32_swap(__float_as_uint(t0[e]), __float_as_uint(t1[e]), false, false);
    v[e] = silu_f(__uint_as_float(gu[0])) * __uint_as_float(gu[1]);
  }
  uint2 hi, lo;
  split4_bf16(v[0], v[1], v[2], v[3], hi, lo);
  const auto x = __builtin_amdgcn_permlane16_swap(hi.x, lo.x, false, false);
  const auto y = __builtin_amdgcn_permlane16_swap(hi.y, lo.y, false, false);
  if (valid && (two || g < 2)) {
    const int f = (nt + (g >> 1)) * 8;
    uint16_t* out = (uint16_t*)p.out + (!TILE && p.frag ? frag_offset(m, f, p.ldo >> 5) : plane_offset(m, f, p.ldo));
    *(uint4*)(out + (g & 1 ? p.out_lo_offset : 0)) = make_uint4(x[0], y[0], x[1], y[1]);
  }
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// K splits joined inside their launch.  Every split's wavefront stores its partial tile, takes a ticket, and the one that
// takes the last ticket adds the others' parts to its own - in the order of the splits, so that the sum does not
// depend on who came last - and goes on with the epilogue; the others are done.
//   What makes the parts visible, since each XCD has its own L2: they are stored and loaded at the scope of the device (sc1:
//   through to the memory side, and past the L2), and the ticket is drawn only when the stores have been acknowledged.
//   No fence is needed, whose write-back of a whole L2 is what makes a join expensive: 96 column tiles x 8960, 8
//   rows, two splits 10.6 us as planes, 11.9 joined, four 7.6 and 9.1, where a second launch takes 4.
//   The last one sets the ticket back to 0 for the next launch.
// One wavefront's N quads per lane; `tile`: its index among the launch's joined tiles.  True in the last wavefront of
// the `splits`, whose t then holds the sum.
template <int N>
__device__ __forceinline__ bool join_splits(const GemmArgs& p, int tile, int split, int splits, f32x4 (&t)[N], int lane) {
  float* base = p.join + (long long)tile * splits * (N * 256);
  const __amdgpu_buffer_rsrc_t parts = __builtin_amdgcn_make_buffer_rsrc(base, 0, splits * N * 1024, 0x00027000);
#pragma unroll
  for (int q = 0; q < N; ++q)
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, t[q]), parts, lane * 16, (split * N + q) * 1024, kDeviceScope);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  unsigned* ticket = p.tickets + tile * kTicketStride;
  unsigned drawn = 0;
  if (lane == 0) drawn = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  drawn = __builtin_amdgcn_readfirstlane(drawn);
  if ((int)drawn != splits - 1) return false;
  asm volatile("" ::: "memory");  // the loads stay behind the ticket
  if (lane == 0) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
  for (int q = 0; q < N; ++q) t[q] = f32x4{0.f, 0.f, 0.f, 0.f};
  constexpr int ZB = N >= 4 ? 2 : 4;  // splits whose loads are in flight together
  for (int z = 0; z < splits; z += ZB) {
    u32x4 u[ZB][N];
#pragma unroll
    for (int i = 0; i < ZB; ++i)
#pragma unroll
      for (int q = 0; q < N; ++q)
        u[i][q] = __builtin_amdgcn_raw_buffer_load_b128(parts, lane * 16, (min(z + i, splits - 1) * N + q) * 1024, kDeviceScope);
#pragma unroll
    for (int i = 0; i < ZB; ++i)
      if (z + i < splits) {
#pragma unroll
        for (int q = 0; q < N; ++q) {
          const f32x4 v = __builtin_bit_cast(f32x4, u[i][q]);
          t[q][0] += v[0];
          t[q][1] += v[1];
          t[q][2] += v[2];
          t[q][3] += v[3];
        }
      }
  }
  return true;
}

// What bounds it: the weight stream from HBM (6.0 TB/s on this chip for one large read), plus about 3 us of
// launch and latency, plus the activations, which every workgroup reads in full through its CU's
// L2 path (about 60 GB/s): 64 K bytes of hi and lo parts beside 32 NT K bytes of weights.
//   - The weights are read once and bypass the caches' retention (non-temporal loads): they do not push the
//     activations out of L2.
//   - Two chunks of loads per wavefront: while one is multiplied, the next is in flight.
//   - Loads are not predicated: k-tiles, rows and columns past the end read the last valid one and are not
//     multiplied or stored.
// Measured (4 rows, weights from HBM): gate/up 7B shape (272 MB) 49.3 -> 43.1 us, down 7B (136 MB) 38.3 -> 26.8,
// gate/up 1.5B (55 MB) 14.1 -> 12.7.  Narrow outputs in K splits: beside gemm_plan_stream.
template <int MT, int NT, int KU, int NW, bool KEEP, int EPI>
__global__ __launch_bounds__(NW * 64) void gemm_stream_kernel(const void* pw, const void* pa, long long lo_off, const float* rinv_ssq,
                                                              int M, int N, int K, int k_tiles_per_split, int frag,
                                                              int rinv_partials, GemmArgs p) {
  static_assert(MT <= 2 && MT <= NW && (NT % 2 == 0 || EPI != EPI_SWIGLU_BF16), "a wavefront finishes a row tile, SwiGLU in pairs of column tiles");
  __shared__ float4 red[NW * MT * NT * 64];
  __shared__ float rs_part[MT * NW * 64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 15, g = lane >> 4;
  const int n_tiles = N >> 4, k_tiles = K >> 5;
  const int nt0 = blockIdx.x * NT;
  const int kt_begin = blockIdx.y * k_tiles_per_split;
  const int kt_end = min(k_tiles, kt_begin + k_tiles_per_split);

  const u32x4* w_src[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) w_src[j] = (const u32x4*)pw + (long long)min(nt0 + j, n_tiles - 1) * k_tiles * 64 + lane;
  // activation fragments of this lane: row m of each row tile, k = 8 g .. 8 g + 7 of k-tile 0; a k-tile further on is
  // a_step away
  const u32x4* a_src[MT];
  int rows[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    rows[i] = min((int)(blockIdx.z * MT + i) * 16 + r, M - 1);
    a_src[i] = (const u32x4*)((const uint16_t*)pa +
                              (frag ? frag_offset(rows[i], g * 8, k_tiles) : plane_offset(rows[i], g * 8, K)));
  }
  const int a_step = frag ? 64 : 8;

  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  u32x4 wf[2][KU][NT], af[2][KU][MT][2];
  auto load = [&](int kt, u32x4 (&w)[KU][NT], u32x4 (&a)[KU][MT][2]) {
#pragma unroll
    for (int kk = 0; kk < KU; ++kk)
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        const u32x4* at = w_src[j] + (long long)min(kt + kk, kt_end - 1) * 64;
        w[kk][j] = KEEP ? *at : __builtin_nontemporal_load(at);
      }
#pragma unroll
    for (int kk = 0; kk < KU; ++kk)
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const u32x4* at = a_src[i] + (long long)min(kt + kk, kt_end - 1) * a_step;
        a[kk][i][0] = at[0];
        a[kk][i][1] = at[lo_off];
      }
    __builtin_amdgcn_sched_barrier(0);  // all of a chunk's loads leave before the products of the other chunk
  };
  auto multiply = [&](int kt, const u32x4 (&w)[KU][NT], const u32x4 (&a)[KU][MT][2]) {
#pragma unroll
    for (int kk = 0; kk < KU; ++kk) {
      const bool on = kt + kk < kt_end;  // a k-tile past the end counts zero
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int plane = 1; plane >= 0; --plane) {  // lo part first, then hi
          const u32x4 x = on ? a[kk][i][plane] : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
          for (int j = 0; j < NT; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[kk][j]),
                                                                __builtin_bit_cast(bf16x8, x), acc[i][j], 0, 0, 0);
        }
    }
  };
  // This wavefront's chunks of KU k-tiles: wave, wave + NW, ...  The loop body has no branch: with one, the
  // compiler waits at every join for loads that only the other path has in flight.
  constexpr int STEP = NW * KU;
  int kt = kt_begin + wave * KU;
  const int chunks = kt < kt_end ? (kt_end - kt + STEP - 1) / STEP : 0;
  if (chunks > 0) load(kt, wf[0], af[0]);

  // The epilogue belongs to wavefront 0.  Its operands - the input rows' partial sums of squares, the
  // residual values and the gain - are requested behind the first weights and not waited for before the
  // end (loads return in order: ahead of the weights, they held the stream back by round trips to memory).
  // The sums of squares come as one partial per workgroup of the producing launch (hidden/16 of
  // them): every wavefront takes the partials w, w + NW, ... - a lane those of its group g, for
  // row r - so that no wavefront has more than a few of them; the shares meet in LDS with the
  // accumulators.
  constexpr int RS = EPI == EPI_RESID ? 0 : 8;  // the projections that add to the residual read no norm's input
  const int n_rs = rinv_ssq ? rinv_partials : 0;
  const float* rs_src = rinv_ssq ? rinv_ssq : (const float*)pa;
  float rs_of[MT][RS + 1];
#pragma unroll
  for (int q = 0; q < MT; ++q)
#pragma unroll
    for (int i = 0; i < RS; ++i)  // clamped here, masked where they are summed
      rs_of[q][i] = rs_src[(long long)max(min((i * NW + wave) * 4 + g, n_rs - 1), 0) * p.ssq_stride + (rinv_ssq ? rows[q] : 0)];
  const int own = MT > 1 ? min(wave, MT - 1) : 0;  // wavefront i < MT finishes row tile i
  const int m = (blockIdx.z * MT + own) * 16 + r, row = min(m, M - 1);
  float4 xv[NT], gn[NT];
  if (EPI == EPI_RESID) {
#pragma unroll
    for (int q = 0; q < NT; ++q) {
      const int n = min(nt0 + q, n_tiles - 1) * 16 + g * 4;
      xv[q] = *(const float4*)(p.x + (long long)row * N + n);
      gn[q] = *(const float4*)(p.gain + n);
    }
  }

  if (chunks > 0) {
    for (int left = chunks; left > 2; left -= 2) {
      load(kt + STEP, wf[1], af[1]);
      multiply(kt, wf[0], af[0]);
      load(kt + 2 * STEP, wf[0], af[0]);
      multiply(kt + STEP, wf[1], af[1]);
      kt += 2 * STEP;
    }
    if (chunks & 1) {
      multiply(kt, wf[0], af[0]);
    } else {
      load(kt + STEP, wf[1], af[1]);
      multiply(kt, wf[0], af[0]);
      multiply(kt + STEP, wf[1], af[1]);
    }
  }

  // the wavefronts' partial tiles meet in LDS
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
      red[((i * NW + wave) * NT + j) * 64 + lane] = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
  if constexpr (RS > 0) {
#pragma unroll
    for (int q = 0; q < MT; ++q) {
      float rs_share = 0.f;
#pragma unroll
      for (int i = 0; i < RS; ++i) rs_share += (i * NW + wave) * 4 + g < n_rs ? rs_of[q][i] : 0.f;
      for (int pp = (RS * NW + wave) * 4 + g; pp < n_rs; pp += NW * 4)  // hidden sizes beyond 512 NW
        rs_share += rs_src[(long long)pp * p.ssq_stride + rows[q]];
      rs_part[(q * NW + wave) * 64 + lane] = rs_share;
    }
  }
  __syncthreads();
  if (wave >= MT) return;
  const bool valid = m < M;
  f32x4 t[NT];
#pragma unroll
  for (int q = 0; q < NT; ++q) t[q] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < NT; ++q)
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float4 v = red[((own * NW + w) * NT + q) * 64 + lane];
      t[q][0] += v.x;
      t[q][1] += v.y;
      t[q][2] += v.z;
      t[q][3] += v.w;
    }
  if constexpr (EPI == EPI_RESID) {
    if (gridDim.y > 1 && !join_splits(p, (blockIdx.z * MT + own) * gridDim.x + blockIdx.x, blockIdx.y, gridDim.y, t, lane)) return;
  }
  if (RS > 0 && rinv_ssq) {
    // second half of the RMSNorm of this projection's input: scale row m by
    // rsqrt(mean(x^2) + eps); the 4 lanes of a row share the partial sums
    float rs = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) rs += rs_part[(own * NW + w) * 64 + lane];
    rs += __shfl_xor(rs, 16, WAVE);
    rs += __shfl_xor(rs, 32, WAVE);
    const float rinv = 1.0f / sqrtf(rs / (float)K + p.eps);
#pragma unroll
    for (int q = 0; q < NT; ++q) {
      t[q][0] *= rinv;
      t[q][1] *= rinv;
      t[q][2] *= rinv;
      t[q][3] *= rinv;
    }
  }
  if (EPI == EPI_RESID) {
    float ss = 0.f;
#pragma unroll
    for (int q = 0; q < NT; ++q)
      if (valid && nt0 + q < n_tiles) {
        const int n = (nt0 + q) * 16 + g * 4;
        float4 x4 = xv[q];
        x4.x += t[q][0];
        x4.y += t[q][1];
        x4.z += t[q][2];
        x4.w += t[q][3];
        *(float4*)(p.x + (long long)m * N + n) = x4;
        ss += x4.x * x4.x + x4.y * x4.y + x4.z * x4.z + x4.w * x4.w;
        uint2 hi, lo;
        split4_bf16(x4.x * gn[q].x, x4.y * gn[q].y, x4.z * gn[q].z, x4.w * gn[q].w, hi, lo);
        uint16_t* hp = p.h + (frag ? frag_offset(m, n, n_tiles >> 1) : plane_offset(m, n, N));
        *(uint2*)hp = hi;
        *(uint2*)(hp + p.h_lo_offset) = lo;
      }
    ss += __shfl_xor(ss, 16, WAVE);
    ss += __shfl_xor(ss, 32, WAVE);
    if (g == 0 && valid) p.ssq_out[(long long)blockIdx.x * p.ssq_stride + m] = ss;
  } else if constexpr (EPI == EPI_SWIGLU_BF16) {
#pragma unroll
    for (int q = 0; q < NT; q += 2)
      if (nt0 + q < n_tiles) store_swiglu<false>(p, valid, m, nt0 + q, t[q], t[q + 1], g, nt0 + q + 1 < n_tiles);
  } else if (valid) {
#pragma unroll
    for (int q = 0; q < NT; ++q)
      if (nt0 + q < n_tiles) store_tile_f32(p, m, nt0 + q, t[q], g, blockIdx.y);
  }
}

// ------------------------------------------------------------------------------------------
// Tile kernel.  A workgroup computes BM = 16 WM MT rows x BN = 16 WN NT columns; its WM x WN
// wavefronts each own MT x NT tiles of 16 x 16, and with KG = 2 two such groups of wavefronts take
// alternate k-tiles and join their sums through LDS at the end (twice the wavefronts on a tile
// whose size the chip's 256 CUs ask for).
//
// What bounds it.  Long launches with many rows: the power limit.  On zeros the 192 x 256 tiles issue 1.9 PFLOP/s, on
// real data 1.4 to 1.6 (box to box), whatever the tile's shape; so what counts is what a product costs beside itself:
//   - Of each product the lo and the hi part run one after the other, on the same sums: from registers alone 2.0 -> 2.2
//     PFLOP/s, here 1 to 2.5 %.  (32 x 32 products: 1.75 from registers.)
//   - Wide wavefronts: 96 x 128 of a 192 x 256 tile in each of four wavefronts, with a SIMD's registers to itself, instead of 48 x 128
//     in eight reads 20 KB from LDS for 96 products instead of 28.  10568 rows x 3584 x 18944 2.35 -> 2.23 ms (128 x 320 and
//     160 x 256), 2600 x 3584 x 18944 577 -> 540 us, 4600 x 2048 x 1536 53 -> 48; 10568 x 37888 x 3584 4.02 -> 3.94 ms.
// A few hundred rows: wavefronts that have their SIMD
// almost to themselves, where every wait shows.  Decode steps: the weights, and besides them, per k-tile, 128 BM +
// 64 BN bytes through the CU for BM BN / 256 tiles, so wide tiles win, and one round of workgroups that fills all CUs wins
// over a second, mostly empty one: the plan below weighs the two.
//
// Both operands go from memory straight into LDS (global_load_lds_dwordx4, 1 KiB per instruction), S stages ahead, with
// one barrier per stage.  The fragments of stage s + 1 are read between the products of stage s, and the copies of
// stage s + S are issued there too:
//   - A wavefront waits until its own copies of stage s + 1 have arrived (s_waitcnt vmcnt counts in
//     order: the copies of the S - 2 later stages may be outstanding) and its fragments of stage s are in registers
//     (lgkmcnt); then the barrier says the same of every wavefront.  So after it stage s + 1 can be read and the
//     buffer of stage s be overwritten.
//   - The last stage's products stand outside the loop, which therefore has no branch.  Past the end of the K range
//     the last k-tile is copied and read again (never multiplied), so that every stage counts the same number of copies.
// Activations: one instruction brings 8 rows x 128 bytes, a line holding both planes of 32 elements
// (plane_offset).  The 16-byte chunk c of row r lands in slot c ^ (r % 8) of its row, by choosing
// each lane's source address, which makes the fragment reads conflict-free.  Weights: a fragment is
// one instruction and is read back as it lies.  Rows and column tiles past the end read the last
// valid one; their results are not stored.
//
// Measured against the kernel before, which read a stage's fragments after its barrier (back to back, weights from
// HBM, splits' planes included): 24 rows x 37888 x 3584 64 -> 48 us, 24 x 3584 x 18944 34 -> 26, 64 x 1536 x 8960 10.9 ->
// 10.1, 256 x 37888 x 3584 125 -> 105, 512 x 37888 x 3584 229 -> 206, 1700 x 3584 x 18944 373 -> 336, 6000 x 37888 x 3584
// 2.35 -> 2.18 ms (1.5 PFLOP/s issued).
// 16 bytes per lane from base + voff to LDS byte `lds` + 16 * lane.  (The compiler keeps nothing in m0: it sets it
// right before each instruction of its own that reads it.)  As inline assembly, because the compiler makes every
// LDS read wait for all copies into LDS that it knows of.
__device__ __forceinline__ void load_to_lds(unsigned lds, unsigned voff, const void* base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(base)
               : "memory");
}
// the same with a 64-bit address per lane
__device__ __forceinline__ void load_to_lds(unsigned lds, const void* addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(addr) : "memory");
}
// this wavefront's loads but the last N have arrived and its LDS reads are done; then the barrier
template <int N>
__device__ __forceinline__ void wait_and_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// f(0), ..., f(N - 1) with the index as a constant
template <class F, int... I>
__device__ __forceinline__ void unrolled(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}

// GATHER: the rows of `a` come through row_map (experts' grouped projections)
template <int WM, int WN, int MT, int NT, int KG, int S, int EPI, bool GATHER>
__global__ __launch_bounds__(WM* WN* KG * 64, wide_wavefronts(WM, WN, MT, NT, KG, S) ? 1 : 2) void gemm_tile_kernel(
    const void* pw, const void* pa, int M, int N, int K, int k_tiles_per_split, unsigned group, int gy, unsigned by_per,
    unsigned by_nz, unsigned by_gy, unsigned by_m, GemmArgs p) {
  constexpr bool WIDE = wide_wavefronts(WM, WN, MT, NT, KG, S);
  constexpr int NW = WM * WN * KG, BM = WM * MT * 16, BN = WN * NT * 16;
  constexpr int UA = BM / 8, UW = BN / 16, U1 = UA + UW;  // load instructions per k-tile
  constexpr int L = (U1 * KG + NW - 1) / NW;              // per wavefront and stage
  constexpr int RED = KG > 1 ? (KG - 1) * WM * WN * MT * NT : 0;
  constexpr int LDS_KB = S * U1 * KG > RED ? S * U1 * KG : RED;
  static_assert(LDS_KB <= 160 && S >= 2 && KG <= 2 && (S - 1) * L < 64, "fits the CU and the load counter");
  __shared__ __attribute__((aligned(1024))) char lds[LDS_KB * 1024];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 15, g = lane >> 4;
  const int n_tiles = N >> 4, k_tiles = K >> 5;
  TileGrid grid;
  grid.nx = (n_tiles + WN * NT - 1) / (WN * NT);
  grid.nz = (int)(group >> 16);
  grid.group_m = (int)(group & 255);
  grid.group_n = (int)(group >> 8 & 127);
  const bool grouped = group >> 15 & 1;
  grid.ny = grouped ? p.grid.ny : (M + BM - 1) / BM;
  grid.gy = gy;
  grid.by_per = by_per;
  grid.by_nz = by_nz;
  grid.by_gy = by_gy;
  grid.by_m = by_m;
  const TileBlock block = tile_block(grid, blockIdx.x);
  if (!block.inside) return;  // uniform
  const int bx = block.x, by = block.y, bz = block.z;
  const int nt0 = bx * (BN / 16);
  int m0 = by * BM;
  const int kt_begin = bz * k_tiles_per_split;
  const int kt_end = min(k_tiles, kt_begin + k_tiles_per_split);

  // grouped (per-expert) launches: this row block belongs to one group with its own weights
  const char* wp = (const char*)pw;
  int m_limit = M;
  if (grouped) {
    wp += (long long)p.group_of_block[by] * p.group_stride16 * 16;
    m0 = p.block_row_begin[by];
    m_limit = p.block_row_end[by];
    if (m0 >= m_limit) return;  // unused block of the plan (uniform over the workgroup)
  }
  wp += (long long)nt0 * k_tiles * 1024;
  const long long row_bytes = (long long)K * 4;
  const char* ap = (const char*)pa + (GATHER ? 0 : m0 * row_bytes);

  const int kg = wave / (WM * WN), wm = wave % (WM * WN) / WN, wn = wave % WN;
  // this wavefront's loads of a stage: instruction u of the stage's U1 * KG.  An address moves on by a stage's k-tiles
  // as long as there is one to load; then it stays.
  unsigned voff[L], step[L], dst[L];
  int k_of[L];
  const char* base[L];
  const char* row_addr[L];
#pragma unroll
  for (int s = 0; s < L; ++s) {
    const int uu = min(s * NW + wave, U1 * KG - 1);  // an uneven last round loads the last one again
    const int u = __builtin_amdgcn_readfirstlane(uu % U1);
    k_of[s] = __builtin_amdgcn_readfirstlane(uu / U1);
    dst[s] = __builtin_amdgcn_readfirstlane(uu * 1024);
    const unsigned k0 = min(kt_begin + k_of[s], kt_end - 1);
    if (u < UA) {
      const int m = min(m0 + u * 8 + (lane >> 3), m_limit - 1);
      const unsigned chunk = ((lane & 7) ^ (lane >> 3)) * 16;
      if (GATHER) row_addr[s] = ap + p.row_map[m] * row_bytes + chunk + k0 * 128;
      else voff[s] = (unsigned)((m - m0) * row_bytes) + chunk + k0 * 128;
      step[s] = 128;
      base[s] = ap;
    } else {
      voff[s] = (unsigned)(min(nt0 + u - UA, n_tiles - 1) - nt0) * (unsigned)k_tiles * 1024u + lane * 16 + k0 * 1024;
      step[s] = 1024;
      base[s] = wp;
    }
  }
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)lds;
  auto issue = [&](int s, int kt, int buf) __attribute__((always_inline)) {  // load s of the stage that starts at k-tile kt
    const unsigned to = __builtin_amdgcn_readfirstlane(lds0 + buf * (U1 * KG * 1024) + dst[s]);
    const unsigned move = kt + KG + k_of[s] < kt_end ? KG * step[s] : 0u;
    if (GATHER && step[s] == 128) {
      load_to_lds(to, row_addr[s]);
      row_addr[s] += move;
    } else {
      load_to_lds(to, voff[s], base[s]);
      voff[s] += move;
    }
  };
  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < S; ++q)
#pragma unroll
    for (int s = 0; s < L; ++s) issue(s, kt_begin + q * KG, q);

  // fragment reads: row tile i of this wavefront is row groups 2 i and 2 i + 1 (8 rows, 1 KiB each)
  const int a_row = kg * U1 * 1024 + (wm * MT * 2 + (r >> 3)) * 1024 + (r & 7) * 128;
  const int a_hi = a_row + (g ^ (r & 7)) * 16, a_lo = a_row + ((4 + g) ^ (r & 7)) * 16;
  const int w_at = kg * U1 * 1024 + (UA + wn * NT) * 1024 + lane * 16;
  u32x4 w[2][NT], a[2][MT][2];
  constexpr int NR = NT + 2 * MT, NM = MT * NT * 2, NS = NR + L;
  auto read = [&](int x, const char* b, int f) __attribute__((always_inline)) {  // fragment f of a stage, in the order in which they are multiplied
    if (f < 2) a[x][0][1 - f] = *(const u32x4*)(b + (f ? a_hi : a_lo));
    else if (f < 2 + NT) w[x][f - 2] = *(const u32x4*)(b + w_at + (f - 2) * 1024);
    else a[x][(f - NT) >> 1][1 - ((f - NT) & 1)] = *(const u32x4*)(b + ((f - NT) & 1 ? a_hi : a_lo) + ((f - NT) >> 1) * 2048);
  };
  auto mul = [&](int x, int q) __attribute__((always_inline)) {  // row tile by row tile; of each product the lo part, then the hi part
    const int i = q / (2 * NT), plane = 1 - q % 2, j = q / 2 % NT;
    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[x][j]),
                                                        __builtin_bit_cast(bf16x8, a[x][i][plane]), acc[i][j], 0, 0, 0);
  };
  // With a SIMD's registers to itself a wavefront keeps its sums in the accumulation registers.  Left alone, the compiler
  // moves them back and forth between the stages (90 moves each way in two stages of 96 products): it has to
  // have them there at the end of each.
  auto keep_sums = [&]() __attribute__((always_inline)) {
    if constexpr (WIDE) {
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) asm volatile("" : "+a"(acc[i][j]));
    }
  };
  keep_sums();
  wait_and_barrier<(S - 1) * L>();
#pragma unroll
  for (int f = 0; f < NR; ++f) read(0, lds, f);
  int buf = 0;
  auto stage = [&](int x, int kt) __attribute__((always_inline)) {
    wait_and_barrier<(S - 2) * L>();
    const int next = buf == S - 1 ? 0 : buf + 1;
    const char* b = lds + next * (U1 * KG * 1024);
    unrolled([&](auto qc) __attribute__((always_inline)) {
      constexpr int q = decltype(qc)::value, u0 = (q * NS + NM - 1) / NM, u1 = ((q + 1) * NS + NM - 1) / NM;
      mul(x, q);
#pragma unroll
      for (int u = u0; u < u1; ++u) {
        if (u < NR) read(x ^ 1, b, u);
        else issue(u - NR, kt + S * KG, buf);
      }
      __builtin_amdgcn_sched_barrier(0);
    }, std::make_integer_sequence<int, NM>{});
    keep_sums();
    buf = next;
  };
  auto last = [&](int x, int kt) __attribute__((always_inline)) {
    if (KG > 1 && kt + kg >= kt_end) return;  // an odd last k-tile belongs to the first group
    unrolled([&](auto qc) __attribute__((always_inline)) { mul(x, decltype(qc)::value); }, std::make_integer_sequence<int, NM>{});
    keep_sums();
  };
  int kt = kt_begin, left = (kt_end - kt_begin + KG - 1) / KG;
  for (; left > 2; left -= 2) {
    stage(0, kt);
    stage(1, kt + KG);
    kt += 2 * KG;
  }
  if (left == 2) {
    stage(0, kt);
    last(1, kt + KG);
  } else {
    last(0, kt);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing may still be on its way into LDS
  if constexpr (KG > 1) {
    __syncthreads();
    float4* red = (float4*)lds + (wave % (WM * WN)) * (MT * NT * 64) + lane;
    if (kg > 0) {
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
          red[(i * NT + j) * 64] = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
    }
    __syncthreads();
    if (kg == 0) {
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          const float4 v = red[(i * NT + j) * 64];
          acc[i][j][0] += v.x;
          acc[i][j][1] += v.y;
          acc[i][j][2] += v.z;
          acc[i][j][3] += v.w;
        }
    }
  }
  const int wt0 = nt0 + wn * NT;  // this wavefront's first column tile
  if constexpr (EPI == EPI_LSE) {
    // log-sum-exp parts of this workgroup's columns: per wavefront over its NT tiles (the 4
    // lanes of a row meet by shuffles), then over the WN wavefronts of a row through LDS
    __syncthreads();
    float* part = (float*)lds;  // [2][WN][BM]: max, sum
    if (kg == 0) {
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const int ml = (wm * MT + i) * 16 + r, m = m0 + ml;
        const int tgt = m < m_limit ? p.lse_target[m] : -1;
        float mx = -INFINITY;
#pragma unroll
        for (int j = 0; j < NT; ++j)
          if (wt0 + j < n_tiles) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              acc[i][j][e] *= p.lse_scale;
              mx = fmaxf(mx, acc[i][j][e]);
              if ((wt0 + j) * 16 + g * 4 + e == tgt) p.lse_tgt[m] = acc[i][j][e];
            }
          }
        mx = fmaxf(mx, __shfl_xor(mx, 16, WAVE));
        mx = fmaxf(mx, __shfl_xor(mx, 32, WAVE));
        float sm = 0.f;
#pragma unroll
        for (int j = 0; j < NT; ++j)
          if (wt0 + j < n_tiles) {
#pragma unroll
            for (int e = 0; e < 4; ++e) sm += expf(acc[i][j][e] - mx);
          }
        sm += __shfl_xor(sm, 16, WAVE);
        sm += __shfl_xor(sm, 32, WAVE);
        if (g == 0) {
          part[wn * BM + ml] = mx;
          part[(WN + wn) * BM + ml] = sm;
        }
      }
    }
    __syncthreads();
    for (int ml = threadIdx.x; ml < BM; ml += NW * 64) {
      if (m0 + ml >= m_limit) continue;
      float mx = -INFINITY;
#pragma unroll
      for (int w = 0; w < WN; ++w) mx = fmaxf(mx, part[w * BM + ml]);
      float sm = 0.f;
#pragma unroll
      for (int w = 0; w < WN; ++w)
        if (part[w * BM + ml] > -INFINITY) sm += part[(WN + w) * BM + ml] * expf(part[w * BM + ml] - mx);
      p.lse_max[(long long)bx * p.lse_stride + m0 + ml] = mx;
      p.lse_sum[(long long)bx * p.lse_stride + m0 + ml] = sm;
    }
    return;
  } else {
    if (kg > 0) return;
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const int m = m0 + (wm * MT + i) * 16 + r;
      if constexpr (EPI == EPI_SWIGLU_BF16) {
#pragma unroll
        for (int j = 0; j < NT; j += 2)
          if (wt0 + j < n_tiles)
            store_swiglu<true>(p, m < m_limit, m, wt0 + j, acc[i][j], acc[i][j + 1 < NT ? j + 1 : j], g,
                         j + 1 < NT && wt0 + j + 1 < n_tiles);
      } else {
#pragma unroll
        for (int j = 0; j < NT; ++j)
          if (wt0 + j < n_tiles && m < m_limit) store_tile_f32(p, m, wt0 + j, acc[i][j], g, bz);
      }
    }
  }
}

// ------------------------------------------------------------------------------------------
static GemmPlan gemm_plan_tiled(int M, int N, int K, int epi, int max_splits) {
  static thread_local TilePlans plans;
  const TileChoice pick = plans(TileAsk{M, N, K, epi == EPI_F32 ? max_splits : 1, epi == EPI_LSE ? kLseMinTile : 0});
  const TileShape& t = kTileShapes[pick.shape];
  GemmPlan pl{};
  pl.kind = 1;
  pl.shape = pick.shape;
  pl.nt = t.wn * t.nt;
  pl.splits = pick.splits;
  pl.name = t.name[epi == EPI_F32 ? 0 : epi == EPI_SWIGLU_BF16 ? 1 : 2];
  return pl;
}

// The grouped (per-expert) launches.  Few picks: the launch is a stream over the touched experts' weights, and more,
// narrower workgroups have more of it in flight; many picks: wide tiles, which use every fragment for more products.
// Whole decode steps (s) and packed passes of the 30B-A3B shape, 12 layers, 128 experts, by picks per expert; ms with
// 32 x 64 / 32 x 128 / 32 x 192 / 64 x 128 / 64 x 192 / 64 x 256 / 128 x 128 / 128 x 256:
//   s  0.5:  1.07  1.18  1.17  1.25  1.27  1.36                 s  4.0:  1.57  1.45  1.57  1.60  1.57  1.60
//   s  2.0:  1.26  1.36  1.33  1.40  1.42  1.47                    3.8:  1.60  1.59  1.66  1.67  1.75  1.85
//   s  6.0:  1.65  1.54  1.65  1.65  1.74  1.81  1.74  1.86        7.5:  2.06  1.95  1.90  1.96  1.98  2.05  2.36  2.21
//   s  8.0:  1.79  1.79  1.73  1.75  1.87  2.02  1.84  1.96       11.7:  2.41  2.25  2.24  2.34  2.27  2.29  2.85  2.75
//   s   16:  2.65  2.41  2.43  2.42  2.29  2.38  2.68  2.47       21.9:  3.74  3.33  3.26  3.26  3.25  3.21  3.75  3.74
//       31:  4.74  4.24  4.13  4.07  3.96  3.97  4.87  4.62       62.5:  8.18  6.96  6.67  6.77  6.35  6.13  7.23  6.69
//      188:  21.1  17.1  16.2  16.1  14.8  14.0  16.0  14.4        562:                    45.0  41.3  40.0  44.3  40.1
// (before, blocks of 32, 64 or 128 rows x 128 columns and the kernel before: s 0.5 1.23, s 2.0 1.51, s 16 2.67, 31 4.31,
// 188 16.2, 562 45.0)
GemmPlan gemm_plan_grouped(int epi, long long picks, int n_experts) {
  GemmPlan pl{};
  pl.kind = 1;
  pl.shape = picks <= 3ll * n_experts ? 0 : picks <= 7ll * n_experts ? 1 : picks <= 14ll * n_experts ? 2 : picks <= 20ll * n_experts ? 7 : 8;
  const TileShape& t = kTileShapes[pl.shape];
  pl.nt = t.wn * t.nt;
  pl.splits = 1;
  pl.name = t.name[epi == EPI_F32 ? 0 : 3];  // the gate/up launch gathers its rows
  return pl;
}

#define TILE_ARGS a.w, a.a, a.M, a.N, a.K, a.k_tiles_per_split, group, a.grid.gy, a.grid.by_per, a.grid.by_nz, a.grid.by_gy, a.grid.by_m, a
static int launch_tile(GemmArgs a, int epi, const GemmPlan& pl, hipStream_t s) {
  const TileShape& t = kTileShapes[pl.shape];
  const int n_tiles = a.N >> 4, k_tiles = a.K >> 5, bm = t.wm * t.mt * 16;
  a.k_tiles_per_split = ceil_div(k_tiles, epi == EPI_F32 ? pl.splits : 1);
  a.grid.nz = ceil_div(k_tiles, a.k_tiles_per_split);
  a.grid.nx = ceil_div(n_tiles, pl.nt);
  a.grid.ny = a.group_of_block ? a.n_row_blocks : ceil_div(a.M, bm);
  if (a.group_of_block) tile_groups_experts(a.grid);
  else tile_groups(a.grid);
  tile_divisors(a.grid);
  const dim3 grid((unsigned)tile_workgroups(a.grid));
  const unsigned group = (unsigned)a.grid.group_m | (unsigned)a.grid.group_n << 8 | (a.group_of_block ? 1u << 15 : 0u) | (unsigned)a.grid.nz << 16;
  const bool gather = a.row_map != nullptr;
  switch (pl.shape) {
#define X(id, wm, wn, mt, nt, kg, st, ...)                                                                          \
  case id:                                                                                                           \
    if (epi == EPI_F32) gemm_tile_kernel<wm, wn, mt, nt, kg, st, EPI_F32, false><<<grid, wm * wn * kg * 64, 0, s>>>(TILE_ARGS); \
    else if (epi == EPI_LSE) /* never planned with fewer than kLseMinTile column tiles */                             \
      gemm_tile_kernel<wm, wn, mt, nt, kg, st, wn * nt >= kLseMinTile ? EPI_LSE : EPI_F32, false><<<grid, wm * wn * kg * 64, 0, s>>>(TILE_ARGS); \
    else if (grouped_shape(id) && gather)                                                                             \
      gemm_tile_kernel<wm, wn, mt, nt, kg, st, EPI_SWIGLU_BF16, grouped_shape(id)><<<grid, wm * wn * kg * 64, 0, s>>>(TILE_ARGS); \
    else gemm_tile_kernel<wm, wn, mt, nt, kg, st, EPI_SWIGLU_BF16, false><<<grid, wm * wn * kg * 64, 0, s>>>(TILE_ARGS); \
    break;
    TILE_SHAPES(X)
#undef X
  }
  return a.grid.nz;
}

// Narrow outputs are bound by what one CU can fetch, 65 to 90 GB/s: (64 MT + 32 NT) K bytes per workgroup, and as many
// workgroups as there are column blocks.  So the K range is cut until the CUs are full: where the splits' planes are
// summed by the next launch anyway (max_splits > 1: attention sums those of q, k, v), or joined in the launch
// (EPI_RESID), which costs about 1.5 us.  One workgroup more than 256 is another round: that is what the
// plan weighs (stream_plan.h).  us with weights from HBM, 6 / 16 / 32 rows, in one piece and in splits:
//   1536 x 8960    12.7 / 16.4 / 15.6  ->   8.7 /  9.4 / 11.0  (two column tiles, 5 splits)
//   1536 x 1536     4.6 /  5.2 /  5.2  ->   5.1 /  5.3 /  6.0  (4 splits): left in one piece
//   2048 x 1536     4.6 /  5.2 /  5.1  ->   3.8 /  3.9 /  4.7  (4 planes)
//   6144 x 2048     6.8 /  7.5 /  9.1  ->   8.0 /  8.6 / 10.4  (2 planes, 384 workgroups): left in one piece
//   3584 x 18944   26.9 / 34.4 (4 / 12 rows) -> 24.9 / 28.2 with two column tiles and 2 splits, 25.9 / 27.0 with four and 4
//   3584 x 3584     7.5 /  9.1 (4 / 12 rows) ->  8.1 /  8.8 (2 splits)
//   4096 x 4096     8.4 /  9.9 (4 / 12 rows) ->  9.6 / 10.0 (2 splits): left in one piece
//   4608 x 3584     9.2 / 11.0 (4 / 12 rows) ->  9.1 /  9.9 (3 planes)
GemmPlan gemm_plan_stream(int M, int N, int K, int epi, int max_splits) {
  const StreamChoice pick = epi == EPI_SWIGLU_BF16 ? StreamChoice{M > 16 ? 5 : 0, 1} : stream_choose(M, N, K, epi == EPI_RESID, max_splits);
  GemmPlan pl{};
  pl.kind = 0;
  pl.shape = pick.shape;
  pl.splits = pick.splits;
  pl.nt = kStreamShapes[pl.shape].nt;
  pl.name = kStreamShapes[pl.shape].name[epi];
  return pl;
}

GemmPlan gemm_plan(int M, int N, int K, int epi, int max_splits) {
  return M > 16 || epi == EPI_LSE ? gemm_plan_tiled(M, N, K, epi, max_splits) : gemm_plan_stream(M, N, K, epi, max_splits);
}

#define STREAM_ARGS a.w, a.a, lo_off, a.rinv_ssq, a.M, a.N, a.K, a.k_tiles_per_split, (int)a.frag, a.rinv_partials, a
static int launch_stream(GemmArgs a, int epi, const GemmPlan& pl, hipStream_t s) {
  const StreamShape& t = kStreamShapes[pl.shape];
  const int n_tiles = a.N >> 4, k_tiles = a.K >> 5;
  const long long lo_off = ((const uint16_t*)a.a_lo - (const uint16_t*)a.a) >> 3;  // 16-byte pieces
  a.k_tiles_per_split = ceil_div(k_tiles, pl.splits);
  const dim3 grid(ceil_div(n_tiles, t.nt), ceil_div(k_tiles, a.k_tiles_per_split), ceil_div(a.M, 16 * t.mt));
  if (epi == EPI_RESID && grid.y > 1 && (!a.join || (int)(grid.x * grid.z) * t.mt > kJoinTiles || (int)grid.y * t.nt > kJoinParts))
    throw HipError(hipErrorInvalidValue, "joined projection", __FILE__, __LINE__);
  switch (pl.shape) {
#define X(id, mt, nt, ku, nw, keep, e0, e1, ...)                                                      \
  case id:                                                                                         \
    if (epi == e0) gemm_stream_kernel<mt, nt, ku, nw, keep, e0><<<grid, nw * 64, 0, s>>>(STREAM_ARGS);        \
    else if (epi == e1) gemm_stream_kernel<mt, nt, ku, nw, keep, e1><<<grid, nw * 64, 0, s>>>(STREAM_ARGS);   \
    else throw HipError(hipErrorInvalidValue, "streamed projection", __FILE__, __LINE__);              \
    break;
    STREAM_SHAPES(X)
#undef X
  }
  return (int)grid.y;
}

int launch_gemm_bf16(GemmArgs a, int epi, const GemmPlan& pl, hipStream_t s) {
  if (a.M < 1 || a.N < 16) return 0;
  return pl.kind == 1 ? launch_tile(a, epi, pl, s) : launch_stream(a, epi, pl, s);
}

// ---------------------------------------------------------------- log-prob from the parts
// Parts are [part][row].  A workgroup takes 16 rows, 64 threads share a row's parts (a vocabulary of 150000 has
// about 600 or 1200): latency is all there is to it, and so it is divided.  1543 rows x 594 parts: 282 us
// with one thread per row; now below 15 us.
struct LseSum {
  float m, s;  // maximum, and the sum of exp(x - m)
};
__device__ inline LseSum join(const LseSum& a, const LseSum& b) {
  const float m = fmaxf(a.m, b.m);
  if (m == -INFINITY) return LseSum{m, 0.f};
  return LseSum{m, a.s * expf(a.m - m) + b.s * expf(b.m - m)};
}
__global__ __launch_bounds__(1024) void lse_finish_kernel(const float* __restrict__ lse_max,
                                                          const float* __restrict__ lse_sum,
                                                          const float* __restrict__ lse_tgt,
                                                          const int* __restrict__ target, int parts, int stride,
                                                          int rows, float* __restrict__ out) {
  __shared__ LseSum wave_s[16][16];
  const int tid = threadIdx.x, row = tid & 15, lane = tid & 63, wave = tid >> 6;
  const int r = blockIdx.x * 16 + row, rr = min(r, rows - 1);
  LseSum acc{-INFINITY, 0.f};
  for (int q0 = tid >> 4; q0 < parts; q0 += 4 * 64) {
    LseSum v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int q = q0 + 64 * e;
      const long long at = (long long)min(q, parts - 1) * stride + rr;
      v[e] = LseSum{lse_max[at], lse_sum[at]};
      if (q >= parts) v[e] = LseSum{-INFINITY, 0.f};
    }
    acc = join(acc, join(join(v[0], v[1]), join(v[2], v[3])));
  }
#pragma unroll
  for (int o = 16; o < WAVE; o <<= 1) acc = join(acc, LseSum{__shfl_xor(acc.m, o, WAVE), __shfl_xor(acc.s, o, WAVE)});
  if (lane < 16) wave_s[wave][row] = acc;
  __syncthreads();
  if (tid >= 16 || r >= rows) return;
  for (int w = 1; w < 16; ++w) acc = join(acc, wave_s[w][row]);
  out[r] = target[r] < 0 ? 0.f : lse_tgt[r] - acc.m - logf(acc.s);
}
void launch_lse_finish(const float* lse_max, const float* lse_sum, const float* lse_tgt, const int* target,
                       int parts, int stride, int rows, float* out, hipStream_t s) {
  if (rows) lse_finish_kernel<<<ceil_div(rows, 16), 1024, 0, s>>>(lse_max, lse_sum, lse_tgt, target, parts, stride, rows, out);
}

// ---------------------------------------------------------------- weight re-ordering
// Rows of src [N][K] (row-major bf16) -> fragments; `half` as in launch_pack_weight.
// A wavefront moves 8 rows x 128 bytes - two k-tiles of half a row tile - so that both its
// reads and its writes are whole cache lines (lane = row * 8 + chunk; chunk = k-tile * 4 +
// column group; the 8 rows of one chunk land in 8 consecutive 16-byte slots of a fragment).
// An odd last k-tile is moved as 16 rows x 64 bytes by the first 64 lanes' worth of pieces.
__global__ void pack_weight_kernel(const uint16_t* __restrict__ src, uint4* __restrict__ dst, int N, int K,
                                   int tile_offset, int half) {
  const int k_tiles = K >> 5, k_pairs = k_tiles >> 1;
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;  // one 16-byte piece each
  const long long paired = (long long)(N >> 4) * k_pairs * 128;
  int n, kt, g;  // source row, k-tile, column group
  if (idx < paired) {
    const int lane = (int)(idx & 63), chunk = lane & 7;
    const long long t = idx >> 7;
    n = (int)(t / k_pairs) * 16 + (int)((idx >> 6) & 1) * 8 + (lane >> 3);
    kt = 2 * (int)(t % k_pairs) + (chunk >> 2);
    g = chunk & 3;
  } else {
    if (!(k_tiles & 1)) return;
    const long long rest = idx - paired;  // the odd last k-tile of every row tile
    if (rest >= (long long)(N >> 4) * 64) return;
    const int lane = (int)(rest & 63);
    n = (int)(rest >> 6) * 16 + (lane & 15);
    kt = k_tiles - 1;
    g = lane >> 4;
  }
  const uint4 v = *(const uint4*)(src + (long long)n * K + kt * 32 + g * 8);
  const int tile = half < 0 ? tile_offset + (n >> 4) : n >> 3, col = half < 0 ? n & 15 : half * 8 + (n & 7);
  dst[((long long)tile * k_tiles + kt) * 64 + g * 16 + col] = v;
}
void launch_pack_weight(const void* src, void* dst, int N, int K, int tile_offset, int half, hipStream_t s) {
  long long total = (long long)(N >> 4) * (K >> 5) * 64;
  if (total) pack_weight_kernel<<<ceil_div(total, 256), 256, 0, s>>>((const uint16_t*)src, (uint4*)dst, N, K,
                                                                      tile_offset, half);
}
