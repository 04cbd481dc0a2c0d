// Weight-streaming GEMMs: y[M,N] = a[M,K] * W[N,K]^T with fused epilogues.
//   bf16: MFMA 16x16x32, weights in the tiled layout of common.h, activations as hi+lo bf16 pairs
//         (two MFMAs per weight tile), fp32 accumulation.
//   fp32: one or four wavefronts per output column (small models only).
#pragma once
#include <type_traits>

#include "common.h"
#include "finish.h"
#include "plan.h"

// FIN_RESID: the last workgroup of a column block finishes the sum (finish.h)
enum { EPI_STORE = 0, EPI_RESID = 1, EPI_SWIGLU = 2, EPI_FIN_RESID = 3 };

struct EpiArgs {
  float* out;   // STORE: out[z*slab + m*ld + n] = partial y of K range z ; RESID (fp32 kernel): out[m*ld + n] += y
  int ld;
  size_t slab;  // elements between the partial results of consecutive K ranges (grid.z)
  void* act;    // SWIGLU: act (GEMM activation operand, row length act_K) [m, j] = silu(gate_j) * up_j
  int act_K;
  // STORE with a single K range, LM head only: fused row argmax.  Every workgroup also writes the best
  // (score, column) of its columns for each of its rows to amax[m * gridDim.x-many parts + part]; score = y
  // (mode 0) or y * inv_T + Gumbel(key, m / B, m % B, purpose 0, column) (mode 1).  out may then be null
  // (logits not wanted).  A second, tiny kernel combines the parts (ties -> lowest column).
  float2* amax = nullptr;
  int amax_mode = 0;
  float amax_inv_T = 1.f;
  const uint64_t* amax_key = nullptr;
  int amax_B = 1;
  // STORE with a single K range, LM head only: fused softmax statistics.  Every workgroup also writes, for each of its
  // rows, (max, sum of exp(y * lse_inv_T - max)) over its columns to lse[m * parts + part] (same partition as amax); a
  // second, tiny kernel combines the parts in ascending order into (max, log-sum-exp).
  float2* lse = nullptr;
  float lse_inv_T = 1.f;
  // grouped launch (routed experts): a 1-D grid over (work item, column block); grp_items[item] = (expert, first band,
  // end band, whether it is the expert's only item) replaces the fixed band range; the workgroup multiplies those bands by the expert's matrix W + expert * grp_w_stride
  // (elements), an item with expert < 0 has nothing to do.  grp_rows (nullable) [bands * 16]: the activation row
  // behind each row of a band (the operand is then read through this list; < 0 = padding, any row will do).
  const int4* grp_items = nullptr;
  int grp_n_items = 0;
  size_t grp_w_stride = 0;
  bool grp_stream = false;   // LDS-staged kernel: weights of an expert's only item with the non-temporal hint
  const int32_t* grp_rows = nullptr;
  // Deferred RMSNorm (streaming kernel only): the operand holds x * gain without the division by the row's rms; row m
  // of the result is multiplied by 1 / sqrt(sum_p ssq[m * ssq_row(ssq_parts) + p] * ssq_inv_D + ssq_eps) before any epilogue
  // sees it (the sums of squares come in ssq_parts pieces, added in ascending order; see gemm_resid.h).
  const float* ssq = nullptr;
  int ssq_parts = 0;
  float ssq_inv_D = 0.f, ssq_eps = 0.f;
  // STORE with a single K range, LM head only: the result goes here as well (the caller's logits beside the workspace's; a
  // copy afterwards read them all again: 4 to 10 us a call)
  float* out2 = nullptr;
  FinishArgs fin = {};   // FIN_RESID (streaming kernel; out: the slabs)
  // fp32 kernel.  norm_gain: A holds rows that are to be normalised, y = (A * gain / rms(A)) W'.  tap (RESID): the new value goes
  // there as well, row length tap_K.
  const float* norm_gain = nullptr;
  float norm_eps = 0.f;
  float* tap = nullptr;
  int tap_K = 0;
  bool groups_side_by_side = false;   // see f32_groups_side_by_side in plan.h
};

// score of logit y at (row m, column col) for the fused argmax
__device__ __forceinline__ float amax_score(const EpiArgs& ep, uint64_t key, float y, int m, int col) {
  return ep.amax_mode ? y * ep.amax_inv_T + gumbel(counter_uniform(key, m / ep.amax_B, m % ep.amax_B, 0, (uint32_t)col)) : y;
}

// Split of K across workgroups (grid.z ranges): the STORE epilogue writes one partial slab per range and
// the kernel that consumes the result (RMSNorm, q/k-norm + RoPE) adds the slabs in ascending order.
// The kernel boundary provides the ordering: no atomics, no fences, and a sum that does not depend on
// which workgroup finished first.

// (max, sum of exponentials relative to that max) of the union of two sets; an empty set is (-inf, 0)
__device__ __forceinline__ void lse_combine(float& m, float& s, float m2, float s2) {
  const float M = fmaxf(m, m2);
  s = (m == -INFINITY ? 0.f : s * __expf(m - M)) + (m2 == -INFINITY ? 0.f : s2 * __expf(m2 - M));
  m = M;
}
// the same over the 4 lanes that hold the other columns of a row (lane bits 4 and 5)
__device__ __forceinline__ void lse_combine_row(float& m, float& s) {
#pragma unroll
  for (int o = 16; o <= 32; o <<= 1) {
    const float om = __shfl_xor(m, o, 64), os = __shfl_xor(s, o, 64);
    lse_combine(m, s, om, os);
  }
}
__device__ __forceinline__ void lse_add4(float& m, float& s, float4 y, float inv_T) {
  const float a = y.x * inv_T, b = y.y * inv_T, c = y.z * inv_T, d = y.w * inv_T;
  const float mx = fmaxf(fmaxf(a, b), fmaxf(c, d));
  lse_combine(m, s, mx, __expf(a - mx) + __expf(b - mx) + __expf(c - mx) + __expf(d - mx));
}

__device__ __forceinline__ float silu_f(float x) { return x / (1.0f + __expf(-x)); }

// ------------------------------------------------------------------------------------------------
// bf16 MFMA kernel.  A workgroup of 4 wavefronts owns NT 16-row bands of W (N tiles) and MT 16-row
// bands of the activations for one K range (grid.z ranges); each wavefront streams a quarter of that
// range, U k-tiles at a time with the next U already in flight, every activation fragment reused for
// the NT weight tiles.  The four partial sums are added in a fixed order through LDS.  The MFMA
// computes D^T = W_tile * a_tile^T: lane l ends up holding y[m = l%16][n = 4*(l/16) .. +3].
// SWIGLU: W rows alternate 16 gate rows / 16 up rows, so tiles (2p, 2p+1) of a workgroup are the
// gate and up values of the same 16 activation columns.
// ------------------------------------------------------------------------------------------------
template <int NT, int MT, int U>
struct GemmBuf {
  u32x4 w[U][NT], ah[U][MT], al[U][MT];
};

template <int NT, int MT, int U, int EPI, bool GRP = false>
__global__ __launch_bounds__(256, 1) void gemm_bf16_kernel(const bf16_t* __restrict__ W, const bf16_t* __restrict__ A,
                                                        int M, int N, int K, EpiArgs ep) {
  constexpr int NW = 4;   // wavefronts of a workgroup, each with its share of the K range
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kz = blockIdx.z;
  const int KT = K >> 5, n_tiles = N >> 4;
  int nt0 = blockIdx.x * NT;
  int mt0 = blockIdx.y * MT, m_tiles = (M + 15) >> 4;   // bands mt0 .. min(mt0 + MT, m_tiles) - 1 are this workgroup's
  if constexpr (GRP) {
    // 1-D grid; consecutive workgroup ids go to different XCDs (round-robin dispatch), so id = 8*j + x is work item
    // 8*(j / columns) + x, column block j % columns: the workgroups that share an item's activation rows run back to
    // back on one XCD and fetch them into one L2 instead of eight
    const int cols = n_tiles / NT, x = blockIdx.x & 7, j = blockIdx.x >> 3;
    const int it = (j / cols) * 8 + x;
    if (it >= ep.grp_n_items) return;
    const int4 item = ep.grp_items[it];
    if (item.x < 0) return;
    W += (size_t)item.x * ep.grp_w_stride;
    nt0 = (j % cols) * NT;
    mt0 = item.y;
    m_tiles = item.z;
  }
  const int ks = gridDim.z;
  const int per = (KT + ks * NW - 1) / (ks * NW);
  const int kb = min(KT, (kz * NW + wave) * per);
  const int ke = min(KT, kb + per);

  f32x4 acc[NT][MT];
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int j = 0; j < MT; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};

  const u32x4* Wp = reinterpret_cast<const u32x4*>(W) + lane;
  const u32x4* Ap = reinterpret_cast<const u32x4*>(A) + (GRP && ep.grp_rows ? 0 : lane);   // row lists carry the lane's offset
  // activation bands past the last one alias the last band (their results are never stored);
  // a band holds, per k tile, the hi tile then the lo tile (64 lanes x 16 bytes each)
  size_t a_band[MT];
#pragma unroll
  for (int j = 0; j < MT; ++j) {
    const int band = min(mt0 + j, m_tiles - 1);
    a_band[j] = (size_t)band * KT * 128;
    if constexpr (GRP) {
      if (ep.grp_rows) {   // lane (row r = lane % 16, k chunk lane / 16) of the fragment reads row grp_rows[16 * band + r]
        const int t = max(ep.grp_rows[band * 16 + (lane & 15)], 0);
        a_band[j] = (size_t)(t >> 4) * KT * 128 + (size_t)((lane >> 4) * 16 + (t & 15));
      }
    }
  }

  auto load = [&](GemmBuf<NT, MT, U>& b, int k0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = k0 + u < ke;
      const int kt = in ? k0 + u : ke - 1;   // past the range: re-read the last tile, with zeroed activations
#pragma unroll
      for (int i = 0; i < NT; ++i) b.w[u][i] = __builtin_nontemporal_load(Wp + ((size_t)kt * n_tiles + nt0 + i) * 64);
#pragma unroll
      for (int j = 0; j < MT; ++j) {
        const u32x4 h = Ap[a_band[j] + (size_t)kt * 128], l = Ap[a_band[j] + (size_t)kt * 128 + 64];
        b.ah[u][j] = in ? h : (u32x4){0u, 0u, 0u, 0u};
        b.al[u][j] = in ? l : (u32x4){0u, 0u, 0u, 0u};
      }
    }
  };
  // all hi products of a k tile, then all lo products: two MFMAs on the same accumulator are never back to back (the
  // second would wait out the first one's passes)
  auto compute = [&](const GemmBuf<NT, MT, U>& b) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, b.w[u][i]),
                                                              __builtin_bit_cast(bf16x8, b.ah[u][j]), acc[i][j], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, b.w[u][i]),
                                                              __builtin_bit_cast(bf16x8, b.al[u][j]), acc[i][j], 0, 0, 0);
    }
  };

  // Deferred RMSNorm: 1 / rms of this workgroup's rows, 16 threads per row.  The pieces of the sums of squares are requested
  // here and added behind the sweep (16 threads a row, each every 16th group of four in ascending order, then a fixed butterfly
  // tree); s_rstd is read after the barrier of the cross-wavefront sum.
  __shared__ float s_rstd[16];
  constexpr int SQ = kSsqAhead / 64;          // groups of four that a thread keeps in registers over the sweep
  const bool deferred = MT == 1 && !GRP && ep.ssq;   // dense, one band of rows only
  const int sq_c = (threadIdx.x & 15) * 4, sq_row = ssq_row(ep.ssq_parts);
  const float* sq_p = ep.ssq + (size_t)min(mt0 * 16 + ((int)threadIdx.x >> 4), M - 1) * sq_row;
  float4 sq[SQ];
  if (deferred) {
#pragma unroll
    for (int i = 0; i < SQ; ++i)
      if (i * 64 < ep.ssq_parts) sq[i] = *reinterpret_cast<const float4*>(sq_p + min(sq_c + i * 64, sq_row - 4));   // uniform condition
  }
  auto rstd_of_rows = [&]() {
    float t = 0.f;
    auto add = [&](float4 v, int p) {   // pieces p .. p + 3 of the row
      v.x = p < ep.ssq_parts ? v.x : 0.f;
      v.y = p + 1 < ep.ssq_parts ? v.y : 0.f;
      v.z = p + 2 < ep.ssq_parts ? v.z : 0.f;
      v.w = p + 3 < ep.ssq_parts ? v.w : 0.f;
      t += (v.x + v.y) + (v.z + v.w);
    };
#pragma unroll
    for (int i = 0; i < SQ; ++i)
      if (i * 64 < ep.ssq_parts) add(sq[i], sq_c + i * 64);
    for (int p = sq_c + kSsqAhead; p < ep.ssq_parts; p += 64) add(*reinterpret_cast<const float4*>(sq_p + p), p);
    t += lane_xor<1>(t);
    t += lane_xor<2>(t);
    t += lane_xor<4>(t);
    t += lane_xor<8>(t);
    if ((threadIdx.x & 15) == 0) s_rstd[threadIdx.x >> 4] = 1.0f / sqrtf(t * ep.ssq_inv_D + ep.ssq_eps);
  };

  // Two register buffers, one being multiplied while the other is on its way.  No load inside the loop is
  // conditional: a load that is skipped on some path would make the number of loads in flight unknown at compile
  // time, and the wait for the older buffer would then have to drain the newer one as well.  The last one or two
  // stages are peeled off; if the range has an odd number of stages the final load re-reads the last tile
  // (still in cache) and meets zeroed activations.
  if (kb < ke) {
    GemmBuf<NT, MT, U> b0, b1;
    load(b0, kb);
    int k0 = kb;
    for (; k0 + 2 * U < ke; k0 += 2 * U) {
      load(b1, k0 + U);
      compute(b0);
      load(b0, k0 + 2 * U);
      compute(b1);
    }
    load(b1, k0 + U);
    compute(b0);
    compute(b1);
  }

  if (deferred) rstd_of_rows();

  // The wavefronts' partial sums meet in LDS.
  __shared__ float4 red[NW][NT * MT][64];
  const int mrow = lane & 15, g = lane >> 4;
  // the wavefronts' partial sums of tile t (= weight tile * MT + band), in wavefront order,
  // times the row's deferred 1 / rms
  auto tile_sum = [&](int t) {
    float4 s = red[0][t][lane];
#pragma unroll
    for (int w = 1; w < NW; ++w) {
      const float4 a = red[w][t][lane];
      s.x += a.x; s.y += a.y; s.z += a.z; s.w += a.w;
    }
    if (deferred) {
      const float rs = s_rstd[mrow];
      s.x *= rs; s.y *= rs; s.z *= rs; s.w *= rs;
    }
    return s;
  };
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int j = 0; j < MT; ++j) red[wave][i * MT + j][lane] = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
  __syncthreads();
  if constexpr (EPI == EPI_SWIGLU) {
    bf16_t* act = reinterpret_cast<bf16_t*>(ep.act);
    for (int t = wave; t < (NT / 2) * MT; t += NW) {
      const int p = t / MT, j = t % MT;
      const float4 gs = tile_sum((2 * p) * MT + j), us = tile_sum((2 * p + 1) * MT + j);
      const int m = (mt0 + j) * 16 + mrow;
      if (mt0 + j < m_tiles && m < M) {
        const int col = ((nt0 + 2 * p) >> 1) * 16 + 4 * g;
        Act<bf16_t>::store4(act, m, col, ep.act_K,
                            make_float4(silu_f(gs.x) * us.x, silu_f(gs.y) * us.y, silu_f(gs.z) * us.z, silu_f(gs.w) * us.w));
      }
    }
  } else if constexpr (EPI == EPI_FIN_RESID) {
    const __amdgpu_buffer_rsrc_t out = coherent_base(ep.out);
    for (int t = wave; t < NT; t += NW) {
      const float4 s = tile_sum(t);
      if (mrow < M) store_coherent(out, (unsigned)((size_t)kz * ep.slab + (size_t)mrow * ep.ld + (nt0 + t) * 16 + 4 * g) * 4u, s);
    }
    if (!last_to_arrive(ep.fin.arrive + blockIdx.x * kArriveStride, gridDim.z)) return;
    finish_resid<NT>(ep.fin, ep.out, ep.ld, ep.slab, (int)gridDim.z, M, (int)blockIdx.x, (int)gridDim.x, reinterpret_cast<float*>(&red[0][0][0]));
  } else if (ep.out) {
    for (int t = wave; t < NT * MT; t += NW) {
      const int i = t / MT, j = t % MT;
      const float4 s = tile_sum(t);
      const int m = (mt0 + j) * 16 + mrow;
      if (mt0 + j < m_tiles && m < M) {
        const size_t at = (size_t)m * ep.ld + (nt0 + i) * 16 + 4 * g;
        *reinterpret_cast<float4*>(ep.out + (size_t)kz * ep.slab + at) = s;
        if (ep.out2) *reinterpret_cast<float4*>(ep.out2 + at) = s;
      }
    }
  }

  if constexpr (EPI == EPI_STORE) {
    if (ep.amax) {   // fused argmax over this workgroup's NT*16 columns (host guarantees a single K range)
      __shared__ float2 wbest[NW][MT * 16];
      const uint64_t key = ep.amax_mode ? ep.amax_key[0] : 0ull;
#pragma unroll
      for (int j = 0; j < MT; ++j) {
        const int m = (mt0 + j) * 16 + mrow;
        float bv = -INFINITY;
        int bi = 0x7FFFFFFF;
        for (int i = wave; i < NT; i += NW) {
          const float4 s = tile_sum(i * MT + j);
          const int col = (nt0 + i) * 16 + 4 * g;
          argmax_combine(bv, bi, amax_score(ep, key, s.x, m, col), col);
          argmax_combine(bv, bi, amax_score(ep, key, s.y, m, col + 1), col + 1);
          argmax_combine(bv, bi, amax_score(ep, key, s.z, m, col + 2), col + 2);
          argmax_combine(bv, bi, amax_score(ep, key, s.w, m, col + 3), col + 3);
        }
        argmax_swap16(bv, bi);
        argmax_swap32(bv, bi);
        if (g == 0) wbest[wave][j * 16 + mrow] = make_float2(bv, __int_as_float(bi));
      }
      __syncthreads();
      for (int r = threadIdx.x; r < MT * 16; r += 64 * NW) {
        const int m = mt0 * 16 + r;
        if (m >= M) continue;
        float bv = wbest[0][r].x;
        int bi = __float_as_int(wbest[0][r].y);
#pragma unroll
        for (int w = 1; w < NW; ++w) argmax_combine(bv, bi, wbest[w][r].x, __float_as_int(wbest[w][r].y));
        ep.amax[(size_t)m * gridDim.x + blockIdx.x] = make_float2(bv, __int_as_float(bi));
      }
    }
    if (ep.lse) {   // fused softmax statistics over this workgroup's NT*16 columns (single K range)
      __shared__ float2 wl[NW][MT * 16];
      __syncthreads();
#pragma unroll
      for (int j = 0; j < MT; ++j) {
        float lm = -INFINITY, ls = 0.f;
        for (int i = wave; i < NT; i += NW) lse_add4(lm, ls, tile_sum(i * MT + j), ep.lse_inv_T);
        lse_combine_row(lm, ls);
        if (g == 0) wl[wave][j * 16 + mrow] = make_float2(lm, ls);
      }
      __syncthreads();
      for (int r = threadIdx.x; r < MT * 16; r += 64 * NW) {
        const int m = mt0 * 16 + r;
        if (m >= M) continue;
        float lm = wl[0][r].x, ls = wl[0][r].y;
#pragma unroll
        for (int w = 1; w < NW; ++w) lse_combine(lm, ls, wl[w][r].x, wl[w][r].y);
        ep.lse[(size_t)m * gridDim.x + blockIdx.x] = make_float2(lm, ls);
      }
    }
  }
}

// ------------------------------------------------------------------------------------------------
// fp32 kernel (small models): block = 4 wavefronts, 4 / KW output columns (SWIGLU: one activation column = a gate row
// and the up row 16 below it), KW wavefronts per column that take every KW-th 256-wide piece of K; lanes stride over K; eight
// rows a workgroup (groups of them: one after the other in a workgroup, a step of the 2 + 1 layer model of width 256 took 320 us
// at 64 rows, side by side 182; width 2048, 128 rows 3208 and 2923).  Bound by latency: all loads of a piece go out together (rows past the last one repeat it, a load under
// a condition would be waited for by itself), a lane for each row of a column's first wavefront finishes it (eight read-modify-writes
// by one lane were eight round trips).  N = 256, K = 1024, 8 rows, RESID: 10.5 us, now 4.3 (the launch floor).
// ------------------------------------------------------------------------------------------------
// NORM: the RMSNorm in front of the product is taken along, y = (1 / rms(a)) ((a * gain) W'): a wavefront multiplies the gain in and
// the sums of squares come out of the same sweep, two of the eight rows a wavefront where all four see the whole K.  Costs 0.6 to 0.8
// us at 8 rows of width 256 and saves a launch of 3.6 (fold_norm in plan.h).
template <int EPI, int KW, bool NORM>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ W, const float* __restrict__ A, int M,
                                                       int N, int K, EpiArgs ep) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kw = wave % KW;
  const int n_cols = (EPI == EPI_SWIGLU) ? N / 2 : N;
  // grid (column blocks, groups of eight rows), or the groups of a column block one after the other on one XCD: workgroup ids are dealt to
  // the eight XCDs round-robin, x first, so grid (8 * groups, column blocks / 8) and XCD x % 8 takes the block y * 8 + x % 8
  const int col_block = ep.groups_side_by_side ? (int)blockIdx.y * 8 + ((int)blockIdx.x & 7) : (int)blockIdx.x;
  const int row_group = ep.groups_side_by_side ? (int)blockIdx.x >> 3 : (int)blockIdx.y;
  if (col_block * (4 / KW) >= n_cols) return;
  const int col_raw = col_block * (4 / KW) + wave / KW, col = min(col_raw, n_cols - 1);   // a column past the end is not stored
  const int row0 = (EPI == EPI_SWIGLU) ? (col >> 4) * 32 + (col & 15) : col;
  const float* w0 = W + (size_t)row0 * K;
  const float* w1 = w0 + (size_t)16 * K;  // SWIGLU only
  constexpr int SQ = KW == 1 ? 2 : 8;     // rows whose squares a wavefront adds, from row SQ * wave of the eight (KW == 1) or all
  __shared__ float sum[2][4][8];
  __shared__ float sq[KW == 1 ? 1 : 4][8];
  const int m0 = row_group * 8;
  float acc0[8], acc1[8], ss[SQ];
#pragma unroll
  for (int r = 0; r < 8; ++r) acc0[r] = acc1[r] = 0.f;
#pragma unroll
  for (int r = 0; r < SQ; ++r) ss[r] = 0.f;
  for (int k = kw * 256 + lane * 4; k < K; k += 256 * KW) {
    float4 a[8], own[SQ];
    const float4 wa = *reinterpret_cast<const float4*>(w0 + k);
    float4 wb = make_float4(0.f, 0.f, 0.f, 0.f), g = make_float4(1.f, 1.f, 1.f, 1.f);
    if (EPI == EPI_SWIGLU) wb = *reinterpret_cast<const float4*>(w1 + k);
    if constexpr (NORM) g = *reinterpret_cast<const float4*>(ep.norm_gain + k);
#pragma unroll
    for (int r = 0; r < 8; ++r) a[r] = *reinterpret_cast<const float4*>(A + (size_t)min(m0 + r, M - 1) * K + k);
    if constexpr (NORM && KW == 1) {   // again, from the L1: which rows they are depends on the wavefront
#pragma unroll
      for (int r = 0; r < SQ; ++r) own[r] = *reinterpret_cast<const float4*>(A + (size_t)min(m0 + SQ * wave + r, M - 1) * K + k);
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (NORM) {
#pragma unroll
      for (int r = 0; r < SQ; ++r) {
        const float4 x = KW == 1 ? own[r] : a[r];
        ss[r] += x.x * x.x + x.y * x.y + x.z * x.z + x.w * x.w;
      }
    }
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      if constexpr (NORM) a[r] = make_float4(a[r].x * g.x, a[r].y * g.y, a[r].z * g.z, a[r].w * g.w);
      acc0[r] += a[r].x * wa.x + a[r].y * wa.y + a[r].z * wa.z + a[r].w * wa.w;
      if (EPI == EPI_SWIGLU) acc1[r] += a[r].x * wb.x + a[r].y * wb.y + a[r].z * wb.z + a[r].w * wb.w;
    }
  }
  // one lane of eight finishes row m0 + r
  const int r = wave_sum8_index(lane);
  const bool finish = (lane & 7) == 0;
  float s0 = wave_sum8(acc0), s1 = EPI == EPI_SWIGLU ? wave_sum8(acc1) : 0.f;
  if constexpr (NORM) {
    if constexpr (SQ == 8) {
      const float t = wave_sum8(ss);
      if (finish) sq[wave][r] = t;
    } else {
#pragma unroll
      for (int i = 0; i < SQ; ++i) {
        const float t = wave_reduce_sum(ss[i]);
        if (lane == 0) sq[0][SQ * wave + i] = t;
      }
    }
  }
  if constexpr (KW > 1) {
    if (finish) {
      sum[0][wave][r] = s0;
      if (EPI == EPI_SWIGLU) sum[1][wave][r] = s1;
    }
  }
  if constexpr (KW > 1 || NORM) __syncthreads();
  if constexpr (KW > 1) {
    if (kw == 0 && finish) {
#pragma unroll
      for (int i = 1; i < KW; ++i) {
        s0 += sum[0][wave + i][r];
        if (EPI == EPI_SWIGLU) s1 += sum[1][wave + i][r];
      }
    }
  }
  if constexpr (NORM) {
    if (finish) {
      float t = sq[0][r];
#pragma unroll
      for (int i = 1; i < KW; ++i) t += sq[i][r];
      const float rstd = 1.0f / sqrtf(t / (float)K + ep.norm_eps);
      s0 *= rstd;
      s1 *= rstd;
    }
  }
  const int m = m0 + r;
  if (kw == 0 && finish && m < M && col_raw < n_cols) {
    if (EPI == EPI_SWIGLU) {
      reinterpret_cast<float*>(ep.act)[(size_t)m * ep.act_K + col] = silu_f(s0) * s1;
    } else if (EPI == EPI_RESID) {
      const float h = ep.out[(size_t)m * ep.ld + col] + s0;
      ep.out[(size_t)m * ep.ld + col] = h;
      if (ep.tap) ep.tap[(size_t)m * ep.tap_K + col] = h;
    } else {
      ep.out[(size_t)m * ep.ld + col] = s0;
      if (ep.out2) ep.out2[(size_t)m * ep.ld + col] = s0;
    }
  }
}
