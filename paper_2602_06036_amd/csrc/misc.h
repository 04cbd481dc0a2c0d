// Small memory-bound kernels of the step: embedding gather, RMSNorm, q/k-norm + RoPE + KV page
// write, row argmax / Gumbel-max, acceptance, commit bookkeeping, weight packing and
// KV import/export.
#pragma once
#include <type_traits>

#include "common.h"
#include "exp_nonpositive.h"
#include "finish.h"
#include "plan.h"

// ---- block assembly + embedding gather -------------------------------------------------------
// Rotary table of one model for the rows of a call: out[m * hd/2 + i] = (cos, sin) of pos(m) * theta^(-2i/hd),
// pos(m) = seq_lens[m / B] + m % B.  Angles are formed in double precision (reduced by sincos) so that long
// contexts do not lose phase accuracy; every layer and head of the call then reads the same rounded pair.
struct RopeTab {
  float2* out;   // null: no table
  double log_theta;
  int hd;
};

// h[m, :] = float(E[tokens[m], :]); ids outside the vocabulary raise the status flag and read row 0; so does a sequence
// longer than the host's hint.
// Up to two rotary tables are written by further workgroups of the launch.
// With `fuse.a_out` the row is also handed on as the first layer's GEMM operand with the RMSNorm deferred (see
// gemm_resid.h): a_out[m, :] = h * gain, ssq[m] = sum of squares of the row (one piece per row).
struct EmbedFuse {
  const float* gain = nullptr;
  void* a_out = nullptr;
  float* ssq = nullptr;
};
// Arrival counters of the GEMMs behind it that finish their own sums (finish.h).  They are zeroed here, at the head of every call that
// has such GEMMs, so that nothing has to survive in the workspace between calls; for a store per counter, hidden behind the rows.
struct EmbedArrive {
  unsigned* counters = nullptr;
  int n = 0;
};
// Drafting: tokens are assembled here, block[s, 0] = anchor[s], block[s, j > 0] = mask_id (Section 4.2: clean anchor + masks),
// and left in `block`; otherwise (block null) they are read.
struct EmbedBlock {
  const int32_t* anchor = nullptr;
  int32_t* block = nullptr;
  int mask_id = 0;
};

template <typename T>
__global__ __launch_bounds__(256) void embed_kernel(const T* __restrict__ E, const int32_t* __restrict__ tokens,
                                                    float* __restrict__ h, int D, int vocab, int32_t* status,
                                                    const int32_t* __restrict__ seq_lens, int B, int len_hint, int n_rows, RopeTab t0, RopeTab t1,
                                                    EmbedFuse fuse, EmbedBlock blk, EmbedArrive arrive) {
  // workgroups M .. of the grid write the rotary tables (angles in double precision take longer than a row's copy): one
  // entry of a table per thread
  if ((int)blockIdx.x >= n_rows) {
    const int half0 = t0.out ? t0.hd >> 1 : 0, half1 = t1.out ? t1.hd >> 1 : 0;
    const int i = ((int)blockIdx.x - n_rows) * 256 + threadIdx.x, per = half0 + half1;
    if (i >= n_rows * per) return;
    const int row = i / per, e = i % per;
    const RopeTab rt = e < half0 ? t0 : t1;
    const int d = e < half0 ? e : e - half0;
    double sn, cs;
    sincos((double)(seq_lens[row / B] + row % B) * exp(-rt.log_theta * (2.0 * d / rt.hd)), &sn, &cs);
    rt.out[(size_t)row * (rt.hd >> 1) + d] = make_float2((float)cs, (float)sn);
    return;
  }
  const int m = blockIdx.x;
  // the host sized the attention launches of this call for sequences of at most len_hint committed tokens: a longer
  // one would have its last keys left out, so it is reported
  if (threadIdx.x == 0 && seq_lens[m / B] > len_hint) atomicOr(status, DF_STATUS_CAPACITY);
  if (m == 0)
    for (int i = threadIdx.x; i < arrive.n; i += 256) arrive.counters[i * kArriveStride] = 0u;
  int tok;
  if (blk.block) {
    tok = m % B == 0 ? blk.anchor[m / B] : blk.mask_id;
    if (threadIdx.x == 0) blk.block[m] = tok;
  } else {
    tok = tokens[m];
  }
  if (tok < 0 || tok >= vocab) {
    if (threadIdx.x == 0) atomicOr(status, DF_STATUS_CAPACITY);
    tok = 0;
  }
  // eight columns a thread and round, whole rounds' loads together (one column at a time a row of 4096 was sixteen trips to memory)
  const T* src = E + (size_t)tok * D;
  float ss = 0.f;
  constexpr int U = 2;
  for (int d0 = threadIdx.x * 8; d0 < D; d0 += 256 * 8 * U) {
    float v[U][8], g[U][8];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int d = min(d0 + u * 2048, D - 8);   // past the end: the last eight again, not stored
#pragma unroll
      for (int e = 0; e < 8; ++e) v[u][e] = Store<T>::to(src[d + e]);
#pragma unroll
      for (int e = 0; e < 8; ++e) g[u][e] = fuse.a_out ? fuse.gain[d + e] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int d = d0 + u * 2048;
      if (d >= D) break;
      float* to = h + (size_t)m * D + d;
      *reinterpret_cast<float4*>(to) = make_float4(v[u][0], v[u][1], v[u][2], v[u][3]);
      *reinterpret_cast<float4*>(to + 4) = make_float4(v[u][4], v[u][5], v[u][6], v[u][7]);
      if (fuse.a_out) {
#pragma unroll
        for (int e = 0; e < 8; e += 4)
          Act<T>::store4(reinterpret_cast<T*>(fuse.a_out), m, d + e, D,
                         make_float4(v[u][e] * g[u][e], v[u][e + 1] * g[u][e + 1], v[u][e + 2] * g[u][e + 2], v[u][e + 3] * g[u][e + 3]));
#pragma unroll
        for (int e = 0; e < 8; ++e) ss += v[u][e] * v[u][e];
      }
    }
  }
  if (fuse.a_out) {   // uniform over the workgroup
    __shared__ float part[4];
    ss = wave_reduce_sum(ss);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
    __syncthreads();
    if (threadIdx.x == 0) fuse.ssq[(size_t)m * ssq_row(1)] = (part[0] + part[1]) + (part[2] + part[3]);
  }
}

// ---- RMSNorm with pending-sum reduction -----------------------------------------------------------
// x[m,:] = base[m,:] (if base) + sum_z delta[z*slab + m*D + :] (ascending z: the K-range partial results of
// the preceding GEMM).  When delta is given the completed row is written to h_out (the residual stream).
// Optionally the completed row is also stored as tap `tap_idx` (GEMM activation operand, row length tap_K).
// out[m,:] = x * gain / sqrt(mean(x^2) + eps) as GEMM activation operand (Act<T>).
// MIX (routed experts): the pending sum of row m is instead sum_j mix.w[m*k + j] * delta[mix.pos[m*k + j] * D + :], j
// ascending -- the weighted sum of the row's experts' outputs, which sit at the row's positions of the expert-sorted list.
struct RowMix {
  const int32_t* pos = nullptr;
  const float* w = nullptr;
  int k = 0;
};

template <typename T, int NTHR, bool MIX = false>
__global__ __launch_bounds__(NTHR) void rmsnorm_kernel(const float* base, const float* __restrict__ delta, int ks,
                                                      size_t slab, float* h_out, const float* __restrict__ gain,
                                                      T* __restrict__ out, int D, float eps, T* __restrict__ taps, int tap_idx,
                                                      int tap_K, RowMix mix = RowMix{}) {
  // Consecutive workgroup ids go to different XCDs (round-robin dispatch), and the 16 rows of a band share the cache
  // lines of an operand tile: with many rows, XCD x takes the rows [x * M/8, (x+1) * M/8), so that the 16-byte pieces
  // of a line are merged in one L2 and leave it as whole lines instead of eight partial writes from eight L2s.
  const int n_rows = (int)gridDim.x;
  const int m = (n_rows % 128 == 0) ? (int)(blockIdx.x & 7) * (n_rows >> 3) + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
  const size_t ro = (size_t)m * D;
  // completed row chunk d..d+3: base + pending slabs (four independent loads in flight, added in ascending order)
  auto gather = [&](int d) {
    float4 v = base ? *reinterpret_cast<const float4*>(base + ro + d) : make_float4(0.f, 0.f, 0.f, 0.f);
    if constexpr (MIX) {
      const int32_t* pj = mix.pos + (size_t)m * mix.k;
      const float* wj = mix.w + (size_t)m * mix.k;
      int j = 0;
      for (; j + 4 <= mix.k; j += 4) {   // four experts' rows in flight at a time
        const float4 p0 = *reinterpret_cast<const float4*>(delta + (size_t)pj[j] * D + d);
        const float4 p1 = *reinterpret_cast<const float4*>(delta + (size_t)pj[j + 1] * D + d);
        const float4 p2 = *reinterpret_cast<const float4*>(delta + (size_t)pj[j + 2] * D + d);
        const float4 p3 = *reinterpret_cast<const float4*>(delta + (size_t)pj[j + 3] * D + d);
        const float w0 = wj[j], w1 = wj[j + 1], w2 = wj[j + 2], w3 = wj[j + 3];
        v.x += w0 * p0.x; v.y += w0 * p0.y; v.z += w0 * p0.z; v.w += w0 * p0.w;
        v.x += w1 * p1.x; v.y += w1 * p1.y; v.z += w1 * p1.z; v.w += w1 * p1.w;
        v.x += w2 * p2.x; v.y += w2 * p2.y; v.z += w2 * p2.z; v.w += w2 * p2.w;
        v.x += w3 * p3.x; v.y += w3 * p3.y; v.z += w3 * p3.z; v.w += w3 * p3.w;
      }
      for (; j < mix.k; ++j) {
        const float4 p = *reinterpret_cast<const float4*>(delta + (size_t)pj[j] * D + d);
        const float w0 = wj[j];
        v.x += w0 * p.x; v.y += w0 * p.y; v.z += w0 * p.z; v.w += w0 * p.w;
      }
      *reinterpret_cast<float4*>(h_out + ro + d) = v;
      if (taps) Act<T>::store4(taps, m, tap_idx * D + d, tap_K, v);
      return v;
    }
    int z = 0;
    for (; z + 8 <= ks; z += 8) {   // eight slabs (what a few-row GEMM leaves) in one round trip
      const float* pz = delta + (size_t)z * slab + ro + d;
      float4 p[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) p[i] = *reinterpret_cast<const float4*>(pz + i * slab);
#pragma unroll
      for (int i = 0; i < 8; ++i) { v.x += p[i].x; v.y += p[i].y; v.z += p[i].z; v.w += p[i].w; }
    }
    for (; z + 4 <= ks; z += 4) {
      const float* pz = delta + (size_t)z * slab + ro + d;
      const float4 p0 = *reinterpret_cast<const float4*>(pz), p1 = *reinterpret_cast<const float4*>(pz + slab);
      const float4 p2 = *reinterpret_cast<const float4*>(pz + 2 * slab), p3 = *reinterpret_cast<const float4*>(pz + 3 * slab);
      v.x += p0.x; v.y += p0.y; v.z += p0.z; v.w += p0.w;
      v.x += p1.x; v.y += p1.y; v.z += p1.z; v.w += p1.w;
      v.x += p2.x; v.y += p2.y; v.z += p2.z; v.w += p2.w;
      v.x += p3.x; v.y += p3.y; v.z += p3.z; v.w += p3.w;
    }
    for (; z < ks; ++z) {
      const float4 p = *reinterpret_cast<const float4*>(delta + (size_t)z * slab + ro + d);
      v.x += p.x; v.y += p.y; v.z += p.z; v.w += p.w;
    }
    if (ks > 0) *reinterpret_cast<float4*>(h_out + ro + d) = v;
    if (taps) Act<T>::store4(taps, m, tap_idx * D + d, tap_K, v);
    return v;
  };
  // NTHR threads per row (1024 for wide rows: one 16-byte chunk per thread keeps every load independent).
  // The first KEEP chunks of a thread stay in registers between the two passes (rows up to 8192 wide);
  // wider rows re-read the rest from where it was written
  constexpr int KEEP = 8192 / (NTHR * 4);
  float4 keep[KEEP], gk[KEEP];   // the gains are requested together with the row: no extra round trip after the barrier
  float ss = 0.f;
  __shared__ float upper[NTHR == 512 ? KEEP : 1][256];   // 512 threads: the chunks' sums of the upper 256 (see below)
#pragma unroll
  for (int c = 0; c < KEEP; ++c) {
    const int d = (c * NTHR + (int)threadIdx.x) * 4;
    gk[c] = d < D ? *reinterpret_cast<const float4*>(gain + d) : make_float4(0.f, 0.f, 0.f, 0.f);
  }
#pragma unroll
  for (int c = 0; c < KEEP; ++c) {
    const int d = (c * NTHR + (int)threadIdx.x) * 4;
    keep[c] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (d < D) {
      keep[c] = gather(d);
      if constexpr (NTHR != 512) ss += keep[c].x * keep[c].x + keep[c].y * keep[c].y + keep[c].z * keep[c].z + keep[c].w * keep[c].w;
    }
  }
  // With 512 threads (rows of up to 8192) the squares are added as 256 threads add them, every 256th chunk of four in ascending order, then over the
  // lanes and wavefronts of the lower 256: the router's near-ties turn another order of these sums into another expert (one row of sixteen that goes
  // the other way is 1 % of the logits).  The exchange through LDS does not show: a two-layer verification of 512 routed rows 935.5 us without and 936 with it.
  if constexpr (NTHR == 512) {
    float q[KEEP];
#pragma unroll
    for (int c = 0; c < KEEP; ++c) {
      q[c] = keep[c].x * keep[c].x + keep[c].y * keep[c].y + keep[c].z * keep[c].z + keep[c].w * keep[c].w;
      if (threadIdx.x >= 256) upper[c][threadIdx.x - 256] = q[c];
    }
    __syncthreads();
    if (threadIdx.x < 256) {
#pragma unroll
      for (int c = 0; c < KEEP; ++c) ss = (ss + q[c]) + upper[c][threadIdx.x];
    }
  }
  for (int d = (KEEP * NTHR + (int)threadIdx.x) * 4; d < D; d += NTHR * 4) {
    const float4 v = gather(d);
    ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
  }
  __shared__ float part[NTHR / 64];
  ss = wave_reduce_sum(ss);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < NTHR / 64; ++w) tot += part[w];
  const float rstd = 1.0f / sqrtf(tot / (float)D + eps);
#pragma unroll
  for (int c = 0; c < KEEP; ++c) {
    const int d = (c * NTHR + (int)threadIdx.x) * 4;
    if (d < D) {
      const float4 v = keep[c], g = gk[c];
      Act<T>::store4(out, m, d, D, make_float4(v.x * rstd * g.x, v.y * rstd * g.y, v.z * rstd * g.z, v.w * rstd * g.w));
    }
  }
  const float* src = ks > 0 ? h_out : base;   // each thread re-reads exactly what it wrote
  for (int d = (KEEP * NTHR + (int)threadIdx.x) * 4; d < D; d += NTHR * 4) {
    const float4 v = *reinterpret_cast<const float4*>(src + ro + d);
    const float4 g = *reinterpret_cast<const float4*>(gain + d);
    Act<T>::store4(out, m, d, D, make_float4(v.x * rstd * g.x, v.y * rstd * g.y, v.z * rstd * g.z, v.w * rstd * g.w));
  }
}

// ---- q/k RMSNorm + RoPE + cache write ------------------------------------------------------------
// One wavefront per (row m, head), four heads per workgroup; lane i owns the rotate-half pair (i, i + hd/2) [hd <= 128].
// Input row: fp32 [.. q heads | k heads | v heads ..] starting at in + m*in_ld, given as `ks` partial
// slabs (K ranges of the producing GEMM) `slab` elements apart that are added in ascending order.
// q heads -> q_out [M, Hq, hd] row-major storage type; k/v heads -> page of position seq_len + slot.
// (cos, sin) come from the call's rotary table (RopeTab), written by embed_kernel.
struct RopeArgs {
  int n_q_heads, n_kv_heads, head_dim;
  int q_off, k_off, v_off;  // element offsets inside an input row
  int qk_norm;
  float eps;
  const float2* rope;       // rotary table [M, hd/2] of this model for the rows of the call
  int layer;                // layer index inside the pool
  // grid.z > 1 handles several layers in one launch (the draft's context K/V at commit): layer z reads its
  // k/v columns z * col_stride further along the input row and its k-norm gain kn_stride floats further on
  int col_stride = 0;
  size_t kn_stride = 0;
};

template <typename T>
__global__ __launch_bounds__(256) void qkv_post_kernel(const float* __restrict__ in, int in_ld, const float* __restrict__ qn,
                                                       const float* __restrict__ kn, T* __restrict__ q_out,
                                                       T* __restrict__ pool, SeqGeom geo, RopeArgs ra, int ks, size_t slab) {
  // rows of one 16-key page on one XCD (see rmsnorm_kernel): their 16-byte pieces of a K/V page line meet in one L2
  const int n_rows = (int)gridDim.x;
  const int m = (n_rows % 128 == 0) ? (int)(blockIdx.x & 7) * (n_rows >> 3) + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
  const int head = blockIdx.y * 4 + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (head >= ra.n_q_heads + 2 * ra.n_kv_heads) return;   // no barrier in this kernel
  ra.layer += blockIdx.z;
  ra.k_off += blockIdx.z * ra.col_stride;
  ra.v_off += blockIdx.z * ra.col_stride;
  kn += blockIdx.z * ra.kn_stride;
  const int hd = ra.head_dim, half = hd >> 1;
  const int s = m / geo.block_size, slot = m % geo.block_size;
  const bool is_q = head < ra.n_q_heads;
  const bool is_k = !is_q && head < ra.n_q_heads + ra.n_kv_heads;
  const int kvh = is_q ? 0 : (is_k ? head - ra.n_q_heads : head - ra.n_q_heads - ra.n_kv_heads);
  const bool active = lane < half;
  const int l0 = active ? lane : 0;   // idle lanes read along (head_dim 64 and less)
  const float* src = in + (size_t)m * in_ld + (is_q ? ra.q_off + head * hd : (is_k ? ra.k_off : ra.v_off) + kvh * hd) + l0;
  // everything the head needs is requested before any of it is waited for: this kernel is a chain of memory round trips
  // and nothing else (a step of the 8B shape at batch 1, 41 launches: 4416 us with one slab after the other and the gains
  // and angles behind them, 4388 like this; by itself a launch takes 4.6 us either way)
  float2 r = make_float2(1.f, 0.f);
  float g1 = 1.f, g2 = 1.f;
  if (is_q || is_k) {
    r = ra.rope[(size_t)m * half + l0];
    if (ra.qk_norm) {
      const float* gn = is_q ? qn : kn;
      g1 = gn[l0];
      g2 = gn[l0 + half];
    }
  }
  const int n_s = geo.seq_lens[s];
  float x1 = 0.f, x2 = 0.f;
  // the slabs in ascending order, up to four in flight (the same few instructions whatever ks is: no slab is read twice)
  auto add = [&](int z, auto nc) {
    constexpr int C = decltype(nc)::value;
    float p1[C], p2[C];
#pragma unroll
    for (int i = 0; i < C; ++i) {
      p1[i] = src[(size_t)(z + i) * slab];
      p2[i] = src[(size_t)(z + i) * slab + half];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < C; ++i) { x1 += p1[i]; x2 += p2[i]; }
  };
  int z = 0;
  for (; z + 4 <= ks; z += 4) add(z, std::integral_constant<int, 4>{});
  if (z + 2 <= ks) { add(z, std::integral_constant<int, 2>{}); z += 2; }
  if (z < ks) add(z, std::integral_constant<int, 1>{});
  const int pos = n_s + slot;
  T* base = nullptr;
  const int key = pos % DF_PAGE;
  if (!is_q) {
    const int pidx = pos / DF_PAGE;
    int page = -1;
    if (pos >= 0 && pidx < geo.max_pages_per_seq) page = geo.block_table[(size_t)s * geo.max_pages_per_seq + pidx];
    if (page < 0 || page >= geo.n_pages) {
      if (lane == 0) atomicOr(geo.status, DF_STATUS_CAPACITY);
      return;
    }
    base = pool + kv_head_base(ra.layer, geo.n_pages, page, ra.n_kv_heads, kvh, hd);
    if (!is_k) {
      if (active) {
        base[DF_PAGE * hd + v_in_page(key, lane)] = Store<T>::from(x1);
        base[DF_PAGE * hd + v_in_page(key, lane + half)] = Store<T>::from(x2);
      }
      return;
    }
  }
  if (ra.qk_norm) {
    // which product of a sum is rounded by itself is written out here and below: left to the compiler it changes with the code
    // around it, and a last bit here is a bf16 step of one stored value in some ten thousand
    const float ss = wave_reduce_sum(active ? fmaf(x2, x2, x1 * x1) : 0.f);
    const float rstd = 1.0f / sqrtf(ss / (float)hd + ra.eps);
    x1 *= rstd * g1;
    x2 *= rstd * g2;
  }
  if (!active) return;
  const float c = r.x, sf = r.y;
  const T y1 = Store<T>::from(fmaf(x1, c, -(x2 * sf))), y2 = Store<T>::from(fmaf(x2, c, x1 * sf));
  if (is_q) {
    T* dst = q_out + ((size_t)m * ra.n_q_heads + head) * hd;
    dst[lane] = y1;
    dst[lane + half] = y2;
  } else {
    base[k_in_page(key, lane)] = y1;
    base[k_in_page(key, lane + half)] = y2;
  }
}

// ---- row argmax (ties -> lowest index), optionally of logit/T + Gumbel noise ---------------------
// block-wide argmax (up to 1024 threads); result valid in thread 0
__device__ __forceinline__ void block_argmax(float& bv, int& bi) {
  __shared__ float sv[16];
  __shared__ int si[16];
  wave_argmax(bv, bi);
  const int wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  if ((threadIdx.x & 63) == 0) { sv[wave] = bv; si[wave] = bi; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < nw; ++w) argmax_combine(bv, bi, sv[w], si[w]);
  }
}

// mode 0: greedy.  mode 1: draft sampling, score = logit * inv_T + Gumbel(key, seq, slot, purpose 0).
// Stage 1: grid (n_chunks, M): best (score, index) of one chunk of row m -> part[m * n_chunks + chunk].
// With a single chunk a row (n_chunks == 1, `out` given) the winner is written here, as stage 2 would.
// Stage 2 (argmax_finish_kernel): combines the chunks in ascending order (ties -> lowest index) and writes out[m]
// unless (skip_slot0 && slot == 0).
__global__ __launch_bounds__(256) void argmax_rows_kernel(const float* __restrict__ logits, int V, int B, float2* __restrict__ part,
                                                          int mode, float inv_T, const uint64_t* __restrict__ rng_key,
                                                          int32_t* __restrict__ out, int skip_slot0) {
  const int chunk = blockIdx.x, n_chunks = gridDim.x, m = blockIdx.y, slot = m % B, seq = m / B;
  if (out && skip_slot0 && slot == 0) return;
  const int per = (V + n_chunks - 1) / n_chunks, i0 = chunk * per, i1 = min(V, i0 + per);
  const float* row = logits + (size_t)m * V;
  float bv = -INFINITY;
  int bi = 0x7FFFFFFF;
  const uint64_t key = mode ? rng_key[0] : 0ull;
  for (int i = i0 + threadIdx.x; i < i1; i += blockDim.x) {
    float v = row[i];
    if (mode) v = v * inv_T + gumbel(counter_uniform(key, seq, slot, 0, (uint32_t)i));
    argmax_combine(bv, bi, v, i);
  }
  block_argmax(bv, bi);
  if (threadIdx.x != 0) return;
  if (out) out[m] = bi;
  else part[(size_t)m * n_chunks + chunk] = make_float2(bv, __int_as_float(bi));
}

__global__ __launch_bounds__(256) void argmax_finish_kernel(const float2* __restrict__ part, int n_chunks, int B, int32_t* __restrict__ out,
                                                            int skip_slot0) {
  const int m = blockIdx.x;
  if (skip_slot0 && m % B == 0) return;
  float bv = -INFINITY;
  int bi = 0x7FFFFFFF;
  // five parts a thread cover the 1187 column blocks of a 151936-entry vocabulary in one round trip (8.6 us by one
  // wavefront with a load at a time, 5 like this)
  for (int c0 = threadIdx.x; c0 < n_chunks; c0 += 256 * 5) {
    float2 p[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) p[i] = part[(size_t)m * n_chunks + min(c0 + i * 256, n_chunks - 1)];   // the last part again: no other winner
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 5; ++i) argmax_combine(bv, bi, p[i].x, __float_as_int(p[i].y));
  }
  block_argmax(bv, bi);
  if (threadIdx.x == 0) out[m] = bi;
}

// ---- greedy acceptance (Section 3.1) ---------------------------------------------------------------
__global__ void accept_greedy_kernel(const int32_t* __restrict__ draft, const int32_t* __restrict__ tgt, int S, int B,
                                     int32_t* __restrict__ accept_len, int32_t* __restrict__ out_tokens) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= S) return;
  const int32_t* d = draft + (size_t)s * B;
  const int32_t* t = tgt + (size_t)s * B;
  int a = 0;
  while (a + 1 < B && d[a + 1] == t[a]) ++a;
  accept_len[s] = a;
  for (int j = 0; j < B; ++j) out_tokens[(size_t)s * B + j] = (j < a) ? d[j + 1] : (j == a ? t[a] : -1);
}

// ---- speculative sampling ---------------------------------------------------------------------------
// Arrival counters of the sequences, `stride` apart, where the sweep over the vocabulary finishes by itself (finish.h); the statistics launch
// in front of it zeroes them.
struct AcceptArrive {
  unsigned* counters = nullptr;
  int n = 0, stride = 0;
};
// Softmax statistics of stored logits: part[row * gridDim.x + chunk] = (max, sum of exp(logit * inv_T - max)) over one
// chunk of the row; row r < R is row r of `a`, row R + r is row r of `b` (one launch for target and draft).  An empty set is
// (-inf, 0).  Bound by HBM: every logit is read once (running maximum per thread), and a row is shared out over gridDim.x
// workgroups, because a block's few rows alone leave most CUs without work.  VEC: V and both pointers allow 16-byte loads.
// Eight sequences of 16 rows, 151936 columns, both tensors (156 MB): 2 x 99 us as one 1024-thread workgroup per row and
// two sweeps over it, 27.6 us in this form (the anchors' draft rows left out; 29.4 with a branch per element for masked logits and bounds in
// every round), the logits being in the memory-side cache from the pass before; 5.5 TB/s whatever the chunks, eight a row or thirty-two.  The
// rows' log-sum-exp is off by 5.6e-8 rms and 2.6e-7 at worst, as with the library's exponential.
__device__ __forceinline__ void lse_merge(float& m, float& s, float m2, float s2) {   // union of two sets
  const float M = fmaxf(m, m2);
  s = (m == -INFINITY ? s : s * expf(m - M)) + (m2 == -INFINITY ? s2 : s2 * expf(m2 - M));   // an empty set's sum is 0 or NaN
  m = M;
}
template <bool VEC>
__global__ __launch_bounds__(256) void lse_partial_kernel(const float* __restrict__ a, const float* __restrict__ b, int R, int V, float inv_T,
                                                          float2* __restrict__ part, int B, AcceptArrive arrive) {
  const int r = blockIdx.y, chunk = blockIdx.x, n_chunks = gridDim.x;
  if (r == 0 && chunk == 0)
    for (int i = threadIdx.x; i < arrive.n; i += 256) arrive.counters[i * arrive.stride] = 0u;
  if (r >= R && (r - R) % B == 0) return;   // the anchor's draft row: nobody asks for its distribution
  const float* row = (r < R ? a + (size_t)r * V : b + (size_t)(r - R) * V);
  const int per = (((V + n_chunks - 1) / n_chunks) + 3) & ~3;
  const int i0 = min(V, chunk * per), i1 = min(V, i0 + per);
  constexpr int E = VEC ? 4 : 1, U = 5, ROUND = 256 * E * U;
  float m = -INFINITY, s = 0.f, s_left = 0.f;   // the sum, and what is left out of it (see ExpParts)
  auto round = [&](int i, auto whole_c) {
#pragma clang fp contract(off)   // the scaled logit is rounded before the maximum is taken off, as where the maximum was found
    constexpr bool WHOLE = decltype(whole_c)::value;
    float v[U * E];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int at = i + u * 256 * E;
      const bool in = WHOLE || at < i1;
      if constexpr (VEC) {
        const f32x4 x = in ? __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(row + at)) : (f32x4){-INFINITY, -INFINITY, -INFINITY, -INFINITY};
        v[4 * u] = x[0]; v[4 * u + 1] = x[1]; v[4 * u + 2] = x[2]; v[4 * u + 3] = x[3];
      } else {
        v[u] = in ? row[at] : -INFINITY;
      }
    }
    __builtin_amdgcn_sched_barrier(0);   // all loads of a round are out before the first is waited for
    float mx = m;
#pragma unroll
    for (int e = 0; e < U * E; ++e) {
      v[e] *= inv_T;
      mx = fmaxf(mx, v[e]);
    }
    if (mx > m) {
      const float f = expf(m - mx);   // nothing so far: 0
      s *= f;
      s_left *= f;
      m = mx;
    }
    const float base = m == -INFINITY ? 0.f : m;   // a masked logit weighs nothing, also where all are, a NaN stays one
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (!WHOLE && i + u * 256 * E >= i1) continue;   // a last round with little in it (16 x 5 rows of 128256: twelve columns a piece) pays for that only: the call 36.4 -> 32.7 us
#pragma unroll
      for (int e = u * E; e < (u + 1) * E; ++e) {
        const ExpParts x = exp_nonpositive_parts(v[e] - base, [](float p) { return __builtin_amdgcn_exp2f(p); });
        s += x.x;
        s_left = fmaf(x.x, x.left, s_left);
      }
    }
  };
  int c0 = i0;
  for (; c0 + ROUND <= i1; c0 += ROUND) round(c0 + (int)threadIdx.x * E, std::true_type{});
  if (c0 < i1) round(c0 + (int)threadIdx.x * E, std::false_type{});
  s = fmaf(s_left, kExpLn2, s);
  lane_xor16(m, s, [&](float om, float os) { lse_merge(m, s, om, os); });
#pragma unroll
  for (int o = 16; o < 64; o <<= 1) {
    const float om = __shfl_xor(m, o, 64), os = __shfl_xor(s, o, 64);
    lse_merge(m, s, om, os);
  }
  __shared__ float2 w[4];
  if ((threadIdx.x & 63) == 0) w[threadIdx.x >> 6] = make_float2(m, s);
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int i = 1; i < 4; ++i) lse_merge(m, s, w[i].x, w[i].y);
    part[(size_t)r * n_chunks + chunk] = make_float2(m, s);
  }
}

// combines the per-workgroup (max, sum) partials that the LM-head epilogue left for row m, in ascending order of the
// column blocks: stats[m] = (max, log-sum-exp) of logits * inv_T (from stored logits: lse_partial_kernel, row_lse)
__global__ __launch_bounds__(64) void lse_finish_kernel(const float2* __restrict__ part, int n_parts, float2* __restrict__ stats) {
  const int m = blockIdx.x, lane = threadIdx.x;
  float mx = -INFINITY;
#pragma unroll 8
  for (int c = lane; c < n_parts; c += 64) mx = fmaxf(mx, part[(size_t)m * n_parts + c].x);
  mx = wave_reduce_max(mx);
  // every lane sums its stride of the parts in ascending order, then the 64 lane sums are added in lane order
  float s = 0.f;
#pragma unroll 8
  for (int c = lane; c < n_parts; c += 64) {
    const float2 p = part[(size_t)m * n_parts + c];
    s += p.x == -INFINITY ? 0.f : p.y * expf(p.x - mx);
  }
  float tot = 0.f;
#pragma unroll
  for (int i = 0; i < 64; ++i) tot += lane_value(s, i);
  if (lane == 0) stats[m] = make_float2(mx, mx + logf(tot));
}

// Softmax statistics of a set of rows: parts == 0: p[row] = (max, log-sum-exp); parts > 0: p[row * parts ..] = the row's
// pieces (max, sum relative to that max).
struct RowStats {
  const float2* p;
  int parts;
};
// what lane `lane16` of the 16 that share a row begins with: its first piece
__device__ __forceinline__ float2 row_piece(const RowStats& st, size_t row, int lane16) {
  if (st.parts == 0) return st.p[row];
  return lane16 < st.parts ? st.p[row * st.parts + lane16] : make_float2(-INFINITY, 0.f);
}
// log-sum-exp of the row (the same value in each of the lanes)
__device__ __forceinline__ float row_lse(const RowStats& st, size_t row, int lane16, float2 first) {
  if (st.parts == 0) return first.y;
  float m = first.x, s = first.y;
  for (int c = lane16 + 16; c < st.parts; c += 16) {
    const float2 x = st.p[row * st.parts + c];
    lse_merge(m, s, x.x, x.y);
  }
  lane_xor16(m, s, [&](float om, float os) { lse_merge(m, s, om, os); });
  return m + logf(s);
}

// Stage 2, one wavefront per sequence: combines the chunks' bests (ties -> lowest index) and writes the sequence's tokens.
template <typename Best>
__device__ __forceinline__ void accept_finish(int lane, int n_chunks, int a, int B, const int32_t* draft, int32_t* out_tokens, Best best) {
  float bv = -INFINITY;
  int bi = 0x7FFFFFFF;
  for (int c = lane; c < n_chunks; c += 64) {
    const float2 x = best(c);
    argmax_combine(bv, bi, x.x, __float_as_int(x.y));
  }
  wave_argmax(bv, bi);
  if (lane < B) out_tokens[lane] = lane < a ? draft[lane + 1] : (lane == a ? bi : -1);
}

// Speculative sampling, stage 1.  grid (chunks, S).  The slots are tested side by side, lane j for slot j: slot j is accepted
// iff u_j * q_j(d_j) < p_{j-1}(d_j), the first one that is not ends the block.  Then the workgroup takes the best
// Gumbel-perturbed score of its columns for the token that follows the accepted ones,
//   first rejected slot j: log max(p_{j-1} - q_j, 0)   (purpose 1, slot j)
//   none rejected:         log p_{B-1}                 (purpose 2, slot B)
// into best[s * chunks + chunk]; the workgroup of chunk 0 writes accept_len.  Every workgroup of a sequence repeats the (small)
// test, so that the sweep over the vocabulary (two logarithms and a 64-bit hash per column) runs on as many CUs as there are: one
// workgroup per sequence took 124 us for eight sequences of 151936 columns, now 10.7, half of it arithmetic (a column costs some 600
// cycles of a SIMD).  With arrival counters the last workgroup of a sequence writes its tokens: 11.8 us for both stages, 10.7 + 3.9 as two
// launches; the whole call 40.2 -> 37.6 us, one sequence of ten rows of 16000 columns 15.7 -> 12.5.  (128 workgroups a sequence: 38.8.)
// A drafted id outside the vocabulary is never accepted.
__global__ __launch_bounds__(256) void accept_sampling_kernel(const float* __restrict__ p_logits, const float* __restrict__ q_logits,
                                                              RowStats p_stats, RowStats q_stats,
                                                              const int32_t* __restrict__ draft, const float* __restrict__ uniforms,
                                                              const uint64_t* __restrict__ rng_key, int V, int B, float inv_T,
                                                              int32_t* __restrict__ accept_len, float2* __restrict__ best,
                                                              int32_t* __restrict__ out_tokens, AcceptArrive arrive) {
  const int s = blockIdx.y, chunk = blockIdx.x, n_chunks = gridDim.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __shared__ float lse[2][16];   // log-sum-exp of the target rows, of the draft rows (B <= 16)
  __shared__ int sh_a;
  // Everything the test needs is requested at once: the pieces of the rows (sixteen lanes a row, the target's and the draft's), and in the first
  // wavefront the drafted tokens' own logits.
  const int r16 = threadIdx.x >> 4, lane16 = threadIdx.x & 15;
  const size_t row = (size_t)s * B + min(r16, B - 1);
  const float2 piece_p = row_piece(p_stats, row, lane16), piece_q = row_piece(q_stats, row, lane16);
  const uint64_t key = rng_key[0];
  const bool slot = wave == 0 && lane >= 1 && lane < B;
  int d = -1;
  float at_p = 0.f, at_q = 0.f, uniform = 0.f;
  if (slot) {
    d = draft[(size_t)s * B + lane];
    uniform = uniforms[(size_t)s * B + lane];
    const int col = min(max(d, 0), V - 1);
    at_p = p_logits[((size_t)s * B + lane - 1) * V + col];
    at_q = q_logits[((size_t)s * B + lane) * V + col];
  }
  const float lse_p = row_lse(p_stats, row, lane16, piece_p), lse_q = row_lse(q_stats, row, lane16, piece_q);
  if (lane16 == 0 && r16 < B) {
    lse[0][r16] = lse_p;
    lse[1][r16] = lse_q;   // of slot 0: not used
  }
  __syncthreads();
  if (wave == 0) {
    bool rejected = false;
    if (slot) {
      rejected = true;
      if (d >= 0 && d < V) {
        const float p = expf(at_p * inv_T - lse[0][lane - 1]);
        const float q = expf(at_q * inv_T - lse[1][lane]);
        rejected = !(uniform * q < p);
      }
    }
    const unsigned long long m = __builtin_amdgcn_ballot_w64(rejected);
    if (lane == 0) sh_a = m ? __builtin_ctzll(m) - 1 : B - 1;   // a rejection at slot j gives j-1 <= B-2
  }
  __syncthreads();
  const int a = sh_a;
  const int per = (V + n_chunks - 1) / n_chunks, i0 = min(V, chunk * per), i1 = min(V, i0 + per);
  float bv = -INFINITY;
  int bi = 0x7FFFFFFF;
  // the columns of U rounds are requested together: one at a time a workgroup's nine rounds were nine trips to memory
  constexpr int U = 10;
  const bool all = a == B - 1;
  const int j = all ? B - 1 : a + 1;   // the draft row (all: not used)
  const float* pr = p_logits + ((size_t)s * B + (all ? B - 1 : j - 1)) * V;
  const float* qr = q_logits + ((size_t)s * B + j) * V;
  const float lp = lse[0][all ? B - 1 : j - 1], lq = lse[1][j];
  for (int c0 = i0 + threadIdx.x; c0 < i1; c0 += 256 * U) {
    float p[U], q[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = min(c0 + u * 256, i1 - 1);   // past the end: the last column again, left out below
      p[u] = pr[i];
      q[u] = all ? 0.f : qr[i];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = c0 + u * 256;
      if (i >= i1) break;
      if (all) {
        argmax_combine(bv, bi, p[u] * inv_T - lp + gumbel(counter_uniform(key, s, B, 2, (uint32_t)i)), i);
      } else {
        const float r = expf(p[u] * inv_T - lp) - expf(q[u] * inv_T - lq);
        if (r > 0.f) argmax_combine(bv, bi, logf(r) + gumbel(counter_uniform(key, s, j, 1, (uint32_t)i)), i);
      }
    }
  }
  block_argmax(bv, bi);
  if (threadIdx.x == 0 && chunk == 0) accept_len[s] = a;
  if (!arrive.counters) {   // stage 2 is a launch of its own
    if (threadIdx.x == 0) best[(size_t)s * n_chunks + chunk] = make_float2(bv, __int_as_float(bi));
    return;
  }
  uint64_t* mine = reinterpret_cast<uint64_t*>(best + (size_t)s * n_chunks);
  if (threadIdx.x == 0)
    __hip_atomic_store(mine + chunk, (uint64_t)__float_as_uint(bv) | (uint64_t)(unsigned)bi << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (!last_to_arrive(arrive.counters + s * arrive.stride, (unsigned)n_chunks) || wave != 0) return;
  accept_finish(lane, n_chunks, a, B, draft + (size_t)s * B, out_tokens + (size_t)s * B, [&](int c) {
    const uint64_t x = __hip_atomic_load(mine + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_float2(__uint_as_float((unsigned)x), __uint_as_float((unsigned)(x >> 32)));
  });
}

__global__ __launch_bounds__(64) void accept_sampling_finish_kernel(const float2* __restrict__ best, int n_chunks, const int32_t* __restrict__ draft,
                                                                    int B, const int32_t* __restrict__ accept_len, int32_t* __restrict__ out_tokens) {
  const int s = blockIdx.x;
  accept_finish(threadIdx.x, n_chunks, accept_len[s], B, draft + (size_t)s * B, out_tokens + (size_t)s * B,
                [&](int c) { return best[(size_t)s * n_chunks + c]; });
}

// ---- commit bookkeeping ----------------------------------------------------------------------------
__global__ void commit_update_kernel(SeqGeom geo, int32_t* __restrict__ seq_lens, int32_t* __restrict__ anchor,
                                     const int32_t* __restrict__ accept_len, const int32_t* __restrict__ out_tokens, int S,
                                     int64_t* __restrict__ kv_slots) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= S) return;
  const int B = geo.block_size;
  const int n = seq_lens[s];
  int a = accept_len[s];
  a = max(-1, min(a, B - 1));   // -1: nothing of this sequence is committed, anchor kept
  if (kv_slots) {
    for (int j = 0; j < B; ++j) {
      int64_t slot = -1;
      const int pos = n + j, pidx = pos / DF_PAGE;
      if (j <= a && pidx < geo.max_pages_per_seq) {
        const int page = geo.block_table[(size_t)s * geo.max_pages_per_seq + pidx];
        if (page >= 0 && page < geo.n_pages) slot = (int64_t)page * DF_PAGE + pos % DF_PAGE;
      }
      kv_slots[(size_t)s * B + j] = slot;
    }
  }
  if (a >= 0) anchor[s] = out_tokens[(size_t)s * B + a];
  seq_lens[s] = n + a + 1;
}

// ---- weight packing ---------------------------------------------------------------------------------
// dst row r of the packed matrix comes from source matrix/row:
//   mode 0 (concat):      sources stacked in order
//   mode 1 (interleave):  16 rows of src0, 16 rows of src1, 16 rows of src0, ...
struct PackSrc {
  const void* src[3];
  int rows[3];
  int n_src;
  int mode;
};
template <typename T>
__global__ __launch_bounds__(256) void pack_kernel(PackSrc ps, int K, int total_rows, T* __restrict__ dst, int dst_row0,
                                                   int dst_rows) {
  const size_t chunk = (size_t)blockIdx.x * blockDim.x + threadIdx.x;  // one 8-element chunk
  const int chunks_per_row = K >> 3;
  const size_t n_chunks = (size_t)total_rows * chunks_per_row;
  if (chunk >= n_chunks) return;
  const int r = (int)(chunk / chunks_per_row), k = (int)(chunk % chunks_per_row) * 8;
  int si = 0, sr = r;
  if (ps.mode == 1) {
    si = (r >> 4) & 1;
    sr = ((r >> 5) << 4) + (r & 15);
  } else {
    while (si + 1 < ps.n_src && sr >= ps.rows[si]) { sr -= ps.rows[si]; ++si; }
  }
  const T* s = reinterpret_cast<const T*>(ps.src[si]) + (size_t)sr * K + k;
  T* d = dst + tile_index<T>(dst_row0 + r, k, K, dst_rows);   // rows land at dst_row0.. of a dst_rows-row matrix
#pragma unroll
  for (int i = 0; i < 8; ++i) d[i] = s[i];
}

// ---- KV import / export -------------------------------------------------------------------------------
// dir 0: pool -> canonical fp32 [count, Hkv, hd]; dir 1: canonical -> pool
template <typename T>
__global__ __launch_bounds__(128) void kv_copy_kernel(T* __restrict__ pool, SeqGeom geo, int layer, int n_kv_heads, int hd, int seq,
                                                      int start, float* __restrict__ k, float* __restrict__ v, int dir) {
  const int pos = start + blockIdx.x, kvh = blockIdx.y;
  const int pidx = pos / DF_PAGE;
  if (pidx >= geo.max_pages_per_seq) return;
  const int page = geo.block_table[(size_t)seq * geo.max_pages_per_seq + pidx];
  if (page < 0 || page >= geo.n_pages) return;
  T* base = pool + kv_head_base(layer, geo.n_pages, page, n_kv_heads, kvh, hd);
  const int key = pos % DF_PAGE;
  const size_t row = ((size_t)blockIdx.x * n_kv_heads + kvh) * hd;
  for (int d = threadIdx.x; d < hd; d += blockDim.x) {
    if (dir == 0) {
      k[row + d] = Store<T>::to(base[k_in_page(key, d)]);
      v[row + d] = Store<T>::to(base[DF_PAGE * hd + v_in_page(key, d)]);
    } else {
      base[k_in_page(key, d)] = Store<T>::from(k[row + d]);
      base[DF_PAGE * hd + v_in_page(key, d)] = Store<T>::from(v[row + d]);
    }
  }
}

// ---- machine probes ---------------------------------------------------------------------------------
// where the probes drop a value when an impossible condition holds, so that the compiler keeps their work
__device__ unsigned g_probe_sink;

// read-only streaming: wavefronts interleave 8 KB pieces across the whole grid
__global__ __launch_bounds__(256) void probe_read_kernel(const u32x4* __restrict__ p, size_t n_chunks) {
  const size_t wave = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6, lane = threadIdx.x & 63;
  const size_t n_waves = ((size_t)gridDim.x * blockDim.x) >> 6;
  unsigned acc = 0;
  for (size_t c = wave * 8; c < n_chunks; c += n_waves * 8) {
    u32x4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = __builtin_nontemporal_load(p + (c + u < n_chunks ? c + u : c) * 64 + lane);
#pragma unroll
    for (int u = 0; u < 8; ++u) acc ^= v[u][0] ^ v[u][3];
  }
  if (acc == 0x12345677u) g_probe_sink = acc;   // keeps the loads alive; practically never true
}

__global__ __launch_bounds__(256) void probe_mfma_kernel(int iters) {
  const u32x4 a = {threadIdx.x, 1u, 2u, 3u}, b = {4u, 5u, threadIdx.x, 7u};
  f32x4 acc[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int i = 0; i < 16; ++i)
      acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc[i], 0, 0, 0);
  }
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) s += acc[i][0] + acc[i][1] + acc[i][2] + acc[i][3];
  if (s == 12345.678f) g_probe_sink = 1u;   // keeps the MFMAs alive
}

typedef float probe_f32x16 __attribute__((ext_vector_type(16)));
__global__ __launch_bounds__(256) void probe_mfma32_kernel(int iters) {
  const u32x4 a = {threadIdx.x, 1u, 2u, 3u}, b = {4u, 5u, threadIdx.x, 7u};
  probe_f32x16 acc[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc[i], 0, 0, 0);
  }
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) s += acc[i][e];
  if (s == 12345.678f) g_probe_sink = 1u;   // keeps the MFMAs alive
}

// ---- prefill as a many-row pass (Section 4.1: the standard prefill gives the first token and the target's hidden
// features of every prompt token) ------------------------------------------------------------------------------
// The new tokens of all prompts are cut into chunks of B rows; chunk c (counted over all prompts, in order) becomes
// pseudo-sequence c - chunk0 of one verification-shaped pass: committed length = the prompt's cached length + the
// chunk's offset, block-table row = the prompt's.  Inside a layer every K/V row is in the pages before attention runs,
// so the causal block attention of the chunks is a causal prefill.  One workgroup per pseudo-sequence.
struct PrefillPlan {
  const int32_t* lens;         // [S] new tokens per prompt (device copy of the host's array)
  const int32_t* seq_lens;     // [S] tokens already cached
  const int32_t* block_table;  // [S, mpps]
  const int32_t* tokens;       // new tokens of all prompts, concatenated
  int S, B, mpps, chunk0, n_chunks;
  int32_t* p_lens;             // [n_chunks]
  int32_t* p_table;            // [n_chunks, mpps]
  int32_t* p_tokens;           // [n_chunks, B], zero-padded
  int32_t* end_row;            // [.] row (in this pass) of the last token of every prompt that ends in this pass, in prompt order
  int32_t* end_seq;            // [.] and that prompt's index
  int4* tiles;                 // [.] pairs of consecutive pseudo-sequences of a prompt: (first, how many, tokens before, -), in order; see prefill_tiles
};

__global__ __launch_bounds__(256) void prefill_plan_kernel(PrefillPlan p) {
  const int i = blockIdx.x, c = p.chunk0 + i;
  __shared__ int sh[4];
  if (threadIdx.x == 0) {
    int first = 0, s = 0, n_end_before = 0, n_tiles = 0;
    for (; s < p.S; ++s) {
      const int nc = (p.lens[s] + p.B - 1) / p.B;
      const int from = max(first, p.chunk0), to = min(first + nc, p.chunk0 + p.n_chunks);   // its chunks in this pass
      if (c < first + nc) {
        if (((c - from) & 1) == 0) p.tiles[n_tiles + ((c - from) >> 1)] = make_int4(i, min(2, to - c), p.seq_lens[s] + (c - first) * p.B, 0);
        break;
      }
      n_tiles += prefill_tiles(to - from);
      // a prompt before ours whose last chunk lies in this pass takes an earlier place in the end list
      if (nc > 0 && first + nc - 1 >= p.chunk0) ++n_end_before;
      first += nc;
    }
    sh[0] = s;
    sh[1] = (c - first) * p.B;       // offset of the chunk inside the prompt's new tokens
    sh[2] = n_end_before;
    int tok0 = 0;
    for (int t = 0; t < s && t < p.S; ++t) tok0 += p.lens[t];
    sh[3] = tok0;
  }
  __syncthreads();
  const int s = sh[0], off = sh[1];
  if (s >= p.S) return;              // cannot happen when the host counted the chunks from the same lengths
  const int len = p.lens[s], rows = min(p.B, len - off);
  for (int j = threadIdx.x; j < p.mpps; j += blockDim.x) p.p_table[(size_t)i * p.mpps + j] = p.block_table[(size_t)s * p.mpps + j];
  for (int j = threadIdx.x; j < p.B; j += blockDim.x) p.p_tokens[(size_t)i * p.B + j] = j < rows ? p.tokens[sh[3] + off + j] : 0;
  if (threadIdx.x == 0) {
    p.p_lens[i] = p.seq_lens[s] + off;
    if (off + rows == len) {
      p.end_row[sh[2]] = i * p.B + rows - 1;
      p.end_seq[sh[2]] = s;
    }
  }
}

// out row r (GEMM operand, row length K) = row rows[r] of `a`
template <typename T>
__global__ __launch_bounds__(256) void gather_operand_rows_kernel(const T* __restrict__ a, const int32_t* __restrict__ rows, T* __restrict__ out, int K) {
  const int r = blockIdx.x, m = rows[r];
  for (int k = threadIdx.x; k < K; k += blockDim.x) {
    if constexpr (sizeof(T) == 2) {
      const size_t src = Act<bf16_t>::index(m, k, K), dst = Act<bf16_t>::index(r, k, K);
      out[dst] = a[src];
      out[dst + 512] = a[src + 512];
    } else {
      out[(size_t)r * K + k] = a[(size_t)m * K + k];
    }
  }
}

// first generated token of the prompts that ended in a pass: anchor and (optionally) the caller's array
__global__ void prefill_first_kernel(const int32_t* __restrict__ first, const int32_t* __restrict__ end_seq, int n_end, int32_t* anchor,
                                     int32_t* first_out) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n_end) return;
  const int s = end_seq[r];
  anchor[s] = first[r];
  if (first_out) first_out[s] = first[r];
}

__global__ void prefill_advance_kernel(int32_t* seq_lens, const int32_t* __restrict__ lens, int S) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s < S) seq_lens[s] += lens[s];
}
