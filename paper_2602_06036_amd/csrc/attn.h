// Block attention over the paged cache, split along the context ("split-KV") with a deterministic
// log-sum-exp merge.  Used for both halves of the step:
//   verify (Section 3.1): causal -- block row j sees positions 0 .. n_s + j
//   draft  (Section 4.2, Appendix A.3): no mask -- every block row sees the n_s context-feature rows
//                                       and all B block rows (positions 0 .. n_s + B - 1)
// In both cases the block's own K/V rows have already been written to the pool at n_s .. n_s+B-1.
#pragma once
#include "common.h"

struct AttnArgs {
  int n_q_heads, n_kv_heads, head_dim;
  int layer;     // layer inside the pool
  int causal;
  int chunk;     // context tokens per split (multiple of 64)
  int n_splits;
  float scale;   // 1/sqrt(head_dim)
  int q_shift = 0;   // MFMA kernels: the query heads of one kv head are shared out over 2^q_shift workgroups (a workgroup
                     // holds at most 64 query rows = block_size * heads; 8 heads per kv head at block size 16 need two)
  void* out = nullptr;   // MFMA kernels, n_splits == 1: the finished rows go here (GEMM operand, row length Hq*hd), no merge follows
};

// A row that sees no key is zeros: its sums are, and they are divided by infinity where there is no positive sum of exponentials.  A NaN among a
// row's scores is a NaN in the products with V whatever else it sees (maxima pass NaN over, sums do not, and a weight of zero keeps it), so the
// row is NaN, in every kernel and however its context is split.
// partial results: for pr = (m*Hq + hq)*n_splits + split : ml[pr] = (running max, sum exp), o[pr*hd + d]
// (o unnormalised, relative to the running max)

// ------------------------------------------------------------------------------------------------
// Generic kernel (any storage type; plain ALU math).  grid (n_splits, Hkv * row groups, S), block 256.
// A wavefront takes query rows r = group * 4 + wave, + 4 * groups, ... of the B*group rows that share this kv head.
// Bound by latency: a chunk is 64 keys or little more, so what counts is that nothing waits that need not.  A lane owns a
// key for the scores and one or two head dims for P.V; the 64 V rows of a tile are requested together, four keys a load,
// before their weights are known (8 rows, 136 keys, 4 heads of 64, fp32: 35.9 us with one dependent load per key, 8.9 us like this).
// ------------------------------------------------------------------------------------------------
// 4 consecutive keys of one head dim of a page, as they are stored.  (As floats a tile's V rows took 128 registers of bf16 kernels too and
// were waited for one by one to be converted; with the sweep in a function of its own those kernels then came out with 257 registers and one
// wavefront a SIMD: 512 rows, 4 heads of 96, 2000 keys 680 us a two-layer pass before, 1220 with one wavefront, 443 like this; 64 rows
// 148, 197 and 131.)
template <typename T> struct Keys4 { using Raw = float4; };
template <> struct Keys4<bf16_t> { using Raw = ushort4; };
template <typename T>
__device__ __forceinline__ typename Keys4<T>::Raw load_keys4(const T* p) { return *reinterpret_cast<const typename Keys4<T>::Raw*>(p); }
__device__ __forceinline__ float4 keys4_to_float(float4 v) { return v; }
__device__ __forceinline__ float4 keys4_to_float(ushort4 u) {
  return make_float4(Store<bf16_t>::to(u.x), Store<bf16_t>::to(u.y), Store<bf16_t>::to(u.z), Store<bf16_t>::to(u.w));
}

// One wavefront's sweep of a query row (in LDS, qs) over the 64-key tiles first, first + step, ... below c1: running max, sum of
// exponentials and this lane's one or two head dims (d0, d1) of the unnormalised output.
struct SimpleRow {
  float m_run = -INFINITY, l_run = 0.f, o0 = 0.f, o1 = 0.f;
};
template <typename T>
__device__ __forceinline__ SimpleRow attn_simple_sweep(const float* qs, const T* __restrict__ pool, const SeqGeom& geo, const AttnArgs& aa,
                                                       const int32_t* table, int kvh, int first, int step, int c1, int last_vis, int lane, int d0,
                                                       int d1) {
  const int hd = aa.head_dim;
  SimpleRow row;
  for (int t0 = first; t0 < c1; t0 += step) {
    const int pos = t0 + lane;
    const bool vis = pos < c1 && pos <= last_vis;
    int page = -1;
    if (pos < c1) page = table[pos / DF_PAGE];
    const bool page_ok = page >= 0 && page < geo.n_pages;
    const bool ok = vis && page_ok;
    const int any_page = page_ok ? page : 0;     // a page that may be read; keys behind it then weigh nothing
    // the tile's V rows (t0 is a multiple of 64: four whole pages), on their way while the scores are computed
    typename Keys4<T>::Raw v0[16], v1[16];
#pragma unroll
    for (int pg = 0; pg < 4; ++pg) {
      const T* vb = pool + kv_head_base(aa.layer, geo.n_pages, __builtin_amdgcn_readlane(any_page, pg * 16), aa.n_kv_heads, kvh, hd) + DF_PAGE * hd;
#pragma unroll
      for (int k4 = 0; k4 < 4; ++k4) {
        v0[pg * 4 + k4] = load_keys4(vb + v_in_page(k4 * 4, d0));
        if (hd > 64) v1[pg * 4 + k4] = load_keys4(vb + v_in_page(k4 * 4, d1));
      }
    }
    float sc = -INFINITY;
    {
      const T* kb = pool + kv_head_base(aa.layer, geo.n_pages, any_page, aa.n_kv_heads, kvh, hd);
      const int key = pos % DF_PAGE;
      float acc = 0.f;
#pragma unroll 4
      for (int d = 0; d < hd; d += 8) {
        const T* kp = kb + k_in_page(key, d);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc += qs[d + e] * Store<T>::to(kp[e]);
      }
      if (ok) sc = acc * aa.scale;
    }
    // A tile with nothing to see is left out, one with a NaN is not.  Asked ahead of the maximum, the fp32 kernels come out with 218 registers
    // (asked of the maximum with 256 and one wavefront a SIMD; two-layer passes of width 256 with 32 to 256 keys: 8 rows 57 us so and 52 ahead of
    // it, 2048 rows 933 and 664), but the bf16 ones load their K rows one by one (64 rows, head dim 96: 82 and 88).  There the maximum is
    // asked, in which a NaN then has to show.
    constexpr bool ask_first = sizeof(T) == 4;
    if (ask_first && __builtin_amdgcn_ballot_w64(!(sc == -INFINITY)) == 0ull) continue;
    const float tmax = wave_reduce_max(!ask_first && sc != sc ? INFINITY : sc);
    if (!ask_first && tmax == -INFINITY) continue;   // uniform across the wavefront
    const float m_new = fmaxf(row.m_run, tmax);
    const float corr = (row.m_run == -INFINITY) ? 0.f : expf(row.m_run - m_new);
    const float p = ok ? expf(sc - m_new) : 0.f;
    row.l_run = row.l_run * corr + wave_reduce_sum(p);
    row.o0 *= corr;
    row.o1 *= corr;
    row.m_run = m_new;
    // a key that weighs nothing is left out whatever its V row holds (never written, or another sequence's)
    auto add = [&](float& o, float pk, float v) { o += pk == 0.f ? 0.f : pk * v; };
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float p0 = __shfl(p, 4 * i, 64), p1 = __shfl(p, 4 * i + 1, 64), p2 = __shfl(p, 4 * i + 2, 64), p3 = __shfl(p, 4 * i + 3, 64);
      const float4 a = keys4_to_float(v0[i]);
      add(row.o0, p0, a.x); add(row.o0, p1, a.y); add(row.o0, p2, a.z); add(row.o0, p3, a.w);
      if (hd > 64) {
        const float4 b = keys4_to_float(v1[i]);
        add(row.o1, p0, b.x); add(row.o1, p1, b.y); add(row.o1, p2, b.z); add(row.o1, p3, b.w);
      }
    }
  }
  return row;
}

template <typename T>
__global__ __launch_bounds__(256, 2) void attn_partial_simple_kernel(const T* __restrict__ q, const T* __restrict__ pool,
                                                                  SeqGeom geo, AttnArgs aa, float* __restrict__ part_o,
                                                                  float2* __restrict__ part_ml) {
  const int split = blockIdx.x, kvh = (int)blockIdx.y % aa.n_kv_heads, s = blockIdx.z;
  const int row_group = (int)blockIdx.y / aa.n_kv_heads, row_groups = (int)gridDim.y / aa.n_kv_heads;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int hd = aa.head_dim, B = geo.block_size;
  const int group = aa.n_q_heads / aa.n_kv_heads;
  const int rows = B * group;
  const int n_s = geo.seq_lens[s];
  const int cap = geo.max_pages_per_seq * DF_PAGE;
  const int n_tok = min(n_s + B, cap);
  const int c0 = split * aa.chunk;
  const int c1 = min(n_tok, c0 + aa.chunk);
  __shared__ float qs[4][128];
  const int32_t* table = geo.block_table + (size_t)s * geo.max_pages_per_seq;
  const int d0 = min(lane, hd - 1), d1 = min(lane + 64, hd - 1);   // this lane's head dims (clamped: not stored)

  for (int r = row_group * 4 + wave; r < rows; r += 4 * row_groups) {
    const int slot = r / group, hq = kvh * group + r % group;
    const int m = s * B + slot;
    const size_t pr = ((size_t)m * aa.n_q_heads + hq) * aa.n_splits + split;
    const T* qrow = q + ((size_t)m * aa.n_q_heads + hq) * hd;
    for (int d = lane; d < hd; d += 64) qs[wave][d] = Store<T>::to(qrow[d]);
    // (same wavefront writes and reads qs[wave]; LDS ops of one wavefront complete in order)
    const int last_vis = aa.causal ? min(n_s + slot, n_tok - 1) : n_tok - 1;
    const SimpleRow o = attn_simple_sweep<T>(qs[wave], pool, geo, aa, table, kvh, c0, 64, c1, last_vis, lane, d0, d1);
    if (lane == 0) part_ml[pr] = make_float2(o.m_run, o.l_run);
    if (lane < hd) part_o[pr * hd + lane] = o.o0;
    if (lane + 64 < hd) part_o[pr * hd + lane + 64] = o.o1;
  }
}

// Short contexts (short_context in plan.h): a workgroup per query row, its four wavefronts share the keys and merge in LDS, and the row
// is finished: 8.7 us at 136 keys, 8 rows, 4 heads of 64, against 9.6 and a merge launch of 3.6 (with 256 registers; 6.6 with 218).  grid (B * group, Hkv, S).
template <typename T>
__global__ __launch_bounds__(256, 2) void attn_short_simple_kernel(const T* __restrict__ q, const T* __restrict__ pool, SeqGeom geo, AttnArgs aa,
                                                                T* __restrict__ out) {
  const int kvh = blockIdx.y, s = blockIdx.z;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int hd = aa.head_dim, B = geo.block_size, group = aa.n_q_heads / aa.n_kv_heads;
  const int slot = (int)blockIdx.x / group, hq = kvh * group + (int)blockIdx.x % group, m = s * B + slot;
  __shared__ float qs[4][128], so[4][128];
  __shared__ float2 sml[4];
  const T* qrow = q + ((size_t)m * aa.n_q_heads + hq) * hd;
  for (int d = lane; d < hd; d += 64) qs[wave][d] = Store<T>::to(qrow[d]);
  const int n_s = geo.seq_lens[s], n_tok = min(n_s + B, geo.max_pages_per_seq * DF_PAGE);
  const int last_vis = aa.causal ? min(n_s + slot, n_tok - 1) : n_tok - 1;
  const int c1 = min(n_tok, aa.chunk);   // the hint bounds the sweep, as it does the splits'
  const SimpleRow o = attn_simple_sweep<T>(qs[wave], pool, geo, aa, geo.block_table + (size_t)s * geo.max_pages_per_seq, kvh, wave * 64, 256, c1,
                                           last_vis, lane, min(lane, hd - 1), min(lane + 64, hd - 1));
  if (lane == 0) sml[wave] = make_float2(o.m_run, o.l_run);
  if (lane < hd) so[wave][lane] = o.o0;
  if (lane + 64 < hd) so[wave][lane + 64] = o.o1;
  __syncthreads();
  const int d = threadIdx.x;
  if (d >= hd) return;
  float mx = -INFINITY, L = 0.f, x = 0.f;
#pragma unroll
  for (int w = 0; w < 4; ++w) mx = fmaxf(mx, sml[w].y > 0.f ? sml[w].x : -INFINITY);
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const float2 ml = sml[w];
    const float e = ml.y > 0.f ? expf(ml.x - mx) : 0.f;
    L += ml.y * e;
    x += e * so[w][d];
  }
  Act<T>::store(out, m, hq * hd + d, aa.n_q_heads * hd, x / (L > 0.f ? L : INFINITY));
}

// ------------------------------------------------------------------------------------------------
// Merge of the splits in ascending split order, few rows (M < 128, where the number of workgroups matters more than
// the shape of the stores): grid (M*Hq), block 128 (one thread per head dim).
// The (max, sum) pairs are fetched by the first wavefront with one load per split, the partial
// outputs with independent loads four at a time, so the kernel is not a chain of dependent loads.
// Output as GEMM activation operand (Act<T>), row length Hq*hd.  n_splits <= 64.
// ------------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(128) void attn_merge_rows_kernel(const float* __restrict__ part_o, const float2* __restrict__ part_ml,
                                                         T* __restrict__ out, int n_q_heads, int hd, int n_splits) {
  const int row = blockIdx.x;  // m*Hq + hq
  const int m = row / n_q_heads, hq = row % n_q_heads;
  const int d = threadIdx.x;
  __shared__ float wgt[64];
  __shared__ float s_L;
  // the first PRE splits' outputs are requested before the weights are known: their loads do not depend on the
  // (max, sum) loads, so the two memory round trips overlap instead of following each other
  constexpr int PRE = 20;
  float pre[PRE];
  const float* po = part_o + (size_t)row * n_splits * hd + (d < hd ? d : 0);
#pragma unroll
  for (int c = 0; c < PRE; ++c) pre[c] = c < n_splits ? po[(size_t)c * hd] : 0.f;
  if (threadIdx.x < 64) {
    const int c = threadIdx.x;
    float2 ml = make_float2(-INFINITY, 0.f);
    if (c < n_splits) ml = part_ml[(size_t)row * n_splits + c];
    const float mx = wave_reduce_max(ml.y > 0.f ? ml.x : -INFINITY);
    const float w = (ml.y > 0.f) ? expf(ml.x - mx) : 0.f;
    wgt[c] = w;
    // sum in ascending split order (fixed order, independent of the wavefront reduction tree)
    float L = 0.f;
    for (int i = 0; i < n_splits; ++i) L += lane_value(ml.y * w, i);
    if (c == 0) s_L = L;
  }
  __syncthreads();
  if (d < hd) {
    float o = 0.f;
#pragma unroll
    for (int c = 0; c < PRE; ++c)
      if (c < n_splits) o += wgt[c] * pre[c];
    int c = PRE;
    for (; c + 4 <= n_splits; c += 4) {
      const float a0 = po[(size_t)(c + 0) * hd], a1 = po[(size_t)(c + 1) * hd], a2 = po[(size_t)(c + 2) * hd], a3 = po[(size_t)(c + 3) * hd];
      o += wgt[c] * a0;
      o += wgt[c + 1] * a1;
      o += wgt[c + 2] * a2;
      o += wgt[c + 3] * a3;
    }
    for (; c < n_splits; ++c) o += wgt[c] * po[(size_t)c * hd];
    const float L = s_L;
    Act<T>::store(out, m, hq * hd + d, n_q_heads * hd, o / (L > 0.f ? L : INFINITY));
  }
}

// ------------------------------------------------------------------------------------------------
// Merge of the splits in ascending split order.  One workgroup per (band of 16 rows, query head): thread
// (r = tid % 16, c = tid / 16) owns 4 head dims of row r, so that the 16 rows of a band write one contiguous piece
// of the operand tile (the band's rows are interleaved inside a tile) instead of scattered 2-byte stores.
// grid (ceil(M/16), Hq), block 16 * hd/4.  The (max, sum) pairs of a row are fetched by one wavefront with one
// load per split; the partial outputs are requested before the weights are known (their loads do not depend on
// the (max, sum) loads, so the two memory round trips overlap).  Output as GEMM activation operand (Act<T>), row
// length Hq*hd.  n_splits <= 64.
// ------------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(512) void attn_merge_kernel(const float* __restrict__ part_o, const float2* __restrict__ part_ml,
                                                         T* __restrict__ out, int n_q_heads, int hd, int n_splits, int M) {
  const int r = threadIdx.x & 15, c = threadIdx.x >> 4, hq = blockIdx.y;
  const int m_raw = blockIdx.x * 16 + r;
  const bool live = m_raw < M;
  const int m = live ? m_raw : M - 1;
  __shared__ float wgt[16][64];
  __shared__ float s_L[16];
  constexpr int PRE = 8;
  float4 pre[PRE];
  const float* po = part_o + ((size_t)m * n_q_heads + hq) * n_splits * hd + c * 4;
#pragma unroll
  for (int i = 0; i < PRE; ++i) pre[i] = i < n_splits ? *reinterpret_cast<const float4*>(po + (size_t)i * hd) : make_float4(0.f, 0.f, 0.f, 0.f);
  {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n_waves = blockDim.x >> 6;
    for (int rr = wave; rr < 16; rr += n_waves) {
      const int mm = min(blockIdx.x * 16 + rr, M - 1);
      float2 ml = make_float2(-INFINITY, 0.f);
      if (lane < n_splits) ml = part_ml[((size_t)mm * n_q_heads + hq) * n_splits + lane];
      const float mx = wave_reduce_max(ml.y > 0.f ? ml.x : -INFINITY);
      const float w = (ml.y > 0.f) ? expf(ml.x - mx) : 0.f;
      wgt[rr][lane] = w;
      // sum in ascending split order (fixed order, independent of the wavefront reduction tree)
      float L = 0.f;
      for (int i = 0; i < n_splits; ++i) L += lane_value(ml.y * w, i);
      if (lane == 0) s_L[rr] = L;
    }
  }
  __syncthreads();
  float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int i = 0; i < PRE; ++i)
    if (i < n_splits) {
      const float w = wgt[r][i];
      o.x += w * pre[i].x; o.y += w * pre[i].y; o.z += w * pre[i].z; o.w += w * pre[i].w;
    }
  int i = PRE;
  for (; i + 4 <= n_splits; i += 4) {
    float4 a[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) a[u] = *reinterpret_cast<const float4*>(po + (size_t)(i + u) * hd);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float w = wgt[r][i + u];
      o.x += w * a[u].x; o.y += w * a[u].y; o.z += w * a[u].z; o.w += w * a[u].w;
    }
  }
  for (; i < n_splits; ++i) {
    const float4 a = *reinterpret_cast<const float4*>(po + (size_t)i * hd);
    const float w = wgt[r][i];
    o.x += w * a.x; o.y += w * a.y; o.z += w * a.z; o.w += w * a.w;
  }
  if (live) {
    const float L = s_L[r] > 0.f ? s_L[r] : INFINITY;
    Act<T>::store4(out, m, hq * hd + c * 4, n_q_heads * hd, make_float4(o.x / L, o.y / L, o.z / L, o.w / L));
  }
}
