// MFMA block attention for bf16 caches (see attn.h for the split / merge contract).
//
// One workgroup = one (split, kv head, sequence): the B*group query rows that share the kv head
// (<= 64) against the chunk's keys.  Wavefront w owns query rows 16w .. 16w+15 for the whole chunk, so
// the four wavefronts never have to be merged; they read the same K/V tiles (the second to fourth read
// hit the CU's L1) and the next 32-key page pair is in flight while the current one is processed.
//
// Everything streams from the pool in MFMA operand order (page layout in common.h), nothing is
// transposed:  S^T = K . Q^T   (A = 16 keys x 32 dims of a page, B = Q^T), so a lane ends up with
//              4 consecutive keys of one query column for each of the two pages -- exactly the 8
//              k-slots it must supply as B operand of  O^T += V^T . P^T  (A = 16 dims x 32 keys).
// P is fed as a hi+lo bf16 pair (two MFMAs) so that the attention output keeps ~16 significant bits,
// like every other GEMM input of the bf16 model.
#pragma once
#include "attn.h"

template <int HD>
struct KvFrags {
  u32x4 ka[HD / 32], kb[HD / 32];
  u32x4 v[HD / 16];   // (4 keys of page A, 4 keys of page B) x one dim per lane: the A operand of P.V
  int ok_a, ok_b;
};

struct AttnLane {          // per-lane constants of the kernel below
  int c0, c1, n_tok, last_vis, g, lane, kvh;
};

// issues the loads of the page pair p of the chunk; pa, pb: its page ids (a foreign or missing page aliases a readable one)
template <int HD>
__device__ __forceinline__ void attn_load_pair(KvFrags<HD>& f, int p, int pa, int pb, const bf16_t* __restrict__ pool, const SeqGeom& geo,
                                               const AttnArgs& aa, const AttnLane& L) {
  const bool has_b = L.c0 + p * 32 + 16 < L.c1;
  f.ok_a = pa >= 0 && pa < geo.n_pages;
  if (!f.ok_a) pa = 0;
  f.ok_b = has_b && pb >= 0 && pb < geo.n_pages;
  if (!f.ok_b) pb = pa;
  const bf16_t* ka = pool + kv_head_base(aa.layer, geo.n_pages, pa, aa.n_kv_heads, L.kvh, HD);
  const bf16_t* kb = pool + kv_head_base(aa.layer, geo.n_pages, pb, aa.n_kv_heads, L.kvh, HD);
#pragma unroll
  for (int kt = 0; kt < HD / 32; ++kt) {
    f.ka[kt] = reinterpret_cast<const u32x4*>(ka)[kt * 64 + L.lane];
    f.kb[kt] = reinterpret_cast<const u32x4*>(kb)[kt * 64 + L.lane];
  }
#pragma unroll
  for (int dt = 0; dt < HD / 16; ++dt) {
    const uint2 a = reinterpret_cast<const uint2*>(ka + DF_PAGE * HD)[dt * 64 + L.lane];
    const uint2 b = reinterpret_cast<const uint2*>(kb + DF_PAGE * HD)[dt * 64 + L.lane];
    f.v[dt] = (u32x4){a.x, a.y, b.x, b.y};
  }
}

template <int HD>
__device__ __forceinline__ void attn_process_pair(KvFrags<HD>& f, int p, const u32x4 (&qf)[HD / 32], f32x4 (&acc)[HD / 16],
                                                  float& m_run, float& l_run, float scale, const AttnLane& L) {
  constexpr int KT = HD / 32, DT = HD / 16;
  const int base = L.c0 + p * 32;
  // rows at or beyond n_tok were never written (and an invalid page is not ours): 0 * garbage must not
  // become NaN, so clear those V elements.  Only the last pair of a sequence takes this path.
  if (base + 32 > L.n_tok || !f.ok_a || !f.ok_b) {
    const int pos_a = base + 4 * L.g, pos_b = base + 16 + 4 * L.g;
    uint32_t ma0 = 0u, ma1 = 0u, mb0 = 0u, mb1 = 0u;
    if (f.ok_a && pos_a + 0 < L.n_tok) ma0 |= 0x0000FFFFu;
    if (f.ok_a && pos_a + 1 < L.n_tok) ma0 |= 0xFFFF0000u;
    if (f.ok_a && pos_a + 2 < L.n_tok) ma1 |= 0x0000FFFFu;
    if (f.ok_a && pos_a + 3 < L.n_tok) ma1 |= 0xFFFF0000u;
    if (f.ok_b && pos_b + 0 < L.n_tok) mb0 |= 0x0000FFFFu;
    if (f.ok_b && pos_b + 1 < L.n_tok) mb0 |= 0xFFFF0000u;
    if (f.ok_b && pos_b + 2 < L.n_tok) mb1 |= 0x0000FFFFu;
    if (f.ok_b && pos_b + 3 < L.n_tok) mb1 |= 0xFFFF0000u;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      f.v[dt] &= (u32x4){ma0, ma1, mb0, mb1};
    }
  }
  f32x4 sa = {0.f, 0.f, 0.f, 0.f}, sb = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kt = 0; kt < KT; ++kt) {
    sa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f.ka[kt]), __builtin_bit_cast(bf16x8, qf[kt]), sa, 0, 0, 0);
    sb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f.kb[kt]), __builtin_bit_cast(bf16x8, qf[kt]), sb, 0, 0, 0);
  }
  const int pa0 = base + 4 * L.g;
  float v0, v1, v2, v3, v4, v5, v6, v7;
#define DF_VIS(ok, pos) ((ok) && (pos) < L.c1 && (pos) <= L.last_vis)
  v0 = DF_VIS(f.ok_a, pa0 + 0) ? sa[0] * scale : -INFINITY;
  v1 = DF_VIS(f.ok_a, pa0 + 1) ? sa[1] * scale : -INFINITY;
  v2 = DF_VIS(f.ok_a, pa0 + 2) ? sa[2] * scale : -INFINITY;
  v3 = DF_VIS(f.ok_a, pa0 + 3) ? sa[3] * scale : -INFINITY;
  v4 = DF_VIS(f.ok_b, pa0 + 16) ? sb[0] * scale : -INFINITY;
  v5 = DF_VIS(f.ok_b, pa0 + 17) ? sb[1] * scale : -INFINITY;
  v6 = DF_VIS(f.ok_b, pa0 + 18) ? sb[2] * scale : -INFINITY;
  v7 = DF_VIS(f.ok_b, pa0 + 19) ? sb[3] * scale : -INFINITY;
#undef DF_VIS
  float mx = fmaxf(fmaxf(fmaxf(v0, v1), fmaxf(v2, v3)), fmaxf(fmaxf(v4, v5), fmaxf(v6, v7)));
  mx = quarter_max(mx);
  const float m_new = fmaxf(m_run, mx);
  // all keys so far masked: exponent base 0 gives exp(-inf) = 0 for every (masked) key and corr 1
  const float mb = (m_new == -INFINITY) ? 0.f : m_new;
  const float corr = (m_run == -INFINITY) ? (m_new == -INFINITY ? 1.f : 0.f) : __expf(m_run - m_new);
  const float p0 = __expf(v0 - mb), p1 = __expf(v1 - mb), p2 = __expf(v2 - mb), p3 = __expf(v3 - mb);
  const float p4 = __expf(v4 - mb), p5 = __expf(v5 - mb), p6 = __expf(v6 - mb), p7 = __expf(v7 - mb);
  l_run = l_run * corr + (((p0 + p1) + (p2 + p3)) + ((p4 + p5) + (p6 + p7)));
  m_run = m_new;
  u32x4 ph, pl;
#define DF_PACK(i, a, b)                                                                        \
  {                                                                                             \
    const bf16_t h0 = float_to_bf16_bits(a), h1 = float_to_bf16_bits(b);                        \
    const bf16_t l0 = float_to_bf16_bits((a) - bf16_bits_to_float(h0));                         \
    const bf16_t l1 = float_to_bf16_bits((b) - bf16_bits_to_float(h1));                         \
    ph[i] = (uint32_t)h0 | ((uint32_t)h1 << 16);                                                \
    pl[i] = (uint32_t)l0 | ((uint32_t)l1 << 16);                                                \
  }
  DF_PACK(0, p0, p1) DF_PACK(1, p2, p3) DF_PACK(2, p4, p5) DF_PACK(3, p6, p7)
#undef DF_PACK
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) {
    const u32x4 vf = f.v[dt];
    f32x4 a = acc[dt];
    a[0] *= corr; a[1] *= corr; a[2] *= corr; a[3] *= corr;
    a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vf), __builtin_bit_cast(bf16x8, ph), a, 0, 0, 0);
    a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vf), __builtin_bit_cast(bf16x8, pl), a, 0, 0, 0);
    acc[dt] = a;
  }
}

template <int HD>
__global__ __launch_bounds__(256, 2) void attn_mfma_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ pool,
                                                        SeqGeom geo, AttnArgs aa, float* __restrict__ part_o,
                                                        float2* __restrict__ part_ml) {
  constexpr int KT = HD / 32, DT = HD / 16;
  // grid = (splits, kv heads, parts * sequences): the 2^q_shift workgroups that share a kv head's K/V (each with its
  // share of the query heads) differ in blockIdx.z only, by a multiple of the (even) sequence count, and so land on the
  // same XCD and read the K/V pages through one L2; "kvh" below counts head groups (kv head * parts + part)
  const int n_seq = (int)gridDim.z >> aa.q_shift;
  const int part = aa.q_shift ? (int)blockIdx.z / n_seq : 0;
  const int split = blockIdx.x, kvh = ((int)blockIdx.y << aa.q_shift) + part, s = (int)blockIdx.z - part * n_seq;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15, g = lane >> 4;
  const int B = geo.block_size;
  const int group = (aa.n_q_heads / aa.n_kv_heads) >> aa.q_shift;   // query heads of this workgroup: blockIdx.y ("kvh") counts such head groups
  const int rows = B * group;
  const int cap = geo.max_pages_per_seq * DF_PAGE;
  const int32_t* table = geo.block_table + (size_t)s * geo.max_pages_per_seq;
  // page ids of the chunk, 32 pairs at a time: lane l holds page l of the set (the pairs' own table loads would be a
  // chain).  The first set and the queries do not depend on the sequence's length: the three round trips to memory overlap
  auto load_ids = [&](int p0) { return table[min((split * aa.chunk >> 4) + 2 * p0 + lane, geo.max_pages_per_seq - 1)]; };
  int ids = load_ids(0);

  // ---- this lane's query column: row r of the kv head's row set
  const int r = wave * 16 + n;
  const bool valid = r < rows;
  const int slot = valid ? r / group : 0, hq = kvh * group + (valid ? r % group : 0);
  const size_t pr = ((size_t)(s * B + slot) * aa.n_q_heads + hq) * aa.n_splits + split;

  // query fragments (B operand of S^T): lane (n, g) holds Q[row][kt*32 + g*8 .. +8]
  u32x4 qf[KT];
  {
    const u32x4* qp = reinterpret_cast<const u32x4*>(q + ((size_t)(s * B + slot) * aa.n_q_heads + hq) * HD);
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      qf[kt] = qp[kt * 4 + g];
      if (!valid) qf[kt] = (u32x4){0u, 0u, 0u, 0u};
    }
  }
  const int n_s = geo.seq_lens[s];
  AttnLane L;
  L.n_tok = min(n_s + B, cap);
  L.c0 = split * aa.chunk;
  L.c1 = min(L.n_tok, L.c0 + aa.chunk);
  L.last_vis = valid ? (aa.causal ? n_s + slot : 0x7FFFFFFF) : -1;
  L.g = g;
  L.lane = lane;
  L.kvh = kvh >> aa.q_shift;

  float m_run = -INFINITY, l_run = 0.f;   // l_run: this lane's share (its 8 keys per pair) of the row sum
  f32x4 acc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) acc[dt] = (f32x4){0.f, 0.f, 0.f, 0.f};

  const int n_pairs = L.c1 > L.c0 ? (L.c1 - L.c0 + 31) >> 5 : 0;
  // Two fragment sets, one multiplied while the other is on its way.  Inside the loop no load is conditional (a
  // load skipped on some path would force every wait to drain all loads in flight); the last one or two pairs
  // are peeled off.
  for (int p0 = 0; p0 < n_pairs; p0 += 32) {   // one set of page ids, loaded outside the loop below for the same reason
    if (p0) ids = load_ids(p0);
    const int end = min(n_pairs, p0 + 32);
    KvFrags<HD> f0, f1;
    auto load = [&](KvFrags<HD>& f, int p) {
      const int at = 2 * (p - p0);
      attn_load_pair<HD>(f, p, __builtin_amdgcn_readlane(ids, at), __builtin_amdgcn_readlane(ids, at + 1), pool, geo, aa, L);
    };
    load(f0, p0);
    int p = p0;
    for (; p + 2 < end; p += 2) {
      load(f1, p + 1);
      attn_process_pair<HD>(f0, p, qf, acc, m_run, l_run, aa.scale, L);
      load(f0, p + 2);
      attn_process_pair<HD>(f1, p + 1, qf, acc, m_run, l_run, aa.scale, L);
    }
    if (p + 1 < end) {
      load(f1, p + 1);
      attn_process_pair<HD>(f0, p, qf, acc, m_run, l_run, aa.scale, L);
      attn_process_pair<HD>(f1, p + 1, qf, acc, m_run, l_run, aa.scale, L);
    } else {
      attn_process_pair<HD>(f0, p, qf, acc, m_run, l_run, aa.scale, L);
    }
  }

  // ---- partial result of this split: (max, sum) and the unnormalised output row -------------------------
  const float l = quarter_sum(l_run);
  if (!valid) return;
  if (aa.out) {   // the only split: nothing to merge
    const float L1 = l > 0.f ? l : INFINITY;   // no visible key: a row of zeros
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
      Act<bf16_t>::store4(reinterpret_cast<bf16_t*>(aa.out), s * B + slot, hq * HD + dt * 16 + 4 * g, aa.n_q_heads * HD,
                          make_float4(acc[dt][0] / L1, acc[dt][1] / L1, acc[dt][2] / L1, acc[dt][3] / L1));
    return;
  }
  if (g == 0) part_ml[pr] = make_float2(m_run, l);
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
    *reinterpret_cast<float4*>(part_o + pr * HD + dt * 16 + 4 * g) = make_float4(acc[dt][0], acc[dt][1], acc[dt][2], acc[dt][3]);
}

// ------------------------------------------------------------------------------------------------
// Long-chunk variant (hundreds of keys or more per workgroup).  The kernel above keeps only one page pair
// of unique bytes in flight per CU (its four wavefronts read the same keys), which is latency-bound once a
// chunk is long.  Here eight wavefronts split the KEYS instead: wavefront w takes page pairs w, w+8, ...
// of the chunk for all RB blocks of 16 query rows (K/V fragments come from HBM exactly once per workgroup), and the
// partial (max, sum, O) sets are merged through LDS at the end with the same log-sum-exp rule as the cross-split merge.
//
// A long sweep is bound by HBM, a short one by the wavefronts' own chain (scores -> softmax -> P.V), so both have to
// be covered.  The pages go straight to LDS (global_load_lds_dwordx4, a private 16 KB per wavefront): nothing in flight
// costs a register, the accumulators and one pair's scores fit 256 of them, and a SIMD holds two wavefronts, one's
// matrix instructions beside the other's softmax.  K and V halves are refilled separately, K as soon as a pair's scores are
// done, V as soon as its products are, so up to 128 KB per CU are on their way.  The loads are inline assembly and
// counted by hand (8 per half, in order): the compiler would wait for all of them before every LDS read.
// Per launch against four wavefronts with their pairs in registers: 16 ragged sequences of 1k-4k keys 55 -> 47 us, a 2048-token
// prefill pass 137 -> 117, 32 sequences of 8192 178 -> 177 (6.1 TB/s: HBM).
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t pack_bf16_pair(float a, float b) {   // RNE, a in the low half
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  const bf16x2_t r = __builtin_convertvector((f32x2_t){a, b}, bf16x2_t);
  return __builtin_bit_cast(uint32_t, r);
}

template <int HD, int RB>
__global__ __launch_bounds__(512, 2) void attn_mfma_wide_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ pool,
                                                                SeqGeom geo, AttnArgs aa, float* __restrict__ part_o,
                                                                float2* __restrict__ part_ml) {
  constexpr int KT = HD / 32, DT = HD / 16, NW = 8, LD = HD + 4;
  constexpr int PART = DF_PAGE * HD * 2;      // bytes of the K or V part of a page
  constexpr int NI = PART / 1024;             // load instructions per part
  constexpr int RING = NW * 4 * PART;         // per wavefront: K of page A, K of page B, V of page A, V of page B
  static_assert(4 * RB * 16 * LD * 4 <= RING + RB * KT * 1024, "the merge buffer overlays the ring and the queries");
  __shared__ float2 s_ml[NW][RB * 16];
  __shared__ __attribute__((aligned(1024))) char s_raw[RING + RB * KT * 1024];   // page ring and query fragments; outputs in the merge
  float (*s_o)[RB * 16][LD] = reinterpret_cast<float (*)[RB * 16][LD]>(s_raw);
  u32x4* q_lds = reinterpret_cast<u32x4*>(s_raw + RING);               // [rb][kt][lane]
  // grid = (splits, kv heads, parts * sequences): the 2^q_shift workgroups that share a kv head's K/V (each with its
  // share of the query heads) differ in blockIdx.z only, by a multiple of the (even) sequence count, and so land on the
  // same XCD and read the K/V pages through one L2; "kvh" below counts head groups (kv head * parts + part)
  const int n_seq = (int)gridDim.z >> aa.q_shift;
  const int part = aa.q_shift ? (int)blockIdx.z / n_seq : 0;
  const int split = blockIdx.x, kvh = ((int)blockIdx.y << aa.q_shift) + part, s = (int)blockIdx.z - part * n_seq;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15, g = lane >> 4;
  const int B = geo.block_size;
  const int group = (aa.n_q_heads / aa.n_kv_heads) >> aa.q_shift;   // query heads of this workgroup: blockIdx.y ("kvh") counts such head groups
  const int rows = B * group;
  const int cap = geo.max_pages_per_seq * DF_PAGE;
  const int32_t* table = geo.block_table + (size_t)s * geo.max_pages_per_seq;
  const int c0 = split * aa.chunk;
  const int kv = kvh >> aa.q_shift;

  // Page ids of this wavefront's pairs, 32 pairs at a time: lane l holds page l % 2 of its pair k0 + l / 2.  The next set is
  // requested when a set comes into use, long before it is needed.
  auto load_ids = [&](int k0) {
    const int pair = wave + NW * (k0 + (lane >> 1));
    return table[min((c0 >> 4) + 2 * pair + (lane & 1), geo.max_pages_per_seq - 1)];
  };
  // the first set and the queries do not depend on the sequence's length: the three round trips to memory overlap
  int ids = load_ids(0);
  u32x4 qr[KT];
  {
    const int r = (wave < RB ? wave : 0) * 16 + n;
    const bool valid = r < rows;
    const int slot = valid ? r / group : 0, hq = kvh * group + (valid ? r % group : 0);
    const u32x4* qp = reinterpret_cast<const u32x4*>(q + ((size_t)(s * B + slot) * aa.n_q_heads + hq) * HD);
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      qr[kt] = qp[kt * 4 + g];
      if (!valid) qr[kt] = (u32x4){0u, 0u, 0u, 0u};
    }
  }
  const int n_s = geo.seq_lens[s];
  const int n_tok = min(n_s + B, cap);
  const int c1 = min(n_tok, c0 + aa.chunk);
  const int n_all_vis = min(c1, aa.causal ? n_s : n_tok);   // keys below this are visible to every row
  const int n_pairs = c1 > c0 ? (c1 - c0 + 31) >> 5 : 0;
  const int my_pairs = n_pairs > wave ? (n_pairs - wave + NW - 1) / NW : 0;
  int ids_next = my_pairs > 32 ? load_ids(32) : 0;

  const unsigned ring = (unsigned)(size_t)&s_raw[0] + (unsigned)wave * (4 * PART);
  const unsigned voff = lane * 16;
  // one part (K or V) of a page into the ring at byte `at`
  auto fetch = [&](const bf16_t* src, unsigned at) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const unsigned dst = __builtin_amdgcn_readfirstlane(ring + at + i * 1024);
      const bf16_t* from = src + i * 512;
      unsigned keep_m0;   // whatever the compiler keeps in m0 is put back
      asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3 nt\n\ts_nop 0\n\ts_mov_b32 m0, %0"
                   : "=&s"(keep_m0) : "s"(dst), "v"(voff), "s"(from) : "memory");
    }
  };
  struct Pair {
    const bf16_t *a, *b;   // the pages' K parts (V follows)
    bool ok_a, ok_b;
  };
  auto pair_of = [&](int k) {   // this wavefront's k-th pair; foreign or missing pages alias a readable one and weigh nothing
    Pair p;
    const int pa = __builtin_amdgcn_readlane(ids, (k & 31) * 2), pb = __builtin_amdgcn_readlane(ids, (k & 31) * 2 + 1);
    const bool has_b = c0 + (wave + NW * k) * 32 + 16 < c1;
    p.ok_a = pa >= 0 && pa < geo.n_pages;
    p.ok_b = has_b && pb >= 0 && pb < geo.n_pages;
    const int a = p.ok_a ? pa : 0, b = p.ok_b ? pb : a;
    p.a = pool + kv_head_base(aa.layer, geo.n_pages, a, aa.n_kv_heads, kv, HD);
    p.b = pool + kv_head_base(aa.layer, geo.n_pages, b, aa.n_kv_heads, kv, HD);
    return p;
  };
  Pair cur{pool, pool, false, false};
  if (my_pairs > 0) {
    cur = pair_of(0);
    fetch(cur.a, 0);
    fetch(cur.b, PART);
    fetch(cur.a + DF_PAGE * HD, 2 * PART);
    fetch(cur.b + DF_PAGE * HD, 3 * PART);
  }

  // query fragments of the RB row blocks: lane (n, g) holds Q[row rb*16 + n][kt*32 + g*8 .. +8]; wavefront w
  // stages row block w in LDS for everybody
  if (wave < RB) {
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) q_lds[(wave * KT + kt) * 64 + lane] = qr[kt];
  }
  __syncthreads();

  float m_run[RB], l_run[RB];
  f32x4 acc[RB][DT];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    m_run[rb] = -INFINITY;
    l_run[rb] = 0.f;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) acc[rb][dt] = (f32x4){0.f, 0.f, 0.f, 0.f};
  }
  const float scale2 = aa.scale * 1.44269504088896341f;   // scores and running maxima in the base-2 exponent domain
  const char* my_ring = s_raw + wave * (4 * PART);

  for (int k = 0; k < my_pairs; ++k) {
    const int base = c0 + (wave + NW * k) * 32;
    const bool more = k + 1 < my_pairs;
    if (more && ((k + 1) & 31) == 0) {   // uniform over the wavefront
      ids = ids_next;
      if (k + 33 < my_pairs) ids_next = load_ids(k + 33);
    }
    Pair nxt = cur;
    if (more) nxt = pair_of(k + 1);

    // ---- scores of all row blocks: S^T = K . Q^T
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NI) : "memory");   // this pair's K is there (its V still on the way)
    f32x4 sc[RB][2];
    {
      const u32x4* kp = reinterpret_cast<const u32x4*>(my_ring) + lane;
      u32x4 ka[KT], kb[KT];
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) {
        ka[kt] = kp[kt * 64];
        kb[kt] = kp[PART / 16 + kt * 64];
      }
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        asm volatile("" ::: "memory");   // the query fragments of one row block at a time: together they would cost 64 registers
        sc[rb][0] = sc[rb][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
          const u32x4 qf = q_lds[(rb * KT + kt) * 64 + lane];
          sc[rb][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ka[kt]), __builtin_bit_cast(bf16x8, qf), sc[rb][0], 0, 0, 0);
          sc[rb][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kb[kt]), __builtin_bit_cast(bf16x8, qf), sc[rb][1], 0, 0, 0);
        }
      }
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): the K half has been read
    if (more) {
      fetch(nxt.a, 0);
      fetch(nxt.b, PART);
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- visibility (only the last pairs of a sequence and foreign pages take this branch)
    const bool tail = !cur.ok_a || !cur.ok_b || base + 32 > n_all_vis;
    if (tail) {
      const int pa0 = base + 4 * g;
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const int r = rb * 16 + n;
        const int last_vis = r < rows ? (aa.causal ? n_s + r / group : 0x7FFFFFFF) : -1;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (!(cur.ok_a && pa0 + i < c1 && pa0 + i <= last_vis)) sc[rb][0][i] = -INFINITY;
          if (!(cur.ok_b && pa0 + 16 + i < c1 && pa0 + 16 + i <= last_vis)) sc[rb][1][i] = -INFINITY;
        }
      }
    }
    // Lazy reference maximum: m_run only moves when the true row maximum has grown by more than 8 (a factor 256),
    // so the accumulators are rescaled once or twice per sweep instead of after every pair.  exp2(v - m_run) <= 256
    // meanwhile.  A row's maximum has grown that much exactly when the maximum of one of its four lanes has, so the common
    // case is decided from each lane's own scores and the cross-lane exchange happens only inside the rare branch.
    float lmx[RB];
    bool grew = false;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const f32x4 x = sc[rb][0], y = sc[rb][1];
      lmx[rb] = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), fmaxf(fmaxf(y[0], y[1]), fmaxf(y[2], y[3]))) * scale2;
      grew = grew || lmx[rb] > m_run[rb] + 8.f;
    }
    if (__builtin_amdgcn_ballot_w64(grew) != 0ull) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        float mx = lmx[rb];   // the maximum commutes with the positive scale
        mx = quarter_max(mx);
        const bool grow = mx > m_run[rb] + 8.f;
        const float corr = grow ? (m_run[rb] == -INFINITY ? 0.f : exp2f(m_run[rb] - mx)) : 1.f;
        l_run[rb] *= corr;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          acc[rb][dt][0] *= corr; acc[rb][dt][1] *= corr; acc[rb][dt][2] *= corr; acc[rb][dt][3] *= corr;
        }
        if (grow) m_run[rb] = mx;
      }
    }
    // ---- probabilities as hi + lo pairs
    u32x4 ph[RB], pl[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const float mb = (m_run[rb] == -INFINITY) ? 0.f : m_run[rb];   // nothing visible yet: exp2(-inf - 0) = 0
      float pe[8];
#pragma unroll
      for (int i = 0; i < 4; ++i) {   // -inf stays -inf -> 0
        pe[i] = __builtin_amdgcn_exp2f(fmaf(sc[rb][0][i], scale2, -mb));
        pe[4 + i] = __builtin_amdgcn_exp2f(fmaf(sc[rb][1][i], scale2, -mb));
      }
      l_run[rb] += ((pe[0] + pe[1]) + (pe[2] + pe[3])) + ((pe[4] + pe[5]) + (pe[6] + pe[7]));
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t h = pack_bf16_pair(pe[2 * i], pe[2 * i + 1]);
        ph[rb][i] = h;
        pl[rb][i] = pack_bf16_pair(pe[2 * i] - __uint_as_float(h << 16), pe[2 * i + 1] - __uint_as_float(h & 0xFFFF0000u));
      }
    }
    // ---- O^T += V^T . P^T; this pair's V is there (the next pair's K may still be on its way)
    if (more) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NI) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    // never-written rows and foreign pages: 0 * garbage must not become NaN, so those V elements are cleared
    u32x4 keep = {~0u, ~0u, ~0u, ~0u};
    if (base + 32 > n_tok || !cur.ok_a || !cur.ok_b) {
      const int pos_a = base + 4 * g, pos_b = base + 16 + 4 * g;
      auto half = [&](bool ok, int p0) { return (ok && p0 < n_tok ? 0x0000FFFFu : 0u) | (ok && p0 + 1 < n_tok ? 0xFFFF0000u : 0u); };
      keep = (u32x4){half(cur.ok_a, pos_a), half(cur.ok_a, pos_a + 2), half(cur.ok_b, pos_b), half(cur.ok_b, pos_b + 2)};
    }
    {
      const uint2* va = reinterpret_cast<const uint2*>(my_ring + 2 * PART) + lane;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const uint2 a = va[dt * 64], b = va[PART / 8 + dt * 64];
        const u32x4 vf = (u32x4){a.x, a.y, b.x, b.y} & keep;
        // all hi products, then all lo products: two MFMAs on the same accumulator are never back to back
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
          acc[rb][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vf), __builtin_bit_cast(bf16x8, ph[rb]), acc[rb][dt], 0, 0, 0);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
          acc[rb][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vf), __builtin_bit_cast(bf16x8, pl[rb]), acc[rb][dt], 0, 0, 0);
      }
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): the V half has been read
    if (more) {
      fetch(nxt.a + DF_PAGE * HD, 2 * PART);
      fetch(nxt.b + DF_PAGE * HD, 3 * PART);
    }
    cur = nxt;
  }

  // ---- merge the wavefronts' partial results (each over its own keys): the upper four hand theirs to the lower four ----
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const float l = quarter_sum(l_run[rb]);
    if (g == 0) s_ml[wave][rb * 16 + n] = make_float2(m_run[rb], l);
  }
  __syncthreads();   // also: every wavefront is done with the ring and the query fragments that s_o overlays
  float mine[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    float m_all = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) m_all = fmaxf(m_all, s_ml[w][rb * 16 + n].x);
    mine[rb] = (m_run[rb] == -INFINITY) ? 0.f : exp2f(m_run[rb] - m_all);   // m_all is finite whenever m_run is
  }
  if (wave >= 4) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
        *reinterpret_cast<float4*>(&s_o[wave - 4][rb * 16 + n][dt * 16 + 4 * g]) =
            make_float4(acc[rb][dt][0] * mine[rb], acc[rb][dt][1] * mine[rb], acc[rb][dt][2] * mine[rb], acc[rb][dt][3] * mine[rb]);
  }
  __syncthreads();
  if (wave < 4) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        float4* p = reinterpret_cast<float4*>(&s_o[wave][rb * 16 + n][dt * 16 + 4 * g]);
        const float4 u = *p;
        *p = make_float4(acc[rb][dt][0] * mine[rb] + u.x, acc[rb][dt][1] * mine[rb] + u.y, acc[rb][dt][2] * mine[rb] + u.z, acc[rb][dt][3] * mine[rb] + u.w);
      }
  }
  __shared__ float s_L[RB * 16];
  if (aa.out && (int)threadIdx.x < RB * 16) {
    float m_all = -INFINITY, l = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) m_all = fmaxf(m_all, s_ml[w][threadIdx.x].x);
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float2 ml = s_ml[w][threadIdx.x];
      l += (ml.x == -INFINITY) ? 0.f : ml.y * exp2f(ml.x - m_all);
    }
    s_L[threadIdx.x] = l > 0.f ? l : INFINITY;   // no visible key: a row of zeros
  }
  __syncthreads();
  if (aa.out) {
    // The only split: the rows leave as GEMM operand, eight dims (16 bytes of either plane) a thread, the block's rows after each
    // other, so that a block of 16 rows writes whole operand tiles.  The launch takes as long as with partial rows for a merge
    // (2048 prefill rows 121 us against 123, 32 sequences of 8192 tokens 179), and the merge is gone: 22 and 7.7 us.
    for (int idx = threadIdx.x; idx < B * group * (HD / 8); idx += 64 * NW) {
      const int slot = idx % B, c8 = (idx / B) % (HD / 8), h = idx / (B * (HD / 8));
      const int r = slot * group + h;
      float4 o[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        o[i] = *reinterpret_cast<const float4*>(&s_o[0][r][c8 * 8 + 4 * i]);
#pragma unroll
        for (int w = 1; w < 4; ++w) {
          const float4 a = *reinterpret_cast<const float4*>(&s_o[w][r][c8 * 8 + 4 * i]);
          o[i].x += a.x; o[i].y += a.y; o[i].z += a.z; o[i].w += a.w;
        }
      }
      const float L1 = s_L[r];
      const float x[8] = {o[0].x / L1, o[0].y / L1, o[0].z / L1, o[0].w / L1, o[1].x / L1, o[1].y / L1, o[1].z / L1, o[1].w / L1};
      u32x4 hi, lo;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        bf16_t h0, l0, h1, l1;
        Act<bf16_t>::split(x[2 * i], h0, l0);
        Act<bf16_t>::split(x[2 * i + 1], h1, l1);
        hi[i] = (uint32_t)h0 | ((uint32_t)h1 << 16);
        lo[i] = (uint32_t)l0 | ((uint32_t)l1 << 16);
      }
      bf16_t* to = reinterpret_cast<bf16_t*>(aa.out) + Act<bf16_t>::index(s * B + slot, (kvh * group + h) * HD + c8 * 8, aa.n_q_heads * HD);
      *reinterpret_cast<u32x4*>(to) = hi;
      *reinterpret_cast<u32x4*>(to + 512) = lo;
    }
    return;
  }
  for (int idx = threadIdx.x; idx < RB * 16 * (HD / 4); idx += 64 * NW) {
    const int r = idx / (HD / 4), d4 = idx % (HD / 4);
    if (r >= rows) continue;
    const int slot = r / group, hq = kvh * group + r % group;
    const size_t pr = ((size_t)(s * B + slot) * aa.n_q_heads + hq) * aa.n_splits + split;
    float4 o = *reinterpret_cast<const float4*>(&s_o[0][r][d4 * 4]);
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      const float4 a = *reinterpret_cast<const float4*>(&s_o[w][r][d4 * 4]);
      o.x += a.x; o.y += a.y; o.z += a.z; o.w += a.w;
    }
    *reinterpret_cast<float4*>(part_o + pr * HD + d4 * 4) = o;
    if (d4 == 0) {
      float m_all = -INFINITY;
#pragma unroll
      for (int w = 0; w < NW; ++w) m_all = fmaxf(m_all, s_ml[w][r].x);
      float l = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float2 ml = s_ml[w][r];
        l += (ml.x == -INFINITY) ? 0.f : ml.y * exp2f(ml.x - m_all);
      }
      part_ml[pr] = make_float2(m_all * 0.69314718055994531f, l);   // the cross-split merge works with natural exponents
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Prefill: two consecutive blocks of one prompt (a tile) and one group of query heads per workgroup, against all keys up to the tile's last.
// Four wavefronts own 32 of the query rows each, and eight of them two sets: the even and the odd pairs of pages, added at the end.  (A block by
// itself, the kernels above, has its keys in eight parts to merge and pays 6 us a workgroup for ramp and merge whatever its length; one set of
// wavefronts makes the longest tile of a 2048-token prompt the launch: 64 pairs of 1.4 us, each a chain of scores, softmax and products.)
// The pages are staged in an LDS ring that all share, two pairs a stage (a 16-key page's K and V halves are a wavefront's copies each), one
// barrier per stage.  Row r of a block's part is slot r % B of head r / B, so that at B = 16 a store of 64 lanes is 512 bytes of an operand
// tile and the rows leave from registers.  Workgroup id = tile * head groups + head group: an XCD keeps to the K/V of one head group where there
// are eight.  The list is taken from its end: the longest tiles of a prompt first, the prompts in reverse order.
// ------------------------------------------------------------------------------------------------
template <int HD>
__global__ __launch_bounds__(512, 2) void attn_prefill_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ pool, SeqGeom geo, AttnArgs aa,
                                                              const int4* __restrict__ tiles, int n_tiles) {
  constexpr int KT = HD / 32, DT = HD / 16, RB = 2, NS = 4, LD = HD + 4;
  constexpr int PART = DF_PAGE * HD * 2, NI = PART / 1024;   // bytes and load instructions of the K or V half of a page
  // two pairs a stage: K of page A, V of page A, K of page B, V of page B; at the end the second set's rows
  __shared__ __attribute__((aligned(1024))) char ring[NS][2][4 * PART];
  __shared__ float2 s_ml[4][RB * 16];
  static_assert(4 * RB * 16 * LD * 4 <= (int)sizeof(ring), "the second set's rows overlay the ring");
  float (*s_o)[RB * 16][LD] = reinterpret_cast<float (*)[RB * 16][LD]>(&ring[0][0][0]);
  const int lane = threadIdx.x & 63, set = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), wave = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) & 3);
  const int n = lane & 15, g = lane >> 4, B = geo.block_size;
  const int groups = aa.n_kv_heads << aa.q_shift, hg = blockIdx.x % groups, at = blockIdx.x / groups;
  const int t = n_tiles - 1 - at;
  const int4 tile = tiles[t];   // first block, one or two of them, tokens before the first
  const int group = (aa.n_q_heads / aa.n_kv_heads) >> aa.q_shift, rows = B * group, kv = hg >> aa.q_shift;
  const bool live = (wave >> 1) < tile.y;
  const int s = tile.x + min(wave >> 1, tile.y - 1);
  const int cap = geo.max_pages_per_seq * DF_PAGE;
  const int32_t* table = geo.block_table + (size_t)tile.x * geo.max_pages_per_seq;
  auto load_ids = [&](int p0) { return table[min(2 * p0 + lane, geo.max_pages_per_seq - 1)]; };   // 32 pairs' page ids
  int ids = load_ids(0);

  const int n_s = tile.z + (s - tile.x) * B, n_tok = min(n_s + B, cap), n_end = min(tile.z + tile.y * B, cap);
  u32x4 qf[RB][KT];
  int last_vis[RB];   // last key that the lane's row of the block sees
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int r = (wave & 1) * 32 + rb * 16 + n;
    const bool valid = live && r < rows;   // a row that is not reads along and is not stored
    const int slot = valid ? r % B : 0, hq = hg * group + (valid ? r / B : 0);
    last_vis[rb] = valid ? min(n_s + slot, n_tok - 1) : -1;
    const u32x4* qp = reinterpret_cast<const u32x4*>(q + ((size_t)(s * B + slot) * aa.n_q_heads + hq) * HD);
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) qf[rb][kt] = qp[kt * 4 + g];
  }
  const int n_pairs = (n_end + 31) >> 5;
  const int my_pairs = live && (wave & 1) * 32 < rows ? (n_tok + 31) >> 5 : 0;
  int ids_next = n_pairs > 32 ? load_ids(32) : 0;

  const int n_stages = (n_pairs + 1) >> 1;
  const unsigned lds = (unsigned)(size_t)&ring[0][0][0] + (unsigned)(set * 4 + wave) * PART, voff = lane * 16;
  auto page_at = [&](int pages, int p, int b) { return __builtin_amdgcn_readlane(pages, (p & 31) * 2 + b); };
  auto readable = [&](int page) { return page >= 0 && page < geo.n_pages; };
  // this wavefront's quarter of its set's pair of stage st into a slot; a foreign or missing page aliases page 0 and weighs nothing
  auto fetch = [&](int pages, int st, int slot) {
    const int page = page_at(pages, 2 * st + set, wave >> 1);
    const bf16_t* src = pool + kv_head_base(aa.layer, geo.n_pages, readable(page) ? page : 0, aa.n_kv_heads, kv, HD) + (size_t)(wave & 1) * DF_PAGE * HD;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const unsigned dst = __builtin_amdgcn_readfirstlane(lds + (unsigned)((slot & (NS - 1)) * 8 * PART + i * 1024));
      const bf16_t* from = src + i * 512;
      unsigned keep_m0;   // whatever the compiler keeps in m0 is put back
      asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3\n\ts_nop 0\n\ts_mov_b32 m0, %0"
                   : "=&s"(keep_m0) : "s"(dst), "v"(voff), "s"(from) : "memory");
    }
  };
  // (past the end the last stage again, into a slot that is not read: the number of loads in flight stays the same)
  fetch(ids, 0, 0);
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) asm volatile("" : "+v"(qf[rb][kt]));   // the queries are waited for here: inside the loop that would be a wait for every copy
  for (int st = 1; st < NS - 1; ++st) fetch(ids, min(st, n_stages - 1), st);

  float m_run[RB], l_run[RB];
  f32x4 acc[RB][DT];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    m_run[rb] = -INFINITY;
    l_run[rb] = 0.f;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) acc[rb][dt] = (f32x4){0.f, 0.f, 0.f, 0.f};
  }
  const float scale2 = aa.scale * 1.44269504088896341f;   // scores and running maxima in the base-2 exponent domain

  for (int st = 0; st < n_stages; ++st) {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NI * (NS - 2)) : "memory");   // this wavefront's quarter of the stage has landed
    __builtin_amdgcn_s_waitcnt(0xC07F);                                    // lgkmcnt(0): its reads of the stage before are done
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    const int ahead = min(st + NS - 1, n_stages - 1);
    fetch((ahead >> 4) > (st >> 4) ? ids_next : ids, ahead, st + NS - 1);   // into the slot of the stage before
    const int ids_p = ids, p = 2 * st + set;
    if (((st + 1) & 15) == 0) {   // uniform: the next stage's page ids come into use
      ids = ids_next;
      if (2 * st + 34 < n_pairs) {
        ids_next = load_ids(2 * st + 34);
        // waited for here, once in sixteen stages: left to the compiler it is a wait for every copy at the end of every stage.  (Even in time, 82 us for
        // 2048 fresh tokens, 292 for 2000 behind 4000: a stage's scores, softmax and products are longer than its copies.)
        asm volatile("" : "+v"(ids_next));
      }
    }
    if (p >= my_pairs) continue;
    const int base = p * 32;
    const bool ok_a = readable(page_at(ids_p, p, 0)), ok_b = base + 16 < n_end && readable(page_at(ids_p, p, 1));
    const char* slot = ring[st & (NS - 1)][set];
    f32x4 sc[RB][2];
    {
      const u32x4* kp = reinterpret_cast<const u32x4*>(slot) + lane;
      u32x4 ka[KT], kb[KT];
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) {
        ka[kt] = kp[kt * 64];
        kb[kt] = kp[2 * PART / 16 + kt * 64];
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) sc[rb][0] = sc[rb][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          sc[rb][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ka[kt]), __builtin_bit_cast(bf16x8, qf[rb][kt]), sc[rb][0], 0, 0, 0);
          sc[rb][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kb[kt]), __builtin_bit_cast(bf16x8, qf[rb][kt]), sc[rb][1], 0, 0, 0);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    // V is read while the softmax runs
    uint2 va[DT], vb[DT];
    {
      const uint2* vp = reinterpret_cast<const uint2*>(slot + PART) + lane;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        va[dt] = vp[dt * 64];
        vb[dt] = vp[2 * PART / 8 + dt * 64];
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (!ok_a || !ok_b || base + 32 > n_s) {   // the last pairs of a block and foreign pages
      const int p0 = base + 4 * g;
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (!(ok_a && p0 + i <= last_vis[rb])) sc[rb][0][i] = -INFINITY;
          if (!(ok_b && p0 + 16 + i <= last_vis[rb])) sc[rb][1][i] = -INFINITY;
        }
    }
    // the reference maximum moves only when the row's has grown by more than 8, decided from each lane's own scores (see above)
    float lmx[RB];
    bool grew = false;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const f32x4 x = sc[rb][0], y = sc[rb][1];
      lmx[rb] = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), fmaxf(fmaxf(y[0], y[1]), fmaxf(y[2], y[3]))) * scale2;
      grew = grew || lmx[rb] > m_run[rb] + 8.f;
    }
    if (__builtin_amdgcn_ballot_w64(grew) != 0ull) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        float mx = lmx[rb];
        mx = quarter_max(mx);
        const bool grow = mx > m_run[rb] + 8.f;
        const float corr = grow ? (m_run[rb] == -INFINITY ? 0.f : exp2f(m_run[rb] - mx)) : 1.f;
        l_run[rb] *= corr;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          acc[rb][dt][0] *= corr; acc[rb][dt][1] *= corr; acc[rb][dt][2] *= corr; acc[rb][dt][3] *= corr;
        }
        if (grow) m_run[rb] = mx;
      }
    }
    u32x4 ph[RB], pl[RB];   // probabilities as hi + lo pairs
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const float mb = (m_run[rb] == -INFINITY) ? 0.f : m_run[rb];
      float pe[8];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        pe[i] = __builtin_amdgcn_exp2f(fmaf(sc[rb][0][i], scale2, -mb));
        pe[4 + i] = __builtin_amdgcn_exp2f(fmaf(sc[rb][1][i], scale2, -mb));
      }
      l_run[rb] += ((pe[0] + pe[1]) + (pe[2] + pe[3])) + ((pe[4] + pe[5]) + (pe[6] + pe[7]));
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t h = pack_bf16_pair(pe[2 * i], pe[2 * i + 1]);
        ph[rb][i] = h;
        pl[rb][i] = pack_bf16_pair(pe[2 * i] - __uint_as_float(h << 16), pe[2 * i + 1] - __uint_as_float(h & 0xFFFF0000u));
      }
    }
    auto products = [&](auto masked_c) {
      constexpr bool MASKED = decltype(masked_c)::value;
      // rows behind the block (never written, or a later block's) and foreign pages: 0 * whatever is there must stay 0
      u32x4 keep;
      if constexpr (MASKED) {
        const int pos_a = base + 4 * g, pos_b = base + 16 + 4 * g;
        auto half = [&](bool ok, int p0) { return (ok && p0 < n_tok ? 0x0000FFFFu : 0u) | (ok && p0 + 1 < n_tok ? 0xFFFF0000u : 0u); };
        keep = (u32x4){half(ok_a, pos_a), half(ok_a, pos_a + 2), half(ok_b, pos_b), half(ok_b, pos_b + 2)};
      }
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        u32x4 vf = {va[dt].x, va[dt].y, vb[dt].x, vb[dt].y};
        if constexpr (MASKED) vf &= keep;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
          acc[rb][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vf), __builtin_bit_cast(bf16x8, ph[rb]), acc[rb][dt], 0, 0, 0);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
          acc[rb][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vf), __builtin_bit_cast(bf16x8, pl[rb]), acc[rb][dt], 0, 0, 0);
      }
    };
    if (base + 32 > n_tok || !ok_a || !ok_b) products(std::true_type{});
    else products(std::false_type{});
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // nothing may still be on its way into the ring when it is overlaid
  float l_row[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) l_row[rb] = quarter_sum(l_run[rb]);
  __syncthreads();
  if (set == 1) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      if (g == 0) s_ml[wave][rb * 16 + n] = make_float2(m_run[rb], l_row[rb]);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
        *reinterpret_cast<float4*>(&s_o[wave][rb * 16 + n][dt * 16 + 4 * g]) = make_float4(acc[rb][dt][0], acc[rb][dt][1], acc[rb][dt][2], acc[rb][dt][3]);
    }
  }
  __syncthreads();
  if (set == 1) return;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int r = (wave & 1) * 32 + rb * 16 + n;
    if (!live || r >= rows) continue;
    const float2 other = s_ml[wave][rb * 16 + n];
    const float m_all = fmaxf(m_run[rb], other.x);
    const float f0 = m_run[rb] == -INFINITY ? 0.f : exp2f(m_run[rb] - m_all), f1 = other.x == -INFINITY ? 0.f : exp2f(other.x - m_all);
    const float l = l_row[rb] * f0 + other.y * f1;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const float4 o = *reinterpret_cast<const float4*>(&s_o[wave][rb * 16 + n][dt * 16 + 4 * g]);
      acc[rb][dt] = (f32x4){acc[rb][dt][0] * f0 + o.x * f1, acc[rb][dt][1] * f0 + o.y * f1, acc[rb][dt][2] * f0 + o.z * f1, acc[rb][dt][3] * f0 + o.w * f1};
    }
    const float L1 = l > 0.f ? l : INFINITY;   // no visible key: a row of zeros
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
      Act<bf16_t>::store4(reinterpret_cast<bf16_t*>(aa.out), s * B + r % B, (hg * group + r / B) * HD + dt * 16 + 4 * g, aa.n_q_heads * HD,
                          make_float4(acc[rb][dt][0] / L1, acc[rb][dt][1] / L1, acc[rb][dt][2] / L1, acc[rb][dt][3] / L1));
  }
}

// whether the kernels above take this configuration
template <typename T>
inline bool attn_takes_mfma(const AttnArgs& aa, int block_size) {
  const int group = aa.n_q_heads / aa.n_kv_heads;
  return sizeof(T) == 2 && ((block_size * group) >> aa.q_shift) <= 64 && group % (1 << aa.q_shift) == 0 && (aa.head_dim == 128 || aa.head_dim == 64);
}

// pairs of a prompt's consecutive blocks: (first pseudo-sequence, one or two of them, tokens before them, -)
struct PrefillTiles {
  const int4* at = nullptr;
  int n = 0;   // 0: not a prefill, or too little work for one workgroup a tile and group of heads
};

inline void attn_mfma_launch(hipStream_t st, const bf16_t* q, const bf16_t* pool, SeqGeom geo, AttnArgs aa, int S, float* part_o, float2* part_ml,
                             int wide_min_chunk, PrefillTiles tiles) {
  const dim3 grid(aa.n_splits, aa.n_kv_heads, S << aa.q_shift), block(256);
  if (tiles.n) {
    hipLaunchKernelGGL(attn_prefill_kernel<128>, dim3(tiles.n * (aa.n_kv_heads << aa.q_shift)), dim3(512), 0, st, q, pool, geo, aa, tiles.at, tiles.n);
    return;
  }
  // long chunks: wavefronts split the keys
  if (aa.head_dim == 128 && aa.chunk >= wide_min_chunk)
    hipLaunchKernelGGL((attn_mfma_wide_kernel<128, 4>), grid, dim3(512), 0, st, q, pool, geo, aa, part_o, part_ml);
  else if (aa.head_dim == 128)
    hipLaunchKernelGGL(attn_mfma_kernel<128>, grid, block, 0, st, q, pool, geo, aa, part_o, part_ml);
  else
    hipLaunchKernelGGL(attn_mfma_kernel<64>, grid, block, 0, st, q, pool, geo, aa, part_o, part_ml);
}
