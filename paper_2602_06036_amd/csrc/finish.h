// What the workgroup that arrives last at a column block of a K-split GEMM does with the block's complete sums, so that no
// launch of its own has to add the slabs (streaming kernel, one band of rows):
// h += sum of the slabs, and the operand of the RMSNorm that follows with its division deferred (gemm_resid.h).
// A dependent launch costs 4.4 to 5.2 us however little it does; this costs 2.6: down projection of the 8B shape at 16 rows, eight K ranges, 18.6 us + 5.3
// for the normalisation launch behind it before, 21.2 finished, 20.7 with the four ranges of 64 blocks that the plan takes now.  The slabs are written through the L2 (sc1:
// an XCD's L2 is not the others'), waited for, a counter says who is last, and that workgroup reads the slabs back past its
// L2.  Nobody waits for anybody, and the sums are added in ascending order whoever is last.  No fence: a device-scope one
// writes back and invalidates the whole L2.  (The q/k norm and rotation finished the same way behind the QKV GEMM, sixteen
// workgroups a unit of three heads: 18.0 us against 10.6 + 4.6, a chain of five memory round trips.)
#pragma once
#include "common.h"

// Arrival counters are 128 bytes apart (neighbouring ones are hit at the same time); zero before and after every launch: the call's
// embed_kernel clears them, each launch leaves them as it found them.
constexpr int kArriveStride = 32;

// Pieces of the rows' sums of squares: floats from one row to the next, whole groups of four that are read together (what a row does not
// use of its last group is never looked at)
__host__ __device__ constexpr int ssq_row(int parts) { return (parts + 3) & ~3; }

struct FinishArgs {
  unsigned* arrive;         // [column blocks * kArriveStride]
  float* h;                 // [M, N] residual stream, updated in place
  const float* gain_next;   // gain of the RMSNorm that reads the new h
  bf16_t* a_out;            // GEMM operand h * gain_next, row length N
  float* ssq;               // [M, ssq_row(column blocks)] pieces of the rows' sums of squares
  bf16_t* taps;             // nullable: the new h as tapped hidden state `tap_idx` (operand, row length tap_K)
  int tap_idx, tap_K;
};

// write-through stores and loads past the L2, 16 bytes; byte offsets from a uniform base
__device__ __forceinline__ __amdgpu_buffer_rsrc_t coherent_base(const float* p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, 0xFFFFFFFFu, 0x00027000);
}
constexpr int kSc1 = 16;
__device__ __forceinline__ void store_coherent(__amdgpu_buffer_rsrc_t b, unsigned off, float4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), b, off, 0, kSc1);
}
__device__ __forceinline__ float4 load_coherent(__amdgpu_buffer_rsrc_t b, unsigned off) {
  return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(b, off, 0, kSc1));
}

// True in the last of `n` workgroups to come here; everything they stored with store_coherent before is then readable.
__device__ __forceinline__ bool last_to_arrive(unsigned* counter, unsigned n) {
  __shared__ unsigned s_before;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wavefront's stores have reached memory
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned before = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (before == n - 1) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next launch
    s_before = before;
  }
  __syncthreads();
  return s_before == n - 1;
}

__device__ __forceinline__ float4 add4(float4 a, float4 b) { return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); }

// adds ks slabs (`stride` bytes apart) to v[i] in ascending order, Z at a time
template <int C>
__device__ __forceinline__ void add_slabs(float4 (&v)[C], __amdgpu_buffer_rsrc_t b, const unsigned (&off)[C], int ks, unsigned stride) {
  constexpr int Z = 8;
  int z = 0;
  for (; z + Z <= ks; z += Z) {
    float4 p[Z][C];
#pragma unroll
    for (int u = 0; u < Z; ++u)
#pragma unroll
      for (int i = 0; i < C; ++i) p[u][i] = load_coherent(b, off[i] + (unsigned)(z + u) * stride);
#pragma unroll
    for (int u = 0; u < Z; ++u)
#pragma unroll
      for (int i = 0; i < C; ++i) v[i] = add4(v[i], p[u][i]);
  }
  for (; z < ks; ++z) {
    float4 p[C];
#pragma unroll
    for (int i = 0; i < C; ++i) p[i] = load_coherent(b, off[i] + (unsigned)z * stride);
#pragma unroll
    for (int i = 0; i < C; ++i) v[i] = add4(v[i], p[i]);
  }
}

// Column block `blk` of NT * 16 columns, all M <= 16 rows; 256 threads.  s_q: LDS, at least 64 * NT floats.
template <int NT>
__device__ __forceinline__ void finish_resid(const FinishArgs& f, const float* slabs, int ld, size_t slab, int ks, int M, int blk, int n_blk,
                                             float* s_q) {
  constexpr int C4 = NT * 4, ITEMS = 16 * C4, C = (ITEMS + 255) / 256;
  const __amdgpu_buffer_rsrc_t b = coherent_base(slabs);
  const int N = ld;
  float4 v[C], gn[C];
  unsigned off[C];
  int row[C], c4[C];
#pragma unroll
  for (int i = 0; i < C; ++i) {
    const int idx = min(i * 256 + (int)threadIdx.x, ITEMS - 1);   // past the end: the last item again, not stored
    row[i] = idx / C4;
    c4[i] = idx % C4;
    const size_t at = (size_t)min(row[i], M - 1) * N + blk * (NT * 16) + c4[i] * 4;
    off[i] = (unsigned)at * 4u;
    v[i] = *reinterpret_cast<const float4*>(f.h + at);
    gn[i] = *reinterpret_cast<const float4*>(f.gain_next + blk * (NT * 16) + c4[i] * 4);
  }
  add_slabs<C>(v, b, off, ks, (unsigned)slab * 4u);
#pragma unroll
  for (int i = 0; i < C; ++i) {
    if (i * 256 + (int)threadIdx.x >= ITEMS) continue;
    s_q[row[i] * C4 + c4[i]] = (v[i].x * v[i].x + v[i].y * v[i].y) + (v[i].z * v[i].z + v[i].w * v[i].w);
    if (row[i] >= M) continue;
    const int col = blk * (NT * 16) + c4[i] * 4;
    *reinterpret_cast<float4*>(f.h + (size_t)row[i] * N + col) = v[i];
    Act<bf16_t>::store4(f.a_out, row[i], col, N, make_float4(v[i].x * gn[i].x, v[i].y * gn[i].y, v[i].z * gn[i].z, v[i].w * gn[i].w));
    if (f.taps) Act<bf16_t>::store4(f.taps, row[i], f.tap_idx * N + col, f.tap_K, v[i]);
  }
  __syncthreads();
  if ((int)threadIdx.x < M) {
    float q = 0.f;
#pragma unroll
    for (int c = 0; c < C4; ++c) q += s_q[threadIdx.x * C4 + c];
    f.ssq[(size_t)threadIdx.x * ssq_row(n_blk) + blk] = q;
  }
}
