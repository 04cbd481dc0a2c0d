// Shared device/host helpers of the DFlash HIP path: storage types, tile and KV-page layouts.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef uint16_t bf16_t;  // raw bfloat16 bits
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Wavefront index inside a workgroup: kernels compute it as readfirstlane(threadIdx.x >> 6) so that the compiler
// knows it is the same for all 64 lanes; loop bounds, slot numbers and base addresses derived from it then stay
// in scalar registers and the branches on them are plain scalar branches.
#define DF_WAVE 64
#define DF_PAGE 16

__host__ __device__ __forceinline__ float bf16_bits_to_float(bf16_t b) {
  union { uint32_t u; float f; } c;
  c.u = (uint32_t)b << 16;
  return c.f;
}
// round-to-nearest-even; inputs are finite on this path
__host__ __device__ __forceinline__ bf16_t float_to_bf16_bits(float f) {
  union { uint32_t u; float f; } c;
  c.f = f;
  uint32_t u = c.u;
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}

template <typename T> struct Store;
template <> struct Store<float> {
  static __host__ __device__ __forceinline__ float from(float f) { return f; }
  static __host__ __device__ __forceinline__ float to(float v) { return v; }
};
template <> struct Store<bf16_t> {
  static __host__ __device__ __forceinline__ bf16_t from(float f) { return float_to_bf16_bits(f); }
  static __host__ __device__ __forceinline__ float to(bf16_t v) { return bf16_bits_to_float(v); }
};

// ---- GEMM weight layout -------------------------------------------------------------------------
// A matrix of N rows x K (K contiguous in the canonical form).  fp32: plain row-major.  bf16: cut into
// 16-row x 32-column tiles; a tile is 1 KB holding, for lane = (k%32)/8*16 + r%16 of a 64-wide
// wavefront, the 8 consecutive k values that lane feeds to v_mfma_f32_16x16x32_bf16.  Tiles are stored
// k-tile-major: all N/16 tiles of k-tile 0, then all tiles of k-tile 1, ...  A wavefront that owns NT
// adjacent row bands reads NT KB contiguously per k step and neighbouring workgroups read the neighbouring
// KBs, so the whole grid sweeps each k slab of the matrix sequentially (DRAM-friendly), instead of
// thousands of independent 1 KB streams.
template <typename T> __host__ __device__ __forceinline__ size_t tile_index(int r, int k, int K, int N);
template <> __host__ __device__ __forceinline__ size_t tile_index<float>(int r, int k, int K, int) {
  return (size_t)r * K + k;
}
template <> __host__ __device__ __forceinline__ size_t tile_index<bf16_t>(int r, int k, int, int N) {
  return ((size_t)(k >> 5) * (N >> 4) + (r >> 4)) * 512 + (size_t)(((((k & 31) >> 3) << 4) + (r & 15)) * 8 + (k & 7));
}
// rows that a buffer in this layout must provide for M logical rows
template <typename T> __host__ __device__ __forceinline__ int tile_rows(int M) { return M; }
template <> __host__ __device__ __forceinline__ int tile_rows<bf16_t>(int M) { return (M + 15) & ~15; }

// ---- GEMM activation operand ---------------------------------------------------------------------
// fp32 models: plain row-major fp32.  bf16 models: every activation that feeds a GEMM is kept as a
// PAIR of bf16 numbers hi + lo (hi = bf16(x), lo = bf16(x - hi)), i.e. ~16 significand bits, and the
// GEMM issues two MFMAs per weight tile.  Single-bf16 inputs make two correct evaluations of the
// same model drift apart by percents of the logit spread (one flipped rounding perturbs every later
// rounding); the pair removes that at no cost while the GEMM is bandwidth-bound.  Layout: the tile
// layout above with the hi tile (1 KB) immediately followed by the lo tile.
template <typename T> struct Act;
template <> struct Act<float> {
  static constexpr int planes = 1;
  static __host__ __device__ __forceinline__ size_t elems(int M, int K) { return (size_t)M * K; }
  static __device__ __forceinline__ void store(float* base, int m, int k, int K, float v) { base[(size_t)m * K + k] = v; }
  // 4 consecutive k (k % 4 == 0)
  static __device__ __forceinline__ void store4(float* base, int m, int k, int K, float4 v) {
    *reinterpret_cast<float4*>(base + (size_t)m * K + k) = v;
  }
};
template <> struct Act<bf16_t> {
  static constexpr int planes = 2;
  static __host__ __device__ __forceinline__ size_t elems(int M, int K) { return (size_t)((M + 15) & ~15) * K * 2; }
  static __host__ __device__ __forceinline__ size_t index(int m, int k, int K) {  // hi element; lo is 512 further
    return ((size_t)(m >> 4) * (K >> 5) + (k >> 5)) * 1024 + (size_t)(((((k & 31) >> 3) << 4) + (m & 15)) * 8 + (k & 7));
  }
  static __device__ __forceinline__ void split(float v, bf16_t& hi, bf16_t& lo) {
    hi = float_to_bf16_bits(v);
    lo = float_to_bf16_bits(v - bf16_bits_to_float(hi));
  }
  static __device__ __forceinline__ void store(bf16_t* base, int m, int k, int K, float v) {
    bf16_t hi, lo;
    split(v, hi, lo);
    const size_t i = index(m, k, K);
    base[i] = hi;
    base[i + 512] = lo;
  }
  static __device__ __forceinline__ void store4(bf16_t* base, int m, int k, int K, float4 v) {
    ushort4 hi, lo;
    split(v.x, hi.x, lo.x);
    split(v.y, hi.y, lo.y);
    split(v.z, hi.z, lo.z);
    split(v.w, hi.w, lo.w);
    const size_t i = index(m, k, K);
    *reinterpret_cast<ushort4*>(base + i) = hi;
    *reinterpret_cast<ushort4*>(base + i + 512) = lo;
  }
};

// ---- KV page layout ----------------------------------------------------------------------------
// A pool holds, per layer, n_pages pages; a page holds for each kv head 16 keys then 16 values:
//   pool[layer][page][kv_head][K|V][16*hd]
// K part: [hd/8][16 keys][8 dims]   -> a 16-key x 32-dim MFMA A-operand tile is 1 KB contiguous
// V part: [hd/16][4][16 dims][4 keys] -> lane (dim%16, key/4) of the P.V MFMA reads 4 keys contiguously
__host__ __device__ __forceinline__ int k_in_page(int key, int d) { return (d >> 3) * 128 + key * 8 + (d & 7); }
__host__ __device__ __forceinline__ int v_in_page(int key, int d) {
  return (d >> 4) * 256 + (key >> 2) * 64 + (d & 15) * 4 + (key & 3);
}
__host__ __device__ __forceinline__ size_t kv_head_base(int layer, int n_pages, int page, int n_kv_heads, int kvh, int hd) {
  return ((((size_t)layer * n_pages + page) * n_kv_heads + kvh) * 2) * (size_t)(DF_PAGE * hd);
}

struct SeqGeom {          // passed by value to kernels that walk the page table
  const int32_t* seq_lens;
  const int32_t* block_table;
  int32_t max_pages_per_seq;
  int32_t n_pages;
  int32_t block_size;
  int32_t* status;        // sticky device status word
};

#define DF_STATUS_CAPACITY 1

// Sums and maxima over a wavefront in the order of a butterfly (lanes 32 apart first, neighbours last), by lane swaps and rotations inside the
// register file: as shuffles every one of the six steps is a round trip to LDS.  The fp32 step of 4 sequences of 16 tokens behind 300: 184 us,
// now 143 (its products end in such sums, eight to a wavefront: wave_sum8); 16-bit steps 0.3 to 0.8 %, by their norms and softmaxes.
template <int CTRL>
__device__ __forceinline__ float lane_dpp(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
template <int D>
__device__ __forceinline__ float lane_xor(float x) {   // the value of lane ^ D, D < 16
  static_assert(D == 1 || D == 2 || D == 4 || D == 8, "inside sixteen lanes");
  if constexpr (D == 1) return lane_dpp<0xB1>(x);                // quad_perm [1,0,3,2]
  else if constexpr (D == 2) return lane_dpp<0x4E>(x);           // quad_perm [2,3,0,1]
  else if constexpr (D == 4) return lane_dpp<0x1B>(lane_dpp<0x141>(x));   // row_half_mirror, then quad_perm [3,2,1,0]
  else return lane_dpp<0x128>(x);                                // row_ror:8
}
template <typename Op>
__device__ __forceinline__ void lane_xor16(float& a, float& b, Op op) {   // op(the pair of lane ^ 1), then ^ 2, ^ 4, ^ 8
  op(lane_xor<1>(a), lane_xor<1>(b));
  op(lane_xor<2>(a), lane_xor<2>(b));
  op(lane_xor<4>(a), lane_xor<4>(b));
  op(lane_xor<8>(a), lane_xor<8>(b));
}
// Sums in lane order of up to 64 values in a loop of shuffles waited for LDS in every turn; the merges of split
// attention end in one: a step of 4 sequences of 16384 tokens 992 -> 984 us, of one of 1000 4228 -> 4208.
__device__ __forceinline__ float lane_value(float x, int lane) {   // lane: the same in all lanes
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), lane));
}
struct LanePair {
  float lo, hi;
};
// lanes 32 (16) apart: a's lower (even) part and b's behind each other, a's upper (odd) part and b's
__device__ __forceinline__ LanePair lane_swap32(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
  const unsigned lo = r[0], hi = r[1];   // scalars first: a bit cast of a vector's element reads element 0
  return {__builtin_bit_cast(float, lo), __builtin_bit_cast(float, hi)};
}
__device__ __forceinline__ LanePair lane_swap16(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
  const unsigned lo = r[0], hi = r[1];   // scalars first: a bit cast of a vector's element reads element 0
  return {__builtin_bit_cast(float, lo), __builtin_bit_cast(float, hi)};
}
template <typename Op>
__device__ __forceinline__ float wave_reduce(float v, Op op) {
  LanePair p = lane_swap32(v, v);
  v = op(p.lo, p.hi);
  p = lane_swap16(v, v);
  v = op(p.lo, p.hi);
  v = op(v, lane_xor<8>(v));
  v = op(v, lane_xor<4>(v));
  v = op(v, lane_xor<2>(v));
  return op(v, lane_xor<1>(v));
}
// the same over the four lanes that are 16 apart (16 first)
template <typename Op>
__device__ __forceinline__ float quarter_reduce(float v, Op op) {
  LanePair p = lane_swap16(v, v);
  v = op(p.lo, p.hi);
  p = lane_swap32(v, v);
  return op(p.lo, p.hi);
}
__device__ __forceinline__ float quarter_sum(float v) { return quarter_reduce(v, [](float a, float b) { return a + b; }); }
__device__ __forceinline__ float quarter_max(float v) { return quarter_reduce(v, [](float a, float b) { return fmaxf(a, b); }); }
__device__ __forceinline__ float wave_reduce_sum(float v) { return wave_reduce(v, [](float a, float b) { return a + b; }); }
__device__ __forceinline__ float wave_reduce_max(float v) { return wave_reduce(v, [](float a, float b) { return fmaxf(a, b); }); }
// Eight sums at once, in the same order each: lane l ends up with the sum of v[wave_sum8_index(l)] in ten steps instead of 48.
__device__ __forceinline__ int wave_sum8_index(int lane) { return (lane >> 5 & 1) * 4 + (lane >> 4 & 1) * 2 + (lane >> 3 & 1); }
__device__ __forceinline__ float wave_sum8(const float (&v)[8]) {
  float a[4], b[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const LanePair p = lane_swap32(v[i], v[i + 4]);
    a[i] = p.lo + p.hi;
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const LanePair p = lane_swap16(a[i], a[i + 2]);
    b[i] = p.lo + p.hi;
  }
  const bool odd = (threadIdx.x & 8) != 0;
  const float b0 = lane_xor<8>(b[0]), b1 = lane_xor<8>(b[1]);   // outside the choice: every lane takes part
  float c = odd ? b[1] + b1 : b[0] + b0;
  c += lane_xor<4>(c);
  c += lane_xor<2>(c);
  return c + lane_xor<1>(c);
}

// ---- counter-based random numbers and the argmax combine rule (shared by the LM-head epilogues and misc.h) ----
// Draws are a hash of (key, sequence, block slot, purpose, index): the same number whichever kernel asks for it.
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
// u in (0,1), 23 bits (so that x + 0.5 is exact in fp32): counter c = (((seq*64 + slot)*4 + purpose) << 32) | idx
__device__ __forceinline__ float counter_uniform(uint64_t key, int seq, int slot, int purpose, uint32_t idx) {
  const uint64_t c = ((uint64_t)(((uint32_t)seq * 64u + (uint32_t)slot) * 4u + (uint32_t)purpose) << 32) | idx;
  const uint64_t z = mix64(key + 0x9E3779B97F4A7C15ull * (c + 1ull));
  return ((float)(z >> 41) + 0.5f) * 1.1920928955078125e-7f;  // 2^-23
}
__device__ __forceinline__ float gumbel(float u) { return -logf(-logf(u)); }

__device__ __forceinline__ void argmax_combine(float& bv, int& bi, float v, int i) {
  if (v > bv || (v == bv && i < bi)) { bv = v; bi = i; }
}
__device__ __forceinline__ void argmax_combine(float& bv, int& bi, LanePair v, LanePair i) {
  bv = v.lo;
  bi = __float_as_int(i.lo);
  argmax_combine(bv, bi, v.hi, __float_as_int(i.hi));
}
__device__ __forceinline__ void argmax_swap32(float& bv, int& bi) { argmax_combine(bv, bi, lane_swap32(bv, bv), lane_swap32(__int_as_float(bi), __int_as_float(bi))); }
__device__ __forceinline__ void argmax_swap16(float& bv, int& bi) { argmax_combine(bv, bi, lane_swap16(bv, bv), lane_swap16(__int_as_float(bi), __int_as_float(bi))); }
__device__ __forceinline__ void wave_argmax(float& bv, int& bi) {   // over the wavefront, the same in every lane
  auto other = [&](float v, float i) { argmax_combine(bv, bi, v, __float_as_int(i)); };
  argmax_swap32(bv, bi);
  argmax_swap16(bv, bi);
  other(lane_xor<8>(bv), lane_xor<8>(__int_as_float(bi)));
  other(lane_xor<4>(bv), lane_xor<4>(__int_as_float(bi)));
  other(lane_xor<2>(bv), lane_xor<2>(__int_as_float(bi)));
  other(lane_xor<1>(bv), lane_xor<1>(__int_as_float(bi)));
}
