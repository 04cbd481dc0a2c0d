// Compute-bound GEMM for many activation rows (M > 64): y[M,N] = a[M,K] * W[N,K]^T, bf16 MFMA 16x16x32 with
// hi+lo activation pairs, fp32 accumulation, the same operand layouts and epilogues as the streaming kernel.
//
// A workgroup of 2*WY wavefronts (WY = 2 or 4 along N x 2 along M) owns a tile of WY*WN weight row bands x 2*WM
// activation row bands for one K range (grid.y).  Both operands already sit in HBM in MFMA fragment order (1 KB per
// 16x32 fragment), so a k tile is staged in LDS by copying whole fragments; every wavefront reads the WN weight and 2*WM
// activation fragments of its part of the tile (each lane its own 16 bytes: conflict-free ds_read_b128) and issues
// WN*WM*2 MFMAs per k tile.  The eight-wavefront form (WY = 4) is two four-wavefront workgroups fused along N: one
// activation stage for twice the weight rows, i.e. a third less operand traffic from L2 per flop, at one workgroup per CU (two
// of the 256 x 64 tile with a ring of three slots, which the routed items use: 72 KB and 100 registers).
//
// What bounds it: over random operands the best tiling of a large launch ends at 1.3-1.5 PFLOP/s of issued MFMA work (a torch matrix product of
// the same issued size reaches 1.1-1.47), where the clock gives way to the power limit; smaller launches, a round of the CUs or less, wait at the
// seams of their k tiles and for their first and last ones (O projection of the 8B shape at 256 rows 0.69, QKV 0.86).
//
// A ring of NS LDS slots is filled by direct-to-LDS loads (global_load_lds_dwordx4: every lane's 16 bytes go straight to
// consecutive LDS addresses, which is exactly a fragment in operand order), and the fragments are double-buffered in registers:
// while the MFMAs of k tile t run out of one register set, the LDS reads of k tile t+1 fill the other, so no MFMA waits for LDS
// behind the barrier.  One barrier per k tile.  The reads and the refill's copies are issued one behind each MFMA: in bursts ahead
// of the MFMAs (all wavefronts of a SIMD come out of the barrier together) their 14 to 19 instructions kept the matrix cores idle.
// Launch after launch over random operands, bursts and one by one: gate/up of the 8B shape at 512 rows 150 -> 143 us (1.44
// PFLOP/s issued), 256 rows 90 -> 86, 2048 rows on the same 384 x 128 tiles 574 -> 547; 256 x 128 tiles at 512 rows 187 -> 177; a
// step of 512 rows 3 %, of 256 rows 2.5 %.
// Rolling form (512 x 128 tiles): 128 accumulators leave no room for a second set of all activation fragments, so they roll, one
// band ahead, and the seam between two k tiles lies in front of the last band instead of the first.  The fewest bytes a flop from
// L2 and from LDS of all tiles, and the fastest over many rows: gate/up at 2048 rows 541 us (1.52 PFLOP/s issued) against 547 on 384 x 128
// tiles and 563 on 256 x 128 tiles staged through registers, two workgroups a CU (the form before); down projection 276 against 290.
//
// STREAM: the weights are read past the caches' usual order of eviction (nt), so that the activations stay: for the
// eight-wavefront tiles of few activation blocks, whose workgroups read a weight block at the same time (stream_weights in plan.h).  Prefill of
// 1024 (eight blocks) 3008 -> 2985 us; but of 1088 (nine) 3572 -> 3607, of 2048 5605 -> 5630, and with the four-wavefront tiles' weights
// as well, verification of 128 routed rows 624 -> 632.
// Grouped launches choose by the item: the weights of an expert's only item are read once, by anybody.  Two-layer verification of 512 routed
// rows 939 -> 894.  Where an expert has several items they all read its weights, and the memory-side cache serves the later ones: two-layer prefills
// of one prompt with the hint on every item and on the only ones, 1638 tokens of 64 experts of 1024 x 1024 860 and 818 us, four of 421 behind up to 1000 and 128
// experts of 4096 x 1024 3691 and 3495, one of 1579 and 32 of 2048 x 512 478 and 452.
//
// Workgroup order: consecutive workgroup ids go to different XCDs (round-robin dispatch, id = 8*j + x), and the
// workgroups that re-read one weight block run back to back on one XCD and share its L2.  Where the weight blocks divide
// evenly over the XCDs, XCD x takes blocks x, x + 8, ...: the chip sweeps neighbouring blocks together.  Otherwise XCD x
// takes the x-th eighth of the tiles, counted activation block by activation block within a weight block, so that no XCD has
// more than one tile more than another (20 blocks are 3 on four XCDs and 2 on four: a fifth of the launch; the even case is
// 1 % faster the first way).
#pragma once
#include <utility>

#include "gemm.h"

// wavefronts per SIMD to leave registers for: two workgroups share a CU where their staging fits twice
template <int WN, int WM, int NS, int WY>
constexpr int tiled_waves() { return NS * (WY * WN + 4 * WM) <= 80 ? WY : 1; }

template <int WN, int WM>
constexpr bool tiled_rolls() { return WN * WM >= 32; }   // see above

template <typename F, int... I>
__device__ __forceinline__ void unroll_each(F& f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, typename F>
__device__ __forceinline__ void unroll(F f) { unroll_each(f, std::make_integer_sequence<int, N>{}); }

template <int WN, int WM, int EPI, int NS, bool GRP = false, int WY = 2, bool STREAM = false>
__global__ __launch_bounds__(128 * WY, (tiled_waves<WN, WM, NS, WY>())) void gemm_bf16_tiled_kernel(
    const bf16_t* __restrict__ W, const bf16_t* __restrict__ A, int M, int N, int K, int n_blocks, int m_blocks, EpiArgs ep) {
  constexpr int NWV = 2 * WY;                       // wavefronts: WY along N x 2 along M
  constexpr int BNT = WY * WN, BMT = 2 * WM;        // fragments of a stage: BNT weight + 2*BMT activation (hi, lo)
  constexpr int FR = BNT + 2 * BMT, PER = FR / NWV, PW = BNT / NWV;   // fragments copied by each wavefront, PW of them weights
  static_assert(WN % 2 == 0 && WM % 2 == 0 && FR % NWV == 0 && BNT % NWV == 0 && NS >= 2 && NS * FR <= 160 && (WY == 2 || WY == 4),
                "tile shape");
  __shared__ u32x4 stage[NS][FR][64];

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wy = wave >> 1, wx = wave & 1;
  const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
  const int tile = xcd * (int)(gridDim.x >> 3) + j;
  int nb = tile / m_blocks, mb = tile % m_blocks;
  if ((n_blocks & 7) == 0) { nb = (j / m_blocks) * 8 + xcd; mb = j % m_blocks; }
  const int KT = K >> 5, n_tiles = N >> 4;
  int m_tiles = (M + 15) >> 4, mt0 = mb * BMT;
  bool read_once = false;
  if constexpr (GRP) {
    // grouped launch (routed experts, see EpiArgs): m_blocks counts work items of up to BMT bands; the workgroups of
    // one item (its n_blocks weight blocks) run back to back on one XCD and share the item's activation rows there
    mb = (j / n_blocks) * 8 + xcd;
    nb = j % n_blocks;
    if (mb >= m_blocks) return;
    const int4 item = ep.grp_items[mb];
    if (item.x < 0) return;
    W += (size_t)item.x * ep.grp_w_stride;
    mt0 = item.y;
    m_tiles = item.z;
    read_once = item.w != 0 && ep.grp_stream;
  }
  if (nb >= n_blocks) return;                      // whole workgroup leaves before any barrier
  const int ks = gridDim.y, kz = blockIdx.y;
  const int per = (KT + ks - 1) / ks;
  const int kb = min(KT, kz * per), ke = min(KT, kb + per);
  const int nt0 = nb * BNT;

  // the PER fragments this wavefront copies per stage: address at k tile kb (the same for all lanes) and bytes per k tile
  const char* src[PER];
  unsigned step[PER];
  auto fragment = [&](int i) { return i < PW ? wave * PW + i : BNT + wave * (PER - PW) + i - PW; };
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int f = fragment(i);
    if (i < PW) {    // weight fragment: bands past the matrix alias the last band (never stored)
      src[i] = reinterpret_cast<const char*>(W) + ((size_t)kb * n_tiles + min(nt0 + f, n_tiles - 1)) * 1024;
      step[i] = (unsigned)n_tiles * 1024u;
    } else {         // activation fragment: band (f - BNT) / 2, plane (f - BNT) % 2
      const int a = f - BNT;
      src[i] = reinterpret_cast<const char*>(A) + ((size_t)min(mt0 + (a >> 1), m_tiles - 1) * KT + kb) * 2048 + (a & 1) * 1024;
      step[i] = 2048u;
    }
  }
  int at_kt = kb;             // k tile the addresses stand at; past the end of the K range they stay on the last one
  auto advance = [&]() {
    const bool go = ++at_kt < ke;
#pragma unroll
    for (int i = 0; i < PER; ++i) src[i] += go ? step[i] : 0u;
  };

  f32x4 acc[WN][WM];
#pragma unroll
  for (int i = 0; i < WN; ++i)
#pragma unroll
    for (int jj = 0; jj < WM; ++jj) acc[i][jj] = (f32x4){0.f, 0.f, 0.f, 0.f};

  if (kb < ke) {
    // The direct-to-LDS loads are inline assembly so that the compiler does not count them: it would otherwise wait for ALL of
    // them before every LDS read.  Completion is tracked by hand: each wavefront issues PER loads per k tile, in order, so
    // "at most PER*(NS-2) outstanding" says that its share of k tile t+1 has landed.  The barrier extends that to the whole
    // workgroup; every wavefront has waited for its reads of k tile t before it, so slot t may be refilled behind it.
    const unsigned lds_base = (unsigned)(size_t)&stage[0][0][0], voff = lane * 16;
    // m0 carries the LDS address; whatever the compiler keeps in it is put back, so the statement clobbers nothing
#define DF_COPY(hint)                                                                                                                    \
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3" hint "\n\ts_nop 0\n\ts_mov_b32 m0, %0" \
               : "=&s"(keep_m0) : "s"(dst), "v"(at_lane), "s"(from) : "memory")
    auto sweep = [&](auto hint_c) __attribute__((always_inline)) {
      constexpr bool HINT = decltype(hint_c)::value;
      auto dma = [&](int i, int slot) {
        const unsigned dst = __builtin_amdgcn_readfirstlane(lds_base + (unsigned)((slot * FR + fragment(i)) * 1024));
        const unsigned at_lane = voff;
        const char* from = src[i];
        unsigned keep_m0;
        if (HINT && i < PW) DF_COPY(" nt");
        else DF_COPY("");
      };
      for (int d = 0; d < NS; ++d) {
#pragma unroll
        for (int i = 0; i < PER; ++i) dma(i, d);
        advance();
      }
      auto w_at = [&](int sl, int i) { return stage[sl][wy * WN + i][lane]; };
      auto a_at = [&](int sl, int jj, int p) { return stage[sl][BNT + 2 * (wx * WM + jj) + p][lane]; };
      // the next k tile's copies of this wavefront have landed, its reads of the one before are done
      auto seam = [&]() {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PER * (NS - 2)) : "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
      };
      constexpr bool ROLL = tiled_rolls<WN, WM>();
      u32x4 wf[2][WN], ap[2][ROLL ? 1 : WM][2];
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PER * (NS - 1)) : "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
#pragma unroll
      for (int i = 0; i < WN; ++i) wf[0][i] = w_at(0, i);
#pragma unroll
      for (int jj = 0; jj < (ROLL ? 1 : WM); ++jj)
#pragma unroll
        for (int p = 0; p < 2; ++p) ap[0][jj][p] = a_at(0, jj, p);
      int slot = 0;
      // K tile t.  MFMA number q (band, then plane, then weight tile) is followed by at most a few of the loads that are due meanwhile,
      // pinned there: in a burst ahead of the MFMAs they kept the matrix cores idle for a sixth of the k tile.
      auto k_tile = [&](auto cur_c) {
        constexpr int C = decltype(cur_c)::value;
        const int next = slot == NS - 1 ? 0 : slot + 1;
        constexpr int RD = WN + (ROLL ? 2 : 2 * WM), ITEMS = RD + PER;   // the next k tile's fragments, then the refill of this one's slot
        auto item = [&](auto qc) {
          constexpr int q = decltype(qc)::value;
          // past the end of the K range: a landed copy of the last k tile, not used
          if constexpr (q < 1) ap[ROLL ? 0 : C ^ 1][0][0] = a_at(next, 0, 0);
          else if constexpr (q < 1 + WN) wf[C ^ 1][q - 1] = w_at(next, q - 1);
          else if constexpr (q < RD) ap[ROLL ? 0 : C ^ 1][ROLL ? 0 : (q - WN) / 2][(q - WN) & 1] = a_at(next, (q - WN) / 2, (q - WN) & 1);
          else if constexpr (q < ITEMS) dma(q - RD, slot);
        };
        if constexpr (!ROLL) seam();
        unroll<2 * WN * WM>([&](auto mc) {
          constexpr int m = decltype(mc)::value, jj = m / (2 * WN), p = (m / WN) & 1, i = m % WN, at = m % (2 * WN);
          if constexpr (ROLL && jj == WM - 1 && at == 0) seam();   // this k tile is in registers from here on
          const u32x4 a = ROLL ? ap[jj & 1][0][p] : ap[C][ROLL ? 0 : jj][p];
          acc[i][jj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wf[C][i]), __builtin_bit_cast(bf16x8, a), acc[i][jj], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (!ROLL) {
            item(mc);
            static_assert(ITEMS <= 2 * WN * WM, "an item behind each MFMA");
          } else if constexpr (jj < WM - 1) {
            if constexpr (at < 2) ap[(jj + 1) & 1][0][at] = a_at(slot, jj + 1, at);   // the next band
          } else {
            constexpr int EACH = (ITEMS + 2 * WN - 1) / (2 * WN);
            unroll<EACH>([&](auto ec) { item(std::integral_constant<int, at * EACH + decltype(ec)::value>{}); });
          }
          __builtin_amdgcn_sched_barrier(0);
        });
        advance();
        slot = next;
      };
      int kt = kb;
      for (; kt + 1 < ke; kt += 2) {
        k_tile(std::integral_constant<int, 0>{});
        k_tile(std::integral_constant<int, 1>{});
      }
      if (kt < ke) k_tile(std::integral_constant<int, 0>{});
    };
#undef DF_COPY
    if constexpr (GRP) {
      if (read_once) sweep(std::true_type{});
      else sweep(std::false_type{});
    } else {
      sweep(std::integral_constant<bool, STREAM>{});
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // nothing may still be on its way into LDS when the slots are reused or released
  }

  // lane l holds y[m = band*16 + l%16][n = tile*16 + 4*(l/16) .. +3]
  const int mrow = lane & 15, gq = lane >> 4;
#pragma unroll
  for (int jj = 0; jj < WM; ++jj) {
    const int mt = mt0 + wx * WM + jj, m = mt * 16 + mrow;
    if (mt >= m_tiles || m >= M) continue;
    if (EPI == EPI_SWIGLU) {
      bf16_t* act = reinterpret_cast<bf16_t*>(ep.act);
#pragma unroll
      for (int p = 0; p < WN / 2; ++p) {
        const int nt = nt0 + wy * WN + 2 * p;      // gate tile; the up tile follows it
        if (nt + 1 >= n_tiles) continue;
        const f32x4 gs = acc[2 * p][jj], us = acc[2 * p + 1][jj];
        Act<bf16_t>::store4(act, m, (nt >> 1) * 16 + 4 * gq, ep.act_K,
                            make_float4(silu_f(gs[0]) * us[0], silu_f(gs[1]) * us[1], silu_f(gs[2]) * us[2], silu_f(gs[3]) * us[3]));
      }
    } else {
#pragma unroll
      for (int i = 0; i < WN; ++i) {
        const int nt = nt0 + wy * WN + i;
        if (nt >= n_tiles || !ep.out) continue;
        const f32x4 s = acc[i][jj];
        const size_t at = (size_t)m * ep.ld + nt * 16 + 4 * gq;
        *reinterpret_cast<float4*>(ep.out + (size_t)kz * ep.slab + at) = make_float4(s[0], s[1], s[2], s[3]);
        if (ep.out2) *reinterpret_cast<float4*>(ep.out2 + at) = make_float4(s[0], s[1], s[2], s[3]);
      }
    }
  }
  if (EPI == EPI_STORE && ep.amax) {   // fused argmax over this workgroup's columns (host guarantees a single K range)
    __syncthreads();                   // the staging slots are free now: reuse them for the two N halves' bests
    float2* wbest = reinterpret_cast<float2*>(&stage[0][0][0]);   // [wy][BMT * 16 rows]: the bests of the WY column groups
    const uint64_t key = ep.amax_mode ? ep.amax_key[0] : 0ull;
#pragma unroll
    for (int jj = 0; jj < WM; ++jj) {
      const int mt = mt0 + wx * WM + jj, m = mt * 16 + mrow;
      float bv = -INFINITY;
      int bi = 0x7FFFFFFF;
#pragma unroll
      for (int i = 0; i < WN; ++i) {
        const int nt = nt0 + wy * WN + i;
        if (nt >= n_tiles) continue;
        const int col = nt * 16 + 4 * gq;
#pragma unroll
        for (int e = 0; e < 4; ++e) argmax_combine(bv, bi, amax_score(ep, key, acc[i][jj][e], m, col + e), col + e);
      }
      argmax_swap16(bv, bi);
      argmax_swap32(bv, bi);
      if (gq == 0) wbest[wy * (BMT * 16) + (wx * WM + jj) * 16 + mrow] = make_float2(bv, __int_as_float(bi));
    }
    __syncthreads();
    for (int r = threadIdx.x; r < BMT * 16; r += 64 * NWV) {
      const int m = mt0 * 16 + r;
      if (m >= M) continue;
      float bv = wbest[r].x;
      int bi = __float_as_int(wbest[r].y);
#pragma unroll
      for (int y = 1; y < WY; ++y) argmax_combine(bv, bi, wbest[y * BMT * 16 + r].x, __float_as_int(wbest[y * BMT * 16 + r].y));
      ep.amax[(size_t)m * n_blocks + nb] = make_float2(bv, __int_as_float(bi));
    }
  }
  if (EPI == EPI_STORE && ep.lse) {   // fused softmax statistics over this workgroup's columns (single K range)
    __syncthreads();                  // the staging slots (and the argmax scratch in them) are free now
    float2* wl = reinterpret_cast<float2*>(&stage[0][0][0]);   // [wy][BMT * 16 rows]
#pragma unroll
    for (int jj = 0; jj < WM; ++jj) {
      float lm = -INFINITY, ls = 0.f;
#pragma unroll
      for (int i = 0; i < WN; ++i) {
        if (nt0 + wy * WN + i >= n_tiles) continue;
        lse_add4(lm, ls, make_float4(acc[i][jj][0], acc[i][jj][1], acc[i][jj][2], acc[i][jj][3]), ep.lse_inv_T);
      }
      lse_combine_row(lm, ls);
      if (gq == 0) wl[wy * (BMT * 16) + (wx * WM + jj) * 16 + mrow] = make_float2(lm, ls);
    }
    __syncthreads();
    for (int r = threadIdx.x; r < BMT * 16; r += 64 * NWV) {
      const int m = mt0 * 16 + r;
      if (m >= M) continue;
      float lm = wl[r].x, ls = wl[r].y;
#pragma unroll
      for (int y = 1; y < WY; ++y) lse_combine(lm, ls, wl[y * BMT * 16 + r].x, wl[y * BMT * 16 + r].y);
      ep.lse[(size_t)m * n_blocks + nb] = make_float2(lm, ls);
    }
  }
}
