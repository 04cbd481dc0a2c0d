// Which launch a shape gets: the knobs and the rules that choose tiles, K splits, context splits and chunks.  Plain host C++
// without a HIP header, so that the rules can be run where there is no GPU.
#pragma once
#include <stddef.h>
#include <stdlib.h>

#include <algorithm>

inline int env_int(const char* name, int dflt) {
  const char* e = getenv(name);
  const int v = e ? atoi(e) : 0;
  return v > 0 ? v : dflt;
}

constexpr int kTileWgs = 256;   // see attention_by_tiles

// Tuning and testing knobs, read from the environment whenever a context is created (or a workspace is sized): a
// context keeps the values it was created with, so a test that sets one before dflash_create gets exactly that path
// whatever ran earlier in the process.  Defaults are what the measurements in the documentation use.
struct Knobs {
  int gemm_wide;            // DFLASH_GEMM_WIDE: 1 = eight-wavefront tiles by estimated time (default), 2 = always (tests), any other value = never
  int attn_target_wgs;      // DFLASH_ATTN_TARGET_WGS: workgroups an attention launch aims at
  int attn_wide_min_chunk;  // DFLASH_ATTN_WIDE_MIN_CHUNK: keys per workgroup from which the key-split attention kernel is used
  int attn_tile_wgs;        // DFLASH_ATTN_TILE_WGS: workgroups from which a prefill's attention goes by tiles, whatever its contexts (default 256: by rule)
  int gemm_target_wgs;      // DFLASH_GEMM_TARGET_WGS: workgroups a K-split streaming GEMM aims at
  int gemm_u;               // DFLASH_GEMM_U: k tiles per prefetch stage (one band of rows)
  int gemm_nt8;             // DFLASH_GEMM_NT8: matrices with at least 8 * this row bands use 8 weight tiles per activation fragment
  int gemm_fill;            // DFLASH_GEMM_FILL: 1 = weight tiles per wavefront (8, 6 or 4) and K split chosen to fill whole rounds of the CUs
  int gemm_fill4;           // DFLASH_GEMM_FILL4: the same for 17-64 rows
  int gemm_u4;              // DFLASH_GEMM_U4: k tiles per prefetch stage for 17-64 rows
  int gemm_tile, gemm_wm, gemm_ks;   // DFLASH_GEMM_TILE / _WM / _KS: force the tiled GEMM's shape / rows per tile / K split (0 = by estimated time)
  int lm_stats;             // DFLASH_LM_STATS: 1 = softmax statistics from the LM-head epilogue, other = from the stored logits
  int moe_mt;               // DFLASH_MOE_MT: 1, 2, 4 or 8 forces the bands per routed-expert work item (0 = by rows per expert)
  int moe_gather_min_rows;  // DFLASH_MOE_GATHER_MIN_ROWS: rows from which the routed-expert GEMMs get their rows copied into list order
  int moe_kept_kb;          // DFLASH_MOE_KEPT_KB: a target's expert matrices up to this size are taken to stay in the memory-side cache
  int moe_down_u;           // DFLASH_MOE_DOWN_U: k tiles per stage of the one-band down projection
  int fuse;                 // DFLASH_FUSE: few-row path, see dflash_ctx::fuse
  int resid_nw, resid_u;    // DFLASH_RESID_NW / _U: wavefronts per workgroup and k tiles per stage of the unsplit projection kernel
};
inline Knobs read_knobs() {
  Knobs k;
  k.gemm_wide = env_int("DFLASH_GEMM_WIDE", 1);
  k.attn_target_wgs = env_int("DFLASH_ATTN_TARGET_WGS", 256);
  k.attn_wide_min_chunk = env_int("DFLASH_ATTN_WIDE_MIN_CHUNK", 512);
  k.attn_tile_wgs = env_int("DFLASH_ATTN_TILE_WGS", kTileWgs);
  k.gemm_target_wgs = env_int("DFLASH_GEMM_TARGET_WGS", 256);
  k.gemm_u = env_int("DFLASH_GEMM_U", 2);
  k.gemm_nt8 = env_int("DFLASH_GEMM_NT8", 1);
  k.gemm_fill = env_int("DFLASH_GEMM_FILL", 1);
  k.gemm_fill4 = env_int("DFLASH_GEMM_FILL4", 1);
  k.gemm_u4 = env_int("DFLASH_GEMM_U4", 1);
  k.gemm_tile = env_int("DFLASH_GEMM_TILE", 0);
  k.gemm_wm = env_int("DFLASH_GEMM_WM", 0);
  k.gemm_ks = env_int("DFLASH_GEMM_KS", 0);
  k.lm_stats = env_int("DFLASH_LM_STATS", 1);
  k.moe_mt = env_int("DFLASH_MOE_MT", 0);
  k.moe_gather_min_rows = env_int("DFLASH_MOE_GATHER_MIN_ROWS", 64);
  k.moe_kept_kb = env_int("DFLASH_MOE_KEPT_KB", 128 << 10);
  k.moe_down_u = env_int("DFLASH_MOE_DOWN_U", 1);
  k.fuse = env_int("DFLASH_FUSE", 1);
  if (k.fuse != 1 && k.fuse != 2) k.fuse = 0;
  k.resid_nw = env_int("DFLASH_RESID_NW", 4);
  k.resid_u = env_int("DFLASH_RESID_U", 8);
  return k;
}

// ---- attention: context splits ------------------------------------------------------------------------
struct SplitPlan {
  int n_splits, chunk;
  int bound;  // >= n_splits for this and every smaller max_tokens (sizes the partial buffers)
};
inline SplitPlan plan_splits(int S, int n_kv_heads, int max_tokens, int target_wgs) {
  // The attention kernels run one workgroup per CU, or two where their page loads then wait on each other: at most one
  // round of workgroups on the 256 CUs (target_wgs: Knobs::attn_target_wgs).  Rounded down: a second round of a few
  // workgroups costs as much as the first.  Two-layer verify steps of the 8B target, rounded up and down: 24 sequences x
  // 4000 keys 1040 and 951 us, 7 x 8000 532 and 490, 20 x 100..400 738 and 724; slower in one of 19 sizes (13 x 300..5000,
  // lengths that differ so much that more workgroups even the load out: 469 and 476).  It does not fill the chip where S x heads does
  // not divide 256: 11 and 12 sequences of eight heads run 176 and 192 workgroups, 17 to 31 run 136 to 248.
  const int max_splits = 64;
  int splits = target_wgs / (S * n_kv_heads);
  const int by_len = (max_tokens + 63) / 64;
  splits = std::max(1, std::min(splits, std::min(by_len, max_splits)));
  int chunk = (max_tokens + splits - 1) / splits;
  chunk = (chunk + 63) & ~63;
  SplitPlan p;
  p.bound = splits;
  p.chunk = chunk;
  p.n_splits = (max_tokens + chunk - 1) / chunk;
  return p;
}

// Prefill: tiles of two consecutive blocks of a prompt that has `chunks` of them in a pass (constexpr: for host and device)
constexpr int prefill_tiles(int chunks) { return chunks > 0 ? (chunks + 1) / 2 : 0; }
// ... and whether the pass's attention goes by tiles, a workgroup for each and every group of heads.  `blocks`: those of the pass; `cached`: the most tokens
// that lie in front of a prompt's first block in it; `from`: Knobs::attn_tile_wgs, set by hand the only condition.  Attention of a layer block by block and by
// tiles, eight head groups of 64 query rows unless said.
// - Tiles have to fill the CUs, their keys are not split: one prompt of 320 tokens (80 workgroups) 16.5 and 20 us, of 1024 (256) 42.7 and 39.6, of 2048 106 and 82.
// - Contexts below 256 tokens are all ramp, which a block by itself with four wavefronts has less of: 12 prompts of 21 to 170 28 and 31.
// - Equally long tiles go in whole rounds of the CUs, and a block alone in its tile takes a tile's time, while blocks, twice as many and bound by their
//   pages, fill in: 6 prompts of 340 behind 4000 (528 workgroups) 299 and 400, 12 of 170 behind 2652 (576, every sixth tile half empty) 202 and 313.  Where the
//   cached part is short the tiles' lengths differ and even the load out: six of 37 to 311 behind 0 to 600 (296 workgroups, half a round empty) 53 and 37.
// - Behind longer contexts a block's ramp and merge do not count: 1024 behind 4000 142 and 148, 2000 behind 16000 875 and 900.
// - A routed-expert target's attention stays with the blocks, also where the knob asks for tiles: another order of sums ahead of its routers (see stream_plan).
// Over 1600 passes (eight head layouts, blocks of 2 to 16, 1 to 32 prompts, up to 4600 tokens) the rule takes 7 % off the attention time of the passes' mean, and 24 are
// more than 3 % slower by tiles; with 256 workgroups and 4608 tokens as the only conditions 4.5 % and 438.
inline bool attention_by_tiles(int tiles, int blocks, int head_groups, int cached, int max_tokens, int from, bool routed = false) {
  const int wgs = tiles * head_groups, rounds = (wgs + 255) / 256;
  if (routed) return false;
  if (from != kTileWgs) return wgs >= from;
  if (wgs < kTileWgs || max_tokens < 256 || max_tokens > 3072) return false;
  return cached <= 768 || blocks * head_groups * 10 >= rounds * 512 * 9;   // nine tenths of the rounds' places for blocks taken
}

// ---- GEMMs ----------------------------------------------------------------------------------------------
// rows of partial results the split-K arena holds for a context of at most max_rows activation rows
inline int arena_rows(int max_rows) { return std::max(1024, 4 * max_rows); }

constexpr int kMaxKSplit = 16;

// Deferred RMSNorm of one band of rows: pieces of a row's sum of squares that the GEMM behind it requests ahead of its sweep.  The unsplit
// projection leaves one for 16 columns, so this covers rows of 8192; the rest of a longer row is read behind the sweep, in groups of four as well.
// (With 256 here, and anything else one piece at a time behind the sweep, three-layer verifications of 16 rows took 363 us at width 5120, 359
// so; 867 and 859 at 8192, 307 and 300 at 4128 (258 pieces), 611 and 601 at 9216; at 4096, whose 256 pieces either takes, 265 and 264.)
constexpr int kSsqAhead = 512;

// The LDS-staged tiles and what a k tile costs on a CU, in microseconds: `two` with two workgroups of the shape side by
// side (four-wavefront tiles), `one` with a workgroup by itself; `fixed` per round of workgroups (ramp, prologue, epilogue).
// Fitted to launches back to back over random operands (16 row counts from 80 to 2048, ten matrices of 2048 to 28672 rows
// with K of 2048 to 12288, one to eight K ranges); the shape picked with them is on average 1.0 % slower than the fastest one (2.1 %
// before the loads went between the MFMAs and the 512 x 128 tiles came).  A fit that comes within 0.5 % of the fastest launches does not make the faster
// passes: step of 16 sequences 1489 us with these costs and 1510 with it, verification of 11 sequences 899 and 919, of 8 728 and 722, of 20 1231 and
// 1228, prefills even.
struct TileShape {
  int wn, wm, wy;      // weight tiles and activation bands per wavefront, wavefronts along N
  float two, one, fixed;
};
constexpr TileShape kTiles[] = {
    {4, 4, 2, 0.71f, 0.45f, 3.5f},   {6, 4, 2, 1.02f, 0.72f, 1.5f},   {8, 2, 2, 0.727f, 0.438f, 3.1f}, {6, 2, 2, 0.579f, 0.397f, 3.4f},
    {4, 2, 2, 0.444f, 0.269f, 2.9f}, {8, 4, 4, 0.f, 1.249f, 0.6f},    {6, 4, 4, 0.f, 0.964f, 1.5f},    {4, 4, 4, 0.f, 0.697f, 2.0f},
    {6, 2, 4, 0.f, 0.567f, 2.5f},    {4, 2, 4, 0.f, 0.425f, 3.3f}};

struct TilePlan {
  const TileShape* t = nullptr;
  int ks = 1;
};
// Time of a launch = k tiles of a K range x cost of the workgroups on the busiest CU + the partial slabs (written by the
// GEMM, read by its consumer).  XCDs take equal shares of the tiles, so the busiest CU has ceil(share / 32 CUs) workgroups.
// `ranges`: 0 = the number of K ranges is free.
template <size_t SHAPES>
inline TilePlan cheapest_tiles(const TileShape (&shapes)[SHAPES], const Knobs& kn, int M, int N, int K, bool split, int arena, int ranges) {
  const int nt = N / 16, KT = K / 32;
  const bool forced = kn.gemm_tile || kn.gemm_wm || kn.gemm_ks;   // a forced four-wavefront shape stays forced
  auto fits = [&](int k) { return k == 1 || (split && KT / k >= 8 && k * M <= arena); };
  if (kn.gemm_ks && split && fits(kn.gemm_ks)) ranges = kn.gemm_ks;   // any number of ranges that fits
  TilePlan best;
  double best_t = 1e30;
  for (const TileShape& t : shapes) {
    const int nb = (nt + t.wy * t.wn - 1) / (t.wy * t.wn), mb = ((M + 15) / 16 + 2 * t.wm - 1) / (2 * t.wm);
    if (t.wy == 4 && kn.gemm_wide != 2 && (kn.gemm_wide != 1 || forced)) continue;
    if (kn.gemm_tile && kn.gemm_tile != t.wn) continue;
    if (kn.gemm_wm && kn.gemm_wm != t.wm) continue;
    const int tried[] = {1, 2, 3, 4, 6, 8};
    for (int i = 0; i < (ranges ? 1 : 6); ++i) {
      const int k = ranges ? ranges : tried[i];
      if (!fits(k)) continue;
      // a workgroup of eight wavefronts has its CU to itself: not for launches that leave many CUs without one.  Over the sweep that the
      // costs are fitted to any line up to 160 picks the same (0.74 % above the fastest shape on average), 192 loses 0.1 %, 224 0.7 %
      if (t.wy == 4 && kn.gemm_wide == 1 && nb * mb * k < 160) continue;
      const int on_cu = ((nb * mb + 7) / 8 * k + 31) / 32, per = (KT + k - 1) / k;
      const int pairs = t.wy == 2 ? on_cu / 2 : 0, single = on_cu - 2 * pairs;
      double us = (pairs * t.two + single * t.one) * per + (pairs + single) * t.fixed;
      // slabs, at the rate of a large copy; the factor over the sweep: 0 picks 7.3 % above the fastest shape on average, 1 3.1, 2 0.86,
      // 2.25 0.74, 3 0.69, 4 1.2
      if (split) us += 2.25 * k * M * (double)N * 4 / 4.7e6;
      if (t.wy == 4 && kn.gemm_wide == 2) us *= 1e-3;           // before any four-wavefront shape
      if (us < best_t) { best_t = us; best.t = &t; best.ks = k; }
    }
  }
  if (!best.t) {   // a knob that names no shape
    best.t = &shapes[0];
    if (ranges) best.ks = ranges;
  }
  return best;
}

// K ranges of a routed-expert target's layers: by costs of their own, which stay when the tiles' are fitted anew.  Another number of ranges is another order of
// sums, which turns near-ties of the routers behind them into other experts, for targets of any width; whichever tiles then run add the products of a range in
// the same order.  (The costs are those of the tiles of an earlier fit; by the present ones 31 of 348 shapes of a 2048-wide target get other ranges.)
constexpr TileShape kRangeCosts[] = {
    {8, 4, 2, 1.32f, 1.00f, 1.0f},   {6, 4, 2, 1.02f, 0.72f, 1.5f},  {4, 4, 2, 0.747f, 0.464f, 3.5f}, {8, 2, 2, 0.727f, 0.463f, 3.1f},
    {6, 2, 2, 0.579f, 0.397f, 3.4f}, {4, 2, 2, 0.44f, 0.269f, 2.9f}, {6, 4, 4, 0.f, 1.00f, 1.5f},     {4, 4, 4, 0.f, 0.715f, 2.0f},
    {6, 2, 4, 0.f, 0.562f, 2.5f},    {4, 2, 4, 0.f, 0.425f, 3.3f}};
inline TilePlan tile_plan(const Knobs& kn, int M, int N, int K, bool split, int arena, bool routed = false) {
  const bool forced = kn.gemm_tile || kn.gemm_wm || kn.gemm_ks;
  const int ranges = routed && split && !forced ? cheapest_tiles(kRangeCosts, kn, M, N, K, split, arena, 0).ks : 0;
  return cheapest_tiles(kTiles, kn, M, N, K, split, arena, ranges);
}

// Whether the eight-wavefront tiles read the weights with the non-temporal hint (STREAM in gemm_tiled.h): few activation blocks, and weight blocks that
// divide by the XCDs.  Where they do not, a block's workgroups may sit on two XCDs, which then both fetch it past the memory-side cache.  Six-layer verifications
// with and without it there: 140 rows of a 5120-wide model of FFN 14080 1610 and 1500 us, 135 of 3584 and 9856 1114 and 1032, 224 of 3072 and 8448 1060 and
// 1028.  Where they do: four-layer step of 256 rows at the 8B shape 1517 and 1530, verification of 176 901 and 924, 512 rows even.  In a routed target's layers the
// hint pays either way: what follows reads hundreds of megabytes of experts past the caches (two layers of 512 rows 889 and 905 us, deeper ones even).
inline bool stream_weights(int n_blocks, int m_blocks, bool routed) { return m_blocks <= 8 && (n_blocks % 8 == 0 || routed); }

// K split across workgroups: aim at enough workgroups that every CU keeps several wavefronts streaming,
// keep at least 2 k-tiles per wavefront, and stay inside the arena.
inline int pick_ksplit(int n_blocks, int KT, int M, int arena, int target) {
  int ks = 1;
  while (ks < kMaxKSplit && n_blocks * ks * 2 <= target && KT / (ks * 2 * 4) >= 2 && ks * 2 * M <= arena) ks *= 2;
  return ks;
}

// The weight-streaming kernel's launch for up to 64 rows: weight tiles and activation bands per workgroup, k tiles per
// prefetch stage, K ranges.
struct StreamPlan {
  int nt = 0, mt = 0, u = 0, ks = 1;   // nt = 0: another kernel's shape
  bool staged = false;   // its blocks and K ranges as 128 x 64 tiles of the LDS-staged kernel
};
// whether the launch may finish its own sums (finish.h): plans that the finishing kernel is built for
inline bool stream_finishes(const StreamPlan& p) { return p.nt >= 4 && p.mt == 1; }
inline StreamPlan stream_plan(const Knobs& kn, int M, int N, int K, bool split, int arena, bool four_first = true) {
  const int nt = N / 16, KT = K / 32;
  StreamPlan p;
  // a launch of 192 workgroups leaves a quarter of the CUs idle: among 8, 6 or 4 weight tiles per wavefront and any K split
  // (not only powers of two) take the fullest last round.  Ties go to more tiles (a band of activations is read for more of the
  // matrix), for one band of rows of a dense model to four tiles first: half the K ranges, so half the slabs for whoever adds them.  (4096 rows of
  // matrix as 32 blocks x 8 ranges and as 64 x 4: verification of blocks of ten of the 14336-wide model 409 and 401.5 us.)  The layers of a
  // routed-expert target (`four_first` false) gain as much, O projection 16 x 16 and 32 x 8, QKV 40 x 6 and 80 x 3: 709 and 691, but the
  // router's near-ties turn another order of sums into another expert: one row of sixteen that goes the other way is 1 % of the logits.  (Four tiles pay
  // where nothing else fills the chip: an unsplit 16384-column LM head, 128 workgroups with 8, took 31 us at 16 rows and 49 at
  // 64, now 23 and 39.)
  auto fullest = [&]() {
    double best = -1.0;
    const int four[] = {4, 8, 6}, more[] = {8, 6, 4};
    for (int i = 0; i < 3; ++i) {
      const int cand = M <= 16 && four_first ? four[i] : more[i];
      if (nt % cand) continue;
      const int nb = nt / cand;
      for (int k = 1; k <= (split ? kMaxKSplit : 1); ++k) {
        if (k > 1 && (KT / (k * 4) < 2 || k * M > arena)) break;
        const int wgs = nb * k, rounds = (wgs + 255) / 256;
        const double fill = (double)wgs / (rounds * 256.0) - 0.02 * (rounds - 1);   // a single round beats several
        if (fill > best + 1e-9) { best = fill; p.nt = cand; p.ks = k; }
      }
    }
  };
  auto powers = [&](int t) {
    p.nt = t;
    p.ks = split ? pick_ksplit(nt / t, KT, M, arena, kn.gemm_target_wgs) : 1;
  };
  if (M <= 16) {
    const int NT8 = kn.gemm_nt8, U = kn.gemm_u;   // U: k-tiles per prefetch stage
    p.mt = 1;
    if (kn.gemm_fill == 1 && NT8 && nt >= 8 * NT8 && (nt % 8 == 0 || nt % 6 == 0)) {
      fullest();
      p.u = 2;
    } else if (NT8 && nt % 8 == 0 && nt >= 8 * NT8) {
      powers(8);
      p.u = U >= 2 ? 2 : 1;
    } else if (nt % 4 == 0) {
      powers(4);
      p.u = U >= 4 ? 4 : (U >= 2 ? 2 : 1);
    } else {
      powers(nt % 2 == 0 ? 2 : 1);
      p.u = 4;
    }
  } else if (M <= 64 && nt % 8 == 0) {
    // still bandwidth-bound: the same streaming kernel with two or four activation bands per weight tile
    p.mt = M <= 32 ? 2 : 4;
    p.u = 1;
    if (kn.gemm_fill4 == 1) fullest();
    else powers(8);
    if (p.nt == 8 && kn.gemm_u4 >= 2) p.u = 2;   // (measured slower)
    // Four bands: a wavefront that has all of them reads every activation fragment for itself, and what it reads from the L2 waits behind
    // its weights from HBM; staged in LDS a fragment is read once for four wavefronts.  Split matrices of 128-row blocks, as streaming launches and
    // as LDS-staged ones with the same K ranges, 64 rows: 4096 x 12288 24.5 and 22.7 us, 4096 x 4096 11.7 and 10.5, 4096 x 20480 35.6 and 33.7; four-layer
    // steps and verifications 1008 and 992, 546 and 541, 582 and 574.  But three bands (4096 x 12288 22.0 and 20.8 by itself) 517.9 and 518.7 in a
    // verification, two 18.4 and 19.7, half the CUs (2048 x 2048, 64 rows) 5.8 and 6.6, unsplit 96-row blocks (24576 x 4096) 41.9 and 44.5.
    // (Not in a routed target's layers: another order of sums, as above.)
    // The staged launch deals whole blocks to the XCDs, the streaming one workgroups: where the blocks do not divide by eight, an XCD may get more
    // workgroups than its 32 CUs a round.  20 blocks x 12 ranges (36 on most XCDs, none on one) with K = 3072 8.5 and 11.7 us at 64 rows, with 20480 26.0 and
    // 40.3, 28 x 9 17.3 and 21.6; but 28 x 8 (32 each) 8.3 and 7.8, 40 x 6 20.8 and 18.4, 56 x 9 32.8 and 27.0.
    const int wgs = nt / 8 * p.ks, of_xcd = (nt / 8 + 7) / 8 * p.ks;
    p.staged = four_first && split && M > 48 && p.nt == 8 && p.u == 1 && wgs >= 192 && of_xcd <= (wgs + 255) / 256 * 32;
  }
  return p;
}

// fp32 GEMM: whether four wavefronts share an output column's K (each at least a 256-wide piece) instead of taking a column each.
// `cols`: columns of all groups of eight rows (a workgroup does one group; with the columns of a single group here steps of 64 rows and more
// were 1 to 3 % slower).  It pays while the columns alone leave CUs idle, and the fewer pieces a column has the sooner they fill
// the chip; a SwiGLU column is two.  Columns x K at 8 rows, one and four wavefronts a column: 512 x 1024 4.6 and 4.0 us; 1024 x 1024 4.8
// and 5.1; 2048 x 1024 5.4 and 7.2; 1024 x 2048 6.7 and 5.9; 2048 x 2048 7.8 and 8.6; 1536 x 4096 11.3 and 11.5; 2048 x 4096 13.2
// and 15.0.  SwiGLU 512 x 1024 5.8 and 5.3; 768 x 1024 6.1 and 6.3; 1536 x 2048 9.9 and 10.5.  768 x 1024 is even by itself, in a step
// four are faster.
inline bool split_f32_columns(int cols, int K, bool swiglu) { return K >= 1024 && cols <= std::min(swiglu ? K / 2 : K / 4 * 3, 1536); }

// fp32 GEMM: whether the groups of eight rows that share a block of weights run one after the other on one XCD (its L2 serves them), instead of all column
// blocks of one group after those of the other: for matrices that the memory-side cache of 256 MB does not hold from group to group.  `blocks`:
// workgroups of a group (the limit: grid.y).  Verifications, the largest matrix in MB, group by group and side by side: width 1024, 213 MB, 16 rows 194
// and 199 us, 256 rows 2216 and 2337; 268 MB 249 and 251, 3025 and 2854; 328 MB 330 and 291, 4571 and 3346; 622 MB 560 and 481, 8358 and 5935; width
// 2048, 201 MB 241 and 248, 2501 and 2602; 268 MB 303 and 300, 3232 and 3301; 336 MB 383 and 355, 4851 and 4096; width 4096, 470 MB 535 and 494, 7023 and
// 5791.  (As a loop inside a workgroup, before the groups ran as workgroups: 328 MB 342 and 3563, 622 MB 562 and 6146.)
inline bool f32_groups_side_by_side(int groups, int blocks, long long bytes) { return groups > 1 && bytes > (256ll << 20) && blocks <= 8 * 65535; }

// fp32: passes whose products are so small that they are launches more than work
inline bool small_f32(int M, int D) { return M * D <= 16384 && D <= 1024; }

// fp32: whether the GEMM of `cols` (activation) columns behind an RMSNorm of `D` takes the norm along (gemm_f32_kernel, NORM) instead of a launch for it.
// Every workgroup then forms the rows' sums of squares for itself, which costs 17, 22 and 55 us a million rows x columns at width 256, 512 and
// 1024, and a launch is worth 2 to 3.5.  Steps of 2 + 1 layer models with a vocabulary of 1024, with launches and taken along: width 256, 8
// rows 154 and 121 us, 32 159 and 147, 64 191 and 185; width 512, 8 rows 154 and 140, 32 204 and 197; width 1024, 8 rows 197 and 187, 16
// 235 and 229, 32 311 and 320; width 2048, 8 rows 402 and 415, 16 557 and 600.  Verifications of two layers, all with launches and all taken along: width
// 256, vocabulary 8192, 8 rows 87 and 80, 64 rows 142 and 143; 32768, 8 rows 96 and 91, 32 rows 154 and 163; 151936, 8 rows 159 and 169, 64 rows 694 and
// 856; width 1024, 8 rows, 8192 131 and 130, 32768 165 and 172, 151936 372 and 441.
inline bool fold_norm(int M, int D, int cols) { return small_f32(M, D) && (long long)M * D * cols <= 1 << 25; }

// Plain attention kernels: whether a query row's keys are few enough for one workgroup without splits (attn_short_simple_kernel): at most
// a 64-key tile for each of its wavefronts.  `rows`: query rows of all heads, a workgroup each.  They read every key once a row, and with up to 64 keys
// three of four wavefronts have none, so they are for launches that leave the chip room; larger heads fill it sooner.  Two-layer passes with
// splits and a merge launch, and without, at 32, 128 and 256 keys.  fp32: 256 rows of 64 dims 73 and 65, 72 and 66, 74 and 69 us; 512 96 and 86,
// 98 and 89, 101 and 93; 1024 127 and 125, 128 and 129, 139 and 135; 2048 187 and 202, 197 and 207, 210 and 217; 8192 561 and 660, 597 and 677,
// 658 and 705; of 128 dims 512 158 and 152, 159 and 156, 163 and 167; 1024 242 and 248, 247 and 257, 260 and 272.
// bf16: 512 rows of 96 dims 102 and 92, 103 and 96, 107 and 97; 1024 104 and 106, 108 and 109, 122 and 115; 2048 115 and 136, 128 and 137, 146
// and 146; of 32 dims 1024 95 and 88, 99 and 90, 107 and 92; 2048 98 and 107, 109 and 110, 126 and 113; 4096 112 and 144, 130 and 150, 165 and 154;
// of 48 dims 2048 108 and 123, 119 and 128, 135 and 130; 4096 125 and 171, 139 and 175, 170 and 180.  (From three tiles of keys on the splits take more
// than one each.)  Two tiles a wavefront lose (fp32, 316 keys 164 and 170, 508 keys and 32 rows 231 and 238).
inline bool short_context(int rows, int head_dim, int max_tokens, bool bf16) {
  const int limit = !bf16 ? 1 << 16 : max_tokens <= 128 ? 512 * 112 : 1 << 17;
  return max_tokens <= 256 && (long long)rows * head_dim <= limit;
}

// Weight rows per tile of a four-band routed-expert item: 256 (eight wavefronts), or 128 (four) for the short matrices of an odd
// number of 128-row blocks, where the half-empty last 256-row block is a twelfth of the launch or more.  `nt`: 16-row bands of
// the matrix.  Two-layer verifications of 512 rows, 8 of 128 experts, 2048 wide, with 256 and with 128 rows per tile: d_expert 64
// 402 and 388 us, 320 586 and 574, 448 665 and 658, 576 747 and 733, 704 842 and 812 (8 % empty), but 960 939 and 955 (6 %) and 1344
// 1181 and 1192; 192 is 480 and 486 there, 659 and 625 at 896 rows.
inline bool half_height_expert_tiles(int nt) { return nt % 16 != 0 && nt < 96; }

// Argmax of stored logits (fp32 models): whether a row is searched by one workgroup, in one launch, or by 32 and a second launch that combines them.
// A workgroup takes a column a thread and round, a trip to memory each, unless other rows hide it.  Verifications of one layer of width 256, two launches and one: 2048
// columns, 8 rows 38.2 and 37.5 us, 128 75 and 70; 4096, 8 rows 39.2 and 40.8, 128 91 and 89, 512 251 and 235; 8192, 8 rows 42 and 49, 128 123.5 and 126, 512 377
// and 363, 2048 1379 and 1308.
inline bool argmax_in_one_launch(int rows, int V) { return V <= 2048 || (V <= 8192 && V * V <= (long long)rows << 17); }

// ---- sampled acceptance ------------------------------------------------------------------------------------
// Workgroups per row of the statistics launch: enough for 4096 of them (16 a CU), not below 1024 columns each, and no
// more pieces than `room` entries hold.  Workgroups per sequence of the sweep over the vocabulary: 1024 in all, 1024 columns
// each at least, at most `room` in all.
inline int lse_chunks(int rows, int V, size_t room) {
  return (int)std::max<size_t>(1, std::min<size_t>({(size_t)(4096 / rows), (size_t)32, (size_t)(V / 1024), room / rows}));
}
inline int accept_chunks(int S, int V, size_t room) {
  return (int)std::max<size_t>(1, std::min<size_t>({(size_t)(1024 / S), (size_t)64, (size_t)(V / 1024), room / S}));
}
