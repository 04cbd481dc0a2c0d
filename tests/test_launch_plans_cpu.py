"""The rules that choose launches (csrc/plan.h), compiled for the host and run on the CPU."""
import os
import subprocess

import pytest

from tests.helpers import LAST_WORKGROUP, ROLLED_TILES, STREAM_HEADS, TILE_EDGES

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2602_06036_amd", "csrc")

DRIVER = r"""
#include <stdio.h>
#include "plan.h"
int main() {
  int M, N, K, split, max_rows;
  const Knobs kn = read_knobs();
  if (getenv("CONSTANTS")) return printf("%d\n", kSsqAhead), 0;
  if (getenv("PREFILL")) {
    while (scanf("%d %d %d %d %d", &M, &N, &K, &split, &max_rows) == 5) printf("%d\n", attention_by_tiles(M, N, K, split, max_rows, kn.attn_tile_wgs) + 2 * attention_by_tiles(M, N, K, split, max_rows, kn.attn_tile_wgs, true));
    return 0;
  }
  while (scanf("%d %d %d %d %d", &M, &N, &K, &split, &max_rows) == 5) {
    const TilePlan t = tile_plan(kn, M, N, K, split != 0, arena_rows(max_rows));
    const StreamPlan s = stream_plan(kn, M, N, K, split != 0, arena_rows(max_rows)), r = stream_plan(kn, M, N, K, split != 0, arena_rows(max_rows), false);
    const TilePlan tr = tile_plan(kn, M, N, K, split != 0, arena_rows(max_rows), true);
    printf("%d %d %d %d %d %d %d %d %d %d %d %d %d %d %d %d %d %d\n", t.t->wn, t.t->wm, t.t->wy, t.ks, half_height_expert_tiles(N / 16) ? 128 : 256, s.nt, split_f32_columns(N, K, !split) ? 4 : 1,
           short_context(M, K, N, split != 0), fold_norm(M, K, N),
           f32_groups_side_by_side((M + 7) / 8, (N + 3) / 4, (long long)N * K * 4), s.ks, stream_finishes(s), r.nt, r.ks, argmax_in_one_launch(M, N), s.staged + 2 * r.staged, tr.ks, stream_weights(N, M, split != 0));
  }
}
"""


@pytest.fixture(scope="session")
def plans(tmp_path_factory):
    d = tmp_path_factory.mktemp("plans")
    (d / "plans.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(d / "plans.cpp"), "-o", str(d / "plans")], check=True)

    def run(queries, constants=False, prefill=False, **knobs):
        """(weight tiles, bands, wavefronts along N, K ranges, rows of a four-band expert tile, weight tiles of the streaming
        kernel, wavefronts of an fp32 column, whether M query rows of K dims (of bf16, with 'may split') with N
        keys go without splits, whether the norm of K columns goes with the N columns behind it,
        whether groups of eight rows run side by side, K ranges of the streaming kernel, whether its launch may finish its sums,
        weight tiles and K ranges in a routed-expert target's layers, whether the argmax of M rows of N is one launch, whether the streaming plan goes by LDS-staged tiles (2: in a routed
        target's layers), K ranges of the tiled kernel there, whether M activation and N weight blocks (of a
        routed target, with 'may split') read the weights with the hint) for each (rows, height, K, may split, rows of the context)."""
        env = {k: v for k, v in os.environ.items() if not k.startswith("DFLASH_")}
        env.update({"DFLASH_" + k: str(v) for k, v in knobs.items()})
        if constants:
            env["CONSTANTS"] = "1"
        if prefill:   # queries: (tiles, blocks, head groups, cached tokens, tokens of the longest context); 2: a routed target's goes by tiles
            env["PREFILL"] = "1"
        out = subprocess.run([str(d / "plans")], input="\n".join(" ".join(str(int(x)) for x in q) for q in queries), env=env,
                             capture_output=True, text=True, check=True).stdout
        rows = [tuple(int(x) for x in line.split()) for line in out.splitlines()]
        return rows[0] if constants else rows

    return run


def test_forced_k_split_is_taken_whatever_its_value(plans):
    """A number of K ranges that fits (eight k tiles each, slabs inside the arena) is used, and the forced tile with it; one that
    does not fit leaves the choice to the estimate; a launch that may not split ignores the knob."""
    q = (80, 4096, 4096, 1, 400)          # 128 k tiles, room for 1600 rows of slabs
    for ks in range(1, 17):
        assert plans([q], GEMM_KS=ks)[0][3] == ks
        for wn, wm in ((6, 4), (4, 4), (8, 2), (6, 2), (4, 2)):
            assert plans([q], GEMM_KS=ks, GEMM_TILE=wn, GEMM_WM=wm)[0][:4] == (wn, wm, 2, ks)
        assert plans([q], GEMM_KS=ks, GEMM_TILE=8, GEMM_WM=4)[0][:4] == (4, 4, 2, ks)   # no shape of four wavefronts
    assert plans([q], GEMM_KS=17)[0][3] in (1, 2, 3, 4, 6, 8)           # seven k tiles a range
    assert plans([(80, 4096, 4096, 0, 400)], GEMM_KS=5)[0][3] == 1
    assert plans([(400, 4096, 4096, 1, 400)], GEMM_KS=5)[0][3] in (1, 2, 3, 4)   # 2000 rows of slabs, room for 1600


def test_tiles_of_four_band_expert_items_waste_less_than_a_twelfth(plans):
    """Matrices of routed experts are a multiple of 128 rows high; rows past the matrix are work for nothing."""
    heights = [128 * i for i in range(1, 60)]
    for h, p in zip(heights, plans([(512, h, 2048, 0, 512) for h in heights])):
        tile = p[4]
        assert (-h % tile) * 12 < -(-h // tile) * tile, (h, tile)
        assert tile == 256 or h % 256          # the larger tile where it divides


def test_forced_tiles_cover_ragged_geometries(plans):
    """What the GPU tests over TILE_EDGES run: every shape, each with a clamped last weight block; interleaved and contiguous
    shares of the XCDs with several activation blocks; activation blocks of one band; K ranges of 2, 3, 5 and 6, also uneven ones."""
    seen = set()
    for n_seqs, ffn, vocab, wide, tile, wm, ks in TILE_EDGES:
        M = 16 * n_seqs
        mats = [(M, 512, 256, 1, M), (M, 256, 256, 1, M), (M, 2 * ffn, 256, 0, M), (M, 256, ffn, 1, M), (M, vocab, 256, 0, M)]
        for (_, N, K, split, _), (wn, bm, wy, k, *_) in zip(mats, plans(mats, GEMM_WIDE=wide, GEMM_TILE=tile, GEMM_WM=wm, GEMM_KS=ks)):
            assert (wn, bm, wy) == ((tile, wm, 2 * wide) if (tile, wm, wide) != (8, 4, 1) else (4, 4, 2))
            nb, mb = -(-N // 16 // (wy * wn)), -(-n_seqs // (2 * wm))
            shape = (wn, bm, wy)
            if (N // 16) % (wy * wn):
                seen.add(("clamped swiglu" if N == 2 * ffn else "clamped", shape))
            if mb > 1:
                seen.add("interleaved" if nb % 8 == 0 else "contiguous")
            if n_seqs % (2 * wm) == 1:
                seen.add("one band")
            if k > 1:
                seen.add(("K ranges", k, K // 32 % k > 0))
    shapes = {(c[4], c[5], 2 * c[3]) for c in TILE_EDGES} - {(8, 4, 2)}   # no such shape: the default
    assert len(shapes) == 9
    for s in shapes:
        assert ("clamped", s) in seen and ("clamped swiglu", s) in seen, s
    assert {"interleaved", "contiguous", "one band"} <= seen
    assert {c[1] for c in seen if c[0] == "K ranges"} >= {2, 3, 5, 6} and any(c[0] == "K ranges" and c[2] for c in seen)


def test_rolled_tiles_where_the_gpu_test_forces_them_and_over_many_rows(plans):
    for n_seqs, ffn, vocab, wide, tile, wm, ks in ROLLED_TILES:
        M = 16 * n_seqs
        mats = [(M, 512, 256, 1, M), (M, 256, 256, 1, M), (M, 2 * ffn, 256, 0, M), (M, 256, ffn, 1, M), (M, vocab, 256, 0, M)]
        assert all(p[:3] == (8, 4, 4) for p in plans(mats, GEMM_WIDE=wide, GEMM_TILE=tile, GEMM_WM=wm, GEMM_KS=ks))
    assert [p[:4] for p in plans([(2048, 24576, 4096, 0, 2048), (1088, 24576, 4096, 0, 2048), (2048, 4096, 12288, 1, 2048)])] == [(8, 4, 4, 1), (8, 4, 4, 1), (8, 4, 4, 2)]


def test_routed_layers_keep_their_k_ranges(plans):
    """Another order of sums ahead of a router turns near-ties into other experts: QKV and O projections and routers of targets of several widths, whatever the
    costs of the tiles."""
    rows = (80, 128, 160, 200, 256, 288, 320, 384, 448, 512, 1024, 2048)
    want = {(5120, 2048): [3, 3, 2, 3, 3, 2, 2, 1, 2, 2, 1, 1], (2048, 4096): [8, 8, 4, 4, 4, 3, 3, 4, 2, 2, 2, 2],
            (1280, 1024): [4, 4, 4, 4, 4, 4, 4, 3, 3, 3, 1, 1], (2560, 2560): [6, 6, 4, 3, 3, 2, 2, 2, 3, 3, 2, 1],
            (4608, 4096): [3, 3, 4, 3, 3, 4, 4, 3, 2, 3, 1, 1], (8192, 5120): [4, 4, 3, 4, 2, 3, 3, 2, 2, 2, 1, 1],
            (5120, 8192): [6, 6, 4, 3, 3, 4, 3, 4, 3, 3, 3, 1], (128, 4096): [8, 8, 6, 4, 4, 4, 4, 4, 4, 4, 4, 4]}
    for (n, k), ks in want.items():
        assert [p[16] for p in plans([(m, n, k, 1, m) for m in rows])] == ks
    # an unsplit launch, and a forced shape, as anywhere
    assert plans([(512, 5120, 2048, 0, 512)])[0][16] == 1 and plans([(512, 5120, 2048, 1, 512)], GEMM_KS=3)[0][16] == 3


def test_streaming_heads_take_the_weight_tiles_that_the_gpu_test_names(plans):
    q = [(m, v, 256, 0, m) for v, m, _ in STREAM_HEADS]
    assert [p[5] for p in plans(q)] == [nt for _, _, nt in STREAM_HEADS]


def test_small_matrices_of_many_rows_take_four_wavefront_tiles(plans):
    """What the dispatcher picks at the sizes of the GPU test without forced shapes."""
    for n_seqs, d, ffn, vocab in ((5, 256, 1056, 1056), (9, 256, 2560, 4096), (17, 512, 1536, 2080)):
        M = 16 * n_seqs
        q = [(M, d + 256, d, 1, M), (M, d, d, 1, M), (M, 2 * ffn, d, 0, M), (M, d, ffn, 1, M), (M, vocab, d, 0, M)]
        assert all(p[:3] == (4, 2, 2) for p in plans(q))


def test_fp32_columns_are_shared_only_where_that_is_faster(plans):
    """(columns, K, plain or SwiGLU) as measured with one and with four wavefronts a column."""
    four = [(256, 1024, 1), (512, 1024, 1), (768, 1024, 1), (512, 1024, 0), (768, 1536, 0), (512, 2048, 1), (1024, 2048, 0), (1024, 4096, 1),
            (1536, 4096, 0)]
    one = [(1024, 1024, 1), (2048, 1024, 1), (768, 1024, 0), (1536, 1536, 1), (2048, 1536, 1), (2048, 2048, 1), (1536, 2048, 0),
           (4096, 2048, 1), (256, 512, 1), (16384, 1024, 1)]
    got = [p[6] for p in plans([(8, n, k, plain, 8) for n, k, plain in four + one])]
    assert got == [4] * len(four) + [1] * len(one)


def test_deferred_norm_requests_the_pieces_of_8192_wide_rows_ahead(plans):
    """The unsplit projection leaves a piece for 16 columns; rows of up to 8192 are requested ahead of the sweep in whole rounds of 16
    threads and four pieces."""
    (ahead,) = plans([], constants=True)
    assert ahead >= 8192 // 16 and ahead % 64 == 0


def test_plain_attention_goes_without_splits_where_that_is_faster(plans):
    """(query rows of all heads, head dim, keys, bf16) as measured both ways."""
    whole = [(32, 64, 24, 0), (32, 64, 256, 0), (256, 64, 32, 0), (512, 64, 128, 0), (1024, 64, 32, 0), (512, 128, 128, 0), (512, 96, 32, 1), (512, 96, 256, 1),
             (1024, 32, 32, 1), (1024, 96, 144, 1), (2048, 32, 208, 1), (4096, 32, 256, 1), (2048, 48, 256, 1)]
    split = [(32, 64, 257, 0), (512, 96, 272, 1), (2048, 64, 32, 0), (2048, 64, 256, 0), (8192, 64, 64, 0), (1024, 128, 128, 0), (1024, 96, 32, 1), (2048, 32, 32, 1),
             (2048, 96, 128, 1), (2048, 48, 128, 1), (4096, 48, 176, 1), (8192, 96, 256, 1), (16384, 128, 64, 0), (1 << 26, 128, 64, 1)]
    assert [p[7] for p in plans([(r, k, d, bf, 8) for r, d, k, bf in whole + split])] == [1] * len(whole) + [0] * len(split)


def test_fp32_norms_go_with_the_products_that_are_cheaper_for_it(plans):
    """(rows, activation columns, width) as measured both ways: a head of a large vocabulary pays for the norm in every workgroup."""
    along = [(8, 768, 256), (8, 8192, 256), (64, 1024, 256), (32, 2048, 512), (8, 3072, 1024), (16, 1024, 1024)]
    launch = [(64, 8192, 256), (32, 32768, 256), (8, 151936, 256), (64, 4096, 256), (8, 32768, 1024), (8, 8192, 1024), (32, 1024, 1024), (8, 1024, 2048),
              (64, 1 << 28, 256)]
    assert [p[8] for p in plans([(m, n, d, 0, 64) for m, n, d in along + launch])] == [1] * len(along) + [0] * len(launch)


def test_fp32_row_groups_run_side_by_side_where_the_matrix_leaves_the_cache(plans):
    """(rows, columns, K) as measured both ways; a single group has nothing to share, and grid.y holds 65535 blocks of eight."""
    apart = [(8, 151936, 1024), (16, 52000, 1024), (256, 52000, 1024), (64, 65536, 1024), (64, 24576, 2048), (16, 2097153, 1024)]
    beside = [(9, 80000, 1024), (16, 151936, 1024), (256, 151936, 1024), (32, 40960, 2048), (64, 28672, 4096), (16, 2097120, 1024)]
    assert [p[9] for p in plans([(m, n, k, 0, 256) for m, n, k in apart + beside])] == [0] * len(apart) + [1] * len(beside)


def test_down_projections_of_one_band_have_the_plans_that_the_gpu_test_names(plans):
    """Number of K ranges, weight tiles and column blocks of the launches whose last workgroup finishes the sums."""
    for d, _, _, ffn, n_seqs, block, fill, tiles, ranges, blocks in LAST_WORKGROUP:
        M = n_seqs * block
        (p,) = plans([(M, d, ffn, 1, M)], GEMM_FILL=fill)
        assert (p[5], p[10], d // 16 // p[5], p[11]) == (tiles, ranges, blocks, int(tiles >= 4)), (d, ffn)


def test_one_band_of_rows_takes_four_weight_tiles_where_plans_tie(plans):
    """Half the K ranges, so half the slabs; from two bands on, and in the layers of a routed-expert target, whose router's near-ties turn another order of sums
    into another expert, a tie goes to eight tiles."""
    cases = [(4096, 12288, (4, 4), (8, 8)), (4096, 14336, (4, 4), (8, 8)), (2048, 4096, (4, 8), (8, 16)), (5120, 2048, (4, 3), (8, 6)), (6144, 4096, (6, 4), (6, 4))]
    for n, k, dense, routed in cases:
        for m in (1, 16):
            assert [(p[5], p[10], p[12], p[13]) for p in plans([(m, n, k, 1, 16)])] == [dense + routed], (n, k)
    assert [(p[5], p[10]) for p in plans([(32, 4096, 12288, 1, 32), (64, 4096, 12288, 1, 64)])] == [(8, 8), (8, 8)]


def test_split_matrices_of_four_bands_go_by_staged_tiles(plans):
    """(rows, height, K, may split): dense, 49 to 64 rows, blocks of 128 rows that fill the CUs; the model of the GPU test has such a down projection."""
    staged = [(64, 4096, 12288, 1), (49, 4096, 4096, 1), (64, 4096, 20480, 1), (64, 2048, 4096, 1)]
    plain = [(48, 4096, 12288, 1), (64, 24576, 4096, 0), (64, 16384, 4096, 0), (64, 2048, 2048, 1), (64, 6144, 4096, 1), (32, 4096, 12288, 1)]
    assert [p[15] for p in plans([(m, n, k, sp, 64) for m, n, k, sp in staged + plain])] == [1] * len(staged) + [0] * len(plain)


def test_staged_tiles_leave_no_xcd_a_round_more_than_the_others(plans):
    """(height, K) at 64 rows as measured both ways: 20 and 28 blocks of 128 rows give most XCDs 36 workgroups, 28 x 8 and 40 x 6 at most 32, 56 x 9 two rounds."""
    plain = [(2560, 3072), (2560, 8192), (2560, 20480), (3584, 2560), (3584, 8192), (3584, 20480)]
    staged = [(3584, 2048), (5120, 1536), (5120, 8192), (7168, 1024), (7168, 2560), (7168, 16384), (8192, 1024), (8192, 8192)]
    assert [p[15] for p in plans([(64, n, k, 1, 64) for n, k in plain + staged])] == [0] * len(plain) + [1] * len(staged)


def test_argmax_of_stored_logits_is_one_launch_where_that_is_faster(plans):
    """(rows, columns) as measured both ways."""
    one = [(8, 512), (8, 2048), (2048, 2048), (128, 4096), (512, 4096), (512, 8192), (2048, 8192)]
    two = [(8, 2049), (8, 4096), (32, 4096), (8, 8192), (128, 8192), (2048, 8193)]
    assert [p[14] for p in plans([(m, n, 256, 0, m) for m, n in one + two])] == [1] * len(one) + [0] * len(two)


def test_prefill_attention_goes_by_tiles_where_that_is_faster(plans):
    """(prompts of n blocks each, head groups, block, cached tokens) as measured both ways, and the edges of the rule.  A routed target's
    keeps the order of its sums, whatever the knob."""
    def query(blocks, groups, block, cached):
        return sum((n + 1) // 2 for n in blocks), sum(blocks), groups, cached, cached + (max(blocks) + 1) * block

    tiles = [query([128], 8, 16, 0), query([64], 8, 16, 0), query([3, 6, 9, 13, 16, 20], 8, 16, 600), query([32], 32, 16, 0), query([256], 8, 8, 0),
             query([8] * 16, 16, 16, 2000), query([150], 8, 10, 768)]
    blocks = [query([22] * 6, 8, 16, 4000), query([11] * 12, 8, 16, 2652), query([20], 8, 16, 0), query([62], 8, 16, 0), query([125], 8, 16, 4000), query([8] * 32, 8, 8, 69),
              query([43] * 3, 8, 16, 1618), query([150], 8, 10, 769), query([14] * 16, 8, 16, 0)]
    assert [p[0] for p in plans(tiles + blocks, prefill=True)] == [1] * len(tiles) + [0] * len(blocks)
    # longest contexts on both sides of the lines
    assert [p[0] for p in plans([(128, 256, 8, 0, n) for n in (255, 256, 3072, 3073)], prefill=True)] == [0, 1, 1, 0]
    # set by hand, the number of workgroups decides alone
    assert [p[0] for p in plans(tiles + blocks, prefill=True, ATTN_TILE_WGS=1)] == [1] * (len(tiles) + len(blocks))
    assert [p[0] for p in plans([(1, 2, 8, 0, 48), (2, 4, 8, 5000, 6000)], prefill=True, ATTN_TILE_WGS=16)] == [0, 1]


def test_weights_carry_the_hint_where_their_blocks_divide_by_the_xcds(plans):
    """(activation blocks, weight blocks, routed)."""
    hint = [(1, 16, 0), (8, 64, 0), (2, 20, 1), (8, 12, 1)]
    none = [(9, 64, 0), (2, 20, 0), (3, 67, 0), (8, 12, 0), (9, 20, 1)]
    assert [p[17] for p in plans([(m, n, 256, r, 64) for m, n, r in hint + none])] == [1] * len(hint) + [0] * len(none)
