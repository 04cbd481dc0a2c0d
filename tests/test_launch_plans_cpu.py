"""The rules that choose launches (csrc/plan.h), compiled for the host and run on the CPU."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2602_06036_amd", "csrc")

DRIVER = r"""
#include <stdio.h>
#include "plan.h"
int main() {
  int M, N, K, split, max_rows;
  const Knobs kn = read_knobs();
  while (scanf("%d %d %d %d %d", &M, &N, &K, &split, &max_rows) == 5) {
    const TilePlan t = tile_plan(kn, M, N, K, split != 0, arena_rows(max_rows));
    printf("%d %d %d %d %d\n", t.t->wn, t.t->wm, t.t->wy, t.ks, half_height_expert_tiles(N / 16) ? 128 : 256);
  }
}
"""


@pytest.fixture(scope="session")
def plans(tmp_path_factory):
    d = tmp_path_factory.mktemp("plans")
    (d / "plans.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(d / "plans.cpp"), "-o", str(d / "plans")], check=True)

    def run(queries, **knobs):
        """(weight tiles, bands, wavefronts along N, K ranges, rows of a four-band expert tile) for each (rows, height, K, may split,
        rows of the context)."""
        env = {k: v for k, v in os.environ.items() if not k.startswith("DFLASH_")}
        env.update({"DFLASH_" + k: str(v) for k, v in knobs.items()})
        out = subprocess.run([str(d / "plans")], input="\n".join(" ".join(str(int(x)) for x in q) for q in queries), env=env,
                             capture_output=True, text=True, check=True).stdout
        return [tuple(int(x) for x in line.split()) for line in out.splitlines()]

    return run


def test_forced_k_split_is_taken_whatever_its_value(plans):
    """A number of K ranges that fits (eight k tiles each, slabs inside the arena) is used, and the forced tile with it; one that
    does not fit leaves the choice to the estimate; a launch that may not split ignores the knob."""
    q = (80, 4096, 4096, 1, 400)          # 128 k tiles, room for 1600 rows of slabs
    for ks in range(1, 17):
        assert plans([q], GEMM_KS=ks)[0][3] == ks
        for wn, wm in ((8, 4), (6, 4), (4, 4), (8, 2), (6, 2), (4, 2)):
            assert plans([q], GEMM_KS=ks, GEMM_TILE=wn, GEMM_WM=wm)[0][:4] == (wn, wm, 2, ks)
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
