"""Small test-side helpers: cached float64 weight getters and tiny workloads."""
from dataclasses import replace

import numpy as np

from synth import inputs as si


class W64:
    """Callable name -> float64 array with a cache (tiny models only)."""

    def __init__(self, weights, cache=True):
        self.w = weights
        self.cache = {} if cache else None

    def __call__(self, name):
        if self.cache is None:
            return self.w.f64(name)
        if name not in self.cache:
            self.cache[name] = self.w.f64(name)
        return self.cache[name]


def tiny_workload(seed=0, n_layers=2, draft_layers=1, vocab=1024, block=8, qk_norm=False,
                  kv_heads=4, dtype="f32", n_seqs=1, ctx=(128, 128), taps=None, d=256, heads=4,
                  hd=64, ffn=1024):
    t = si.tiny_dims(n_layers, vocab=vocab, d=d, heads=heads, kv_heads=kv_heads, hd=hd, ffn=ffn,
                     qk_norm=qk_norm)
    dd = replace(t, n_layers=draft_layers)
    taps = taps if taps is not None else (0,)
    return si.Workload("tiny", dtype, t, dd, tuple(taps), vocab - 1, block, n_seqs, ctx[0], ctx[1],
                       0.0, seed)


# Forced shapes of the LDS-staged GEMM over row counts and heights that leave tiles, activation blocks and the XCDs' shares ragged:
# (sequences of 16 rows, FFN width, vocabulary, DFLASH_GEMM_WIDE, _TILE, _WM, _KS).  Rows of the model: d_model 256, QKV 512.  The first two name no shape of four
# wavefronts and get 128 x 128 tiles.
TILE_EDGES = [
    (5, 1056, 1056, 1, 8, 4, 3), (9, 2112, 2080, 1, 8, 4, 0),
    (17, 1312, 2080, 1, 6, 4, 0), (5, 2112, 1056, 1, 6, 4, 6),
    (9, 1056, 1056, 1, 4, 4, 0), (17, 2112, 2048, 1, 4, 4, 3),
    (5, 1312, 2080, 1, 8, 2, 0), (17, 1056, 1056, 1, 8, 2, 2),
    (9, 1312, 2080, 1, 6, 2, 5), (5, 1056, 1056, 1, 4, 2, 0),
    (9, 1056, 2080, 2, 6, 4, 3), (17, 1312, 1056, 2, 6, 4, 0),
    (5, 2112, 1056, 2, 4, 4, 6), (9, 1312, 2080, 2, 4, 4, 0),
    (17, 1056, 2080, 2, 6, 2, 2), (5, 2112, 2080, 2, 6, 2, 6),
    (9, 2112, 1056, 2, 4, 2, 3), (17, 1312, 2080, 2, 4, 2, 0),
]
# The same for the 512 x 128 tiles, whose activation fragments roll (nine activation blocks at last: the weights without the hint of few blocks)
ROLLED_TILES = [(5, 1312, 1056, 2, 8, 4, 3), (9, 1056, 2080, 2, 8, 4, 0), (17, 2112, 2080, 2, 8, 4, 2), (8, 256, 512, 2, 8, 4, 5), (1 + 8 * 8, 1312, 1056, 2, 8, 4, 0)]
# (vocabulary, rows, weight tiles per wavefront) of LM heads that the streaming GEMM takes with eight, six and four weight tiles
STREAM_HEADS = [(v, m, nt) for v, nt in ((32768, 8), (24576, 6), (4096, 4)) for m in (16, 32, 48)]

# Down projections of one band of rows: (d_model, heads, kv heads, FFN width, sequences, block, DFLASH_GEMM_FILL, weight tiles, K ranges, column blocks).
# Four weight tiles and more: the last workgroup of a column block finishes the sums.
LAST_WORKGROUP = [
    (256, 4, 2, 64, 1, 16, 1, 4, 1, 4),       # every workgroup is the last one
    (192, 3, 1, 576, 3, 5, 1, 4, 2, 3),       # a block's workgroups on different XCDs
    (320, 5, 1, 1056, 2, 7, 1, 4, 4, 5),      # an uneven last range
    (576, 9, 3, 4096, 1, 10, 1, 4, 16, 9),
    (1152, 18, 2, 1024, 8, 2, 1, 4, 4, 18),
    (256, 4, 2, 1024, 1, 2, 2, 8, 4, 2),
    (1536, 24, 4, 4160, 1, 16, 1, 6, 16, 16),
    (160, 5, 5, 512, 2, 8, 1, 2, 2, 5),       # two weight tiles, which the finishing kernel is not built for
]
