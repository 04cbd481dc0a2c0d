"""Sizes at which single kernels can go wrong (edges of chunks and tiles, remainders, alignment, masked values), each
against the CPU oracle."""
from dataclasses import replace

import numpy as np
import pytest

from oracle import dflash_oracle as O
from synth import inputs as si
from tests.helpers import LAST_WORKGROUP, ROLLED_TILES, STREAM_HEADS, TILE_EDGES, W64, tiny_workload
from tests.test_gpu_parity import ROUTE_CLEAR, Lockstep, _gpu

pytestmark = pytest.mark.gpu

PROF_ATTN, PROF_ATTN_MERGE = 3, 4   # classes of dflash_profile_read


@pytest.mark.parametrize("S,B,V,T,shift", [
    (1, 2, 8, 1.0, 0),          # one chunk, fewer columns than threads
    (3, 5, 1003, 0.7, 0),       # rows of odd length: no 16-byte loads
    (2, 16, 2052, 1.0, 1),      # whole 16-byte rows behind a pointer that is not 16-byte aligned
    (5, 16, 33000, 0.7, 0),     # several chunks per row and per sequence, ragged last ones
    (300, 2, 1040, 1.0, 0),     # many sequences: few chunks
    (1, 16, 151936, 1.0, 0),
    (256, 16, 64, 1.0, 0),      # the most rows the entry point takes
    (1, 2, 164096, 1.0, 0),     # eight columns a piece behind a whole round
])
def test_sampled_acceptance_on_held_logits(S, B, V, T, shift):
    """dflash_accept_sampled_noalloc against the oracle's acceptance rule, with masked (-inf) columns and, for some
    sequences, every slot accepted (uniforms of 0, p = q).  A sequence whose decision hangs on less than 1e-4 (u q against
    p, or the two best scores: fp32 logits of magnitude ~10 are good to 1e-6, their exponentials to ~1e-5) is left out."""
    import torch
    _gpu()
    from paper_2602_06036_amd import binding as Bd
    rng = np.random.default_rng([S, B, V])
    q = (2.5 * rng.standard_normal((S, B, V))).astype(np.float32)
    p = (2.5 * rng.standard_normal((S, B, V))).astype(np.float32)
    p[:, :-1] = q[:, 1:] + (0.5 * rng.standard_normal((S, B - 1, V))).astype(np.float32)
    p[1::3, :-1] = q[1::3, 1:]
    masked = rng.choice(V, max(1, V // 7), replace=False)
    p[:, :, masked] = -np.inf
    q[:, :, masked] = -np.inf
    d = np.zeros((S, B), np.int32)
    for s in range(S):
        for j in range(B):
            d[s, j] = int(np.argmax(q[s, j] / T + rng.gumbel(size=V)))
    u = rng.random((S, B)).astype(np.float32)
    u[1::3] = 0.0
    key = 987654321
    dev = "cuda:0"

    def up(x):
        flat = torch.zeros(x.size + 4, dtype=torch.float32, device=dev)
        v = flat[shift:shift + x.size].view(x.shape)
        v.copy_(torch.from_numpy(x))
        return v

    acc = torch.full((S,), -7, dtype=torch.int32, device=dev)
    out = torch.full((S, B), -7, dtype=torch.int32, device=dev)
    for _ in range(2):
        Bd.dflash_accept_sampled_noalloc(up(p), up(q), torch.from_numpy(d).to(dev), torch.from_numpy(u).to(dev),
                                         torch.tensor([key], dtype=torch.int64, device=dev), T, acc, out)
    acc, out = acc.cpu().numpy(), out.cpu().numpy()
    checked = 0
    for s in range(S):
        P, Q = O.softmax(p[s].astype(np.float64) / T), O.softmax(q[s].astype(np.float64) / T)
        rec = {}

        def draw(w, slot, purpose):
            with np.errstate(divide="ignore"):
                rec["scores"] = O.gumbel_scores(np.log(w), key, s, slot, purpose)
            return int(np.argmax(rec["scores"]))

        a, tok = O.sampling_accept(P, Q, list(d[s]), list(u[s]), draw)
        gaps = [abs(u[s, j] * Q[j, d[s, j]] / P[j - 1, d[s, j]] - 1.0) for j in range(1, min(a + 2, B))]
        top = np.sort(rec["scores"][np.isfinite(rec["scores"])])[-2:]
        if min(gaps) < 1e-4 or (top.size == 2 and top[1] - top[0] < 1e-4):
            continue
        checked += 1
        assert acc[s] == a, (s, acc[s], a)
        want = [int(x) for x in d[s, 1:a + 1]] + [tok] + [-1] * (B - a - 1)
        assert list(out[s]) == want, (s, a)
    assert checked >= 0.9 * S


@pytest.mark.parametrize("hd,heads,kv_heads,ffn,lens", [
    (16, 4, 4, 64, (1, 63)),          # a quarter of the lanes own a head dim; K = 64
    (48, 4, 2, 1040, (64, 65)),       # down projection with its K over four wavefronts, the last piece short
    (96, 6, 2, 2048, (15, 200)),      # second half of the head dims ragged; several chunks of keys
    (128, 2, 1, 512, (129, 16)),
])
def test_fp32_head_dims_and_widths(hd, heads, kv_heads, ffn, lens):
    """fp32 models: generic attention and GEMM kernels over head dims, head groups, widths and context lengths."""
    w = tiny_workload(seed=hd + ffn, n_layers=2, draft_layers=1, vocab=512, block=8, qk_norm=True, kv_heads=kv_heads, n_seqs=2,
                      taps=(0, 1), d=hd * heads, heads=heads, hd=hd, ffn=ffn)
    prompts = [p[:n] for p, n in zip(si.make_prompts(replace(w, ctx_min=200, ctx_max=200)), lens)]
    ls = Lockstep(w, prompts, max_len=200 + 6 * 8)
    _, _, mism = ls.prefill()
    assert not mism
    for i, plan in enumerate([[0, 7], [7, 3], None]):
        ls.step(plan=plan, step_idx=i)
    ls.check_cache([0, 1], [0])
    assert ls.stats["reseeds"] == 0


@pytest.mark.parametrize("hd,qk_norm", [(64, False), (64, True), (128, False), (128, True)])
def test_rotated_keys_are_rounded_in_the_stated_order(hd, qk_norm):
    """q/k norm and rotation, bit for bit: with W_k = W_v = 1 the cached V rows are the vectors that the kernel normalises and
    rotates into the K rows.  Every operation is rounded to fp32, products that a sum takes in unrounded are the ones the kernel
    names (evaluated here with 64 significand bits and rounded once)."""
    from paper_2602_06036_amd import binding as Bd
    GpuModel = _gpu()
    d, f32 = 256, np.float32
    w = tiny_workload(seed=hd, n_layers=1, draft_layers=1, vocab=512, block=16, qk_norm=qk_norm, kv_heads=d // hd, n_seqs=2, taps=(0,),
                      d=d, heads=d // hd, hd=hd, ffn=256)
    wt, wd = si.make_weights(w, 4)
    wt.t["L0.wk"], wt.t["L0.wv"] = np.eye(d, dtype=f32), np.eye(d, dtype=f32)
    g = GpuModel(w, wt, wd, 80, n_seqs=2)
    g.prefill([p[:n] for p, n in zip(si.make_prompts(replace(w, ctx_min=48, ctx_max=48)), (48, 37))])

    def fma(a, b, c):
        return (a.astype(np.longdouble) * b + c).astype(f32)

    half = hd // 2
    freq = np.exp(-np.log(np.float64(f32(w.target.rope_theta))) * (2.0 * np.arange(half) / hd))
    for s, n in enumerate((48, 37)):
        k, x = (r.cpu().numpy() for r in Bd.dflash_kv_read(g.e, g.batch(), Bd.DFLASH_POOL_TARGET, 0, s, 0, n))
        x1, x2 = x[..., :half], x[..., half:]
        if qk_norm:
            ss = np.zeros(x1.shape[:-1] + (64,), f32)
            ss[..., :half] = fma(x2, x2, x1 * x1)
            for o in (32, 16, 8, 4, 2, 1):
                ss = ss + ss[..., np.arange(64) ^ o]
            rstd = f32(1) / np.sqrt(ss[..., :half] / f32(hd) + f32(w.target.rms_eps))
            x1, x2 = x1 * (rstd * wt.t["L0.kn"][:half]), x2 * (rstd * wt.t["L0.kn"][half:])
        ang = np.arange(n)[:, None, None] * freq
        c, sn = np.cos(ang).astype(f32), np.sin(ang).astype(f32)
        want = np.concatenate([fma(x1, c, -(x2 * sn)), fma(x2, c, x1 * sn)], -1)
        assert k.dtype == want.dtype == f32
        wrong = int((k != want).sum())
        assert wrong == 0, (wrong, k.size)
    g.e.close()


def _many_rows(n_seqs, d, ffn, vocab):
    """Prefill, a planned and a free greedy step and a sampled one; returns the launches per kernel family of the steps."""
    w = tiny_workload(seed=d + ffn, n_layers=2, draft_layers=1, vocab=vocab, block=16, qk_norm=True, kv_heads=2, dtype="bf16",
                      n_seqs=n_seqs, taps=(0, 1), d=d, heads=d // 64, hd=64, ffn=ffn)
    lens = [20 + (7 * i) % 31 for i in range(n_seqs)]
    prompts = [p[:n] for p, n in zip(si.make_prompts(replace(w, ctx_min=60, ctx_max=60)), lens)]
    ls = Lockstep(w, prompts, max_len=60 + 4 * 16)
    ls.prefill()
    ls.g.e.gemm_counts()
    ls.step(plan=[(5 * s) % 16 for s in range(n_seqs)], step_idx=0)
    ls.step(step_idx=1)
    ls.step(temperature=0.8, step_idx=2, key=11)
    counts = ls.g.e.gemm_counts()
    ls.check_cache([0, 1], [0])
    assert ls.stats["low_margin_flips"] <= 0.02 * ls.stats["rows"] + 2
    assert ls.stats["reseeds"] <= 1
    return counts


@pytest.mark.parametrize("n_seqs,d,ffn,vocab", [
    (5, 256, 1056, 1008),       # 80 rows; an LM head of 63 row bands, which the LDS-staged kernel does not take
    (9, 256, 2560, 4096),       # 144 rows
    (17, 512, 1536, 2064),      # 272 rows; an LM head of 129 row bands
])
def test_bf16_tile_edges_many_rows(n_seqs, d, ffn, vocab):
    """The GEMMs of many rows with the shapes and K splits that the dispatcher picks for small matrices: four-wavefront 128 x 64 tiles."""
    counts = _many_rows(n_seqs, d, ffn, vocab)
    assert counts[1] > 0 and counts[2] == 0 and (counts[0] > 0) == (vocab % 32 != 0)


@pytest.mark.parametrize("n_seqs,ffn,vocab,wide,tile,wm,ks", TILE_EDGES)
def test_forced_tiles_over_ragged_sizes(n_seqs, ffn, vocab, wide, tile, wm, ks, monkeypatch):
    """Every tile shape of the LDS-staged GEMM, SwiGLU, K-split and LM-head epilogues (argmax, Gumbel-max, softmax statistics), with
    clamped last weight blocks, partly filled activation blocks and both mappings to the XCDs; the geometries are listed and checked
    in test_launch_plans_cpu.py."""
    for k, v in (("WIDE", wide), ("TILE", tile), ("WM", wm), ("KS", ks)):
        monkeypatch.setenv("DFLASH_GEMM_" + k, str(v))
    counts = _many_rows(n_seqs, 256, ffn, vocab)
    assert counts[wide] > 0 and counts[3 - wide] == 0 and counts[0] == 0


@pytest.mark.parametrize("n_seqs,block,ffn", [(4, 16, 4096), (7, 7, 4224), (5, 11, 4096)])
def test_four_bands_of_rows_by_staged_tiles(n_seqs, block, ffn):
    """64, 49 and 55 rows: the down projection of a 2048-wide model as 16 blocks x 16 K ranges of the LDS-staged kernel (the last one uneven)."""
    w = tiny_workload(seed=ffn + block, n_layers=2, draft_layers=1, vocab=512, block=block, qk_norm=True, kv_heads=4, dtype="bf16", n_seqs=n_seqs,
                      taps=(0, 1), d=2048, heads=32, hd=64, ffn=ffn)
    lens = [9 + 5 * i for i in range(n_seqs)]
    prompts = [p[:n] for p, n in zip(si.make_prompts(replace(w, ctx_min=60, ctx_max=60)), lens)]
    ls = Lockstep(w, prompts, max_len=60 + 4 * block)
    ls.prefill()
    ls.g.e.gemm_counts()
    ls.step(plan=[(5 * s) % block for s in range(n_seqs)], step_idx=0)
    assert ls.g.e.gemm_counts()[1] > 0
    ls.check_cache([0, 1], [0])
    assert ls.stats["reseeds"] <= 1


@pytest.mark.parametrize("heads,kv_heads,block,lens,max_seqs,pieces", [
    (8, 2, 16, (16, 17, 150, 33), 16, 1),       # one block and two of them a tile; a last block of one row
    (8, 2, 16, (97, 5, 160), 6, 2),             # several passes, prompts cut at odd blocks; the second call behind cached rows
    (4, 4, 16, (70, 31), 8, 1),                 # sixteen query rows of a group of heads
    (8, 1, 16, (90, 49), 12, 3),                # two groups of heads share a kv head
    (8, 2, 10, (44, 71), 9, 2),                 # blocks that straddle pages
    (6, 2, 5, (23, 37, 4), 7, 1),               # fifteen query rows
    (4, 2, 16, (1100,), 69, 1),                 # page ids beyond the first set of 32 pairs
    (4, 2, 16, (2100, 40), 140, 1),             # ... the third set, loaded inside the loop
    (4, 2, 16, (3150,), 197, 1),                # ... and the fourth
])
def test_prefill_attention_by_tiles(heads, kv_heads, block, lens, max_seqs, pieces, monkeypatch):
    """dflash_prefill with the attention that takes two blocks of a prompt together, forced at every size."""
    monkeypatch.setenv("DFLASH_ATTN_TILE_WGS", "1")
    n = len(lens)
    w = tiny_workload(seed=heads + block, n_layers=2, draft_layers=1, vocab=512, block=block, qk_norm=True, kv_heads=kv_heads, dtype="bf16", n_seqs=n,
                      taps=(0, 1), d=256, heads=heads, hd=128, ffn=512)
    prompts = [p[:k] for p, k in zip(si.make_prompts(replace(w, ctx_min=max(lens), ctx_max=max(lens))), lens)]
    ls = Lockstep(w, prompts, max_len=max(lens) + 5 * block, max_seqs=max_seqs)
    ls.g.e.profile_enable(True)
    ls.prefill(entry=True, pieces=pieces)
    launches = ls.g.e.profile_read()
    ls.g.e.profile_enable(False)
    # by tiles a pass has one attention launch a layer; by blocks, contexts of more than 64 tokens are split over workgroups and merged
    assert launches[PROF_ATTN][1] % 2 == 0 and PROF_ATTN_MERGE not in launches, launches
    ls.check_cache([0, 1], [0])
    ls.step(plan=[(3 * s + 1) % block for s in range(n)], step_idx=0)
    assert ls.stats["reseeds"] <= 1


@pytest.mark.parametrize("poisoned", ["one key", "all keys"])
@pytest.mark.parametrize("ctx", [90, 1500])
def test_nan_scores_make_a_row_nan_in_a_prefill_by_tiles(ctx, poisoned, monkeypatch):
    """A cached key (or every one) of sequence 0 is NaN in the first layer: its new rows are NaN in the second, those of the other sequences keep their bits."""
    import torch
    _gpu()
    import paper_2602_06036_amd as dfl
    from paper_2602_06036_amd import binding as Bd
    from tests.gpu_harness import GpuModel
    monkeypatch.setenv("DFLASH_ATTN_TILE_WGS", "1")
    w = tiny_workload(seed=ctx, n_layers=2, draft_layers=1, vocab=256, block=16, qk_norm=True, kv_heads=2, dtype="bf16", n_seqs=3, taps=(0,), d=256, heads=8, hd=128,
                      ffn=256)
    lens, new = [ctx, 13, ctx - 1], [55, 40, 17]
    g = GpuModel(w, *si.make_weights(w), ctx + 80, max_seqs=9)
    rng = np.random.default_rng(1)
    g.host_lens = np.array(lens, dtype=np.int64)
    g.seq_lens.copy_(torch.tensor(lens, dtype=torch.int32))
    for s, n in enumerate(lens):
        for l in range(2):
            g.write_kv(Bd.DFLASH_POOL_TARGET, l, s, 0, *(rng.standard_normal((n, 2, 128)).astype(np.float32) for _ in range(2)))
    tokens = torch.from_numpy(rng.integers(0, 255, sum(new)).astype(np.int32)).cuda()
    first = torch.zeros(3, dtype=torch.int32, device="cuda")

    def rows():
        g.seq_lens.copy_(torch.tensor(lens, dtype=torch.int32))
        g.e.profile_enable(True)
        dfl.dflash_prefill(g.e, g.batch(), tokens, new, first)
        launches = g.e.profile_read()
        g.e.profile_enable(False)
        g.e.device_status()
        assert launches[PROF_ATTN][1] == 2 and PROF_ATTN_MERGE not in launches, launches
        return [np.stack(g.read_kv(Bd.DFLASH_POOL_TARGET, 1, s, lens[s], new[s])) for s in range(3)]

    sound = rows()
    assert all(np.isfinite(x).all() for x in sound)
    at, n = (77, 1) if poisoned == "one key" else (0, ctx)
    bad = np.full((n, 2, 128), np.nan, dtype=np.float32)
    g.write_kv(Bd.DFLASH_POOL_TARGET, 0, 0, at, bad, rng.standard_normal(bad.shape).astype(np.float32))
    got = rows()
    assert np.isnan(got[0]).all()
    assert all(np.array_equal(x, y) for x, y in zip(got[1:], sound[1:]))


def test_prefill_attention_of_a_routed_target_stays_with_the_blocks(monkeypatch):
    """Whatever the knob asks for: the same bits of the new rows, from launches with a merge behind them."""
    import torch
    _gpu()
    import paper_2602_06036_amd as dfl
    from paper_2602_06036_amd import binding as Bd
    from tests.gpu_harness import GpuModel
    w = si.small_moe_workload(n_seqs=2, ctx_min=100, ctx_max=100, seed=5, n_experts=16, top_k=2)
    wts, blobs, got = si.make_weights(w), None, []
    new = [130, 70]
    tokens = torch.from_numpy(np.random.default_rng(2).integers(0, 255, sum(new)).astype(np.int32)).cuda()
    first = torch.zeros(2, dtype=torch.int32, device="cuda")
    for wgs in ("256", "1"):
        monkeypatch.setenv("DFLASH_ATTN_TILE_WGS", wgs)
        g = GpuModel(w, *wts, 160, blobs=blobs, max_seqs=14)
        blobs = g.blobs()
        g.e.profile_enable(True)
        dfl.dflash_prefill(g.e, g.batch(), tokens, new, first)
        launches = g.e.profile_read()
        g.e.profile_enable(False)
        g.e.device_status()
        assert launches[PROF_ATTN][1] == launches[PROF_ATTN_MERGE][1] == w.target.n_layers
        g.host_lens = np.array(new, dtype=np.int64)
        got.append([np.stack(g.read_kv(Bd.DFLASH_POOL_TARGET, w.target.n_layers - 1, s, 0, n)) for s, n in enumerate(new)])
    assert all(np.isfinite(x).all() and np.array_equal(x, y) for x, y in zip(*got))


@pytest.mark.parametrize("n_seqs,ffn,vocab,wide,tile,wm,ks", ROLLED_TILES)
def test_rolled_tiles_over_ragged_sizes(n_seqs, ffn, vocab, wide, tile, wm, ks, monkeypatch):
    """512 x 128 tiles: clamped last weight blocks, activation blocks of one band, K ranges of a k tile or two (shorter than the ring), odd numbers of k tiles."""
    test_forced_tiles_over_ragged_sizes(n_seqs, ffn, vocab, wide, tile, wm, ks, monkeypatch)


@pytest.mark.parametrize("d,heads,kv_heads,hd,ffn,vocab,n_seqs,block,lens", [
    (256, 4, 4, 64, 1024, 1024, 1, 2, (5,)),              # two rows
    (256, 4, 2, 64, 1024, 8192, 3, 7, (63, 64, 130)),     # 21 rows: a last piece of five; a launch before the head
    (256, 4, 2, 64, 512, 2048, 2, 4, (9, 30)),            # the longest row that one workgroup searches whatever the number of rows
    (256, 4, 2, 64, 512, 2056, 2, 4, (9, 30)),            # ... 32 workgroups
    (256, 4, 2, 64, 256, 4096, 16, 16, (9, 30, 5, 17) * 4),   # ... and one again where there are rows enough
    (256, 4, 4, 64, 512, 8208, 3, 8, (9, 233, 240)),      # 24 rows and 256 keys at first, more behind: one workgroup, then splits
    (256, 4, 4, 64, 512, 512, 9, 7, (20, 31, 8, 90, 64, 1, 3, 5, 7)),   # 63 rows
    (256, 4, 1, 64, 512, 512, 5, 13, (20, 31, 8, 90, 64)),              # 65 rows: norm launches
    (256, 4, 4, 64, 2064, 512, 8, 8, (20, 31, 8, 90, 64, 1, 3, 5)),     # 64 rows: launches in front of the gate/up products only
    (1024, 4, 1, 128, 256, 640, 2, 8, (17, 120)),         # 16 rows; four wavefronts a column in SwiGLU products; head dim 128
    (1024, 4, 1, 128, 256, 640, 1, 7, (33,)),             # ... and in plain ones
])
def test_fp32_folded_norms_and_short_contexts(d, heads, kv_heads, hd, ffn, vocab, n_seqs, block, lens):
    """The RMSNorms that GEMMs take along, taps of an inner and the last layer, attention by one workgroup a row and the argmax of one
    launch, on both sides of the lines where they end."""
    w = tiny_workload(seed=ffn + vocab, n_layers=3, draft_layers=2, vocab=vocab, block=block, qk_norm=True, kv_heads=kv_heads, n_seqs=n_seqs,
                      taps=(1, 2), d=d, heads=heads, hd=hd, ffn=ffn)
    prompts = [p[:n] for p, n in zip(si.make_prompts(replace(w, ctx_min=max(lens), ctx_max=max(lens))), lens)]
    ls = Lockstep(w, prompts, max_len=max(lens) + 5 * block)
    ls.prefill()
    for i, plan in enumerate((None, [block - 1] * n_seqs, [(3 * s + 1) % block for s in range(n_seqs)], None)):
        ls.step(plan=plan, step_idx=i)
    ls.check_cache([0, 2], [0, 1])
    assert ls.stats["reseeds"] == 0


def test_fp32_row_groups_side_by_side_on_a_matrix_that_leaves_the_cache():
    """An LM head of 65605 rows of 1024 (269 MB; 16402 column blocks, no multiple of eight) over 21 rows, three groups of which the last has five: every column
    with the bits that it has in a head of the first and one of the last 16384 rows, whose groups run one after the other."""
    import torch
    _gpu()
    import paper_2602_06036_amd as dfl
    from tests.gpu_harness import GpuModel
    V, n, kw = 65605, 16384, dict(seed=5, n_layers=1, draft_layers=1, block=7, kv_heads=1, n_seqs=3, taps=(0,), d=1024, heads=4, hd=64, ffn=64)
    wt, wd = si.make_weights(tiny_workload(vocab=V, **kw))
    embed, head = wt.t["E"], wt.t["lm"]
    tokens = torch.from_numpy(np.random.default_rng(2).integers(0, n, (3, 7)).astype(np.int32)).cuda()

    def logits(rows):
        wt.t["E"], wt.t["lm"] = wd.t["E"], wd.t["lm"] = embed[:len(rows)], rows
        g = GpuModel(tiny_workload(vocab=len(rows), **kw), wt, wd, 32)
        dfl.dflash_verify(g.e, g.batch(), tokens, g.tgt_argmax, g.logits_t)
        g.e.device_status()
        assert np.array_equal(g.tgt_argmax.cpu().numpy(), g.logits_t.argmax(-1).to(torch.int32).cpu().numpy())
        return g.logits_t.cpu().numpy().copy()

    whole = logits(head)
    assert np.array_equal(whole[..., :n], logits(head[:n]))
    assert np.array_equal(whole[..., -n:], logits(head[-n:]))
    assert np.isfinite(whole).all() and (np.abs(whole).max(axis=(0, 1)) > 0).all()


@pytest.mark.parametrize("hd,heads,kv_heads,n_seqs,block,wide_from", [
    (128, 4, 2, 3, 16, 64),        # key-split kernel
    (128, 8, 2, 2, 7, 64),         # ... with a block that is no whole band: two sequences' rows in one operand tile
    (128, 8, 1, 2, 16, 64),        # ... with two workgroups a kv head
    (128, 4, 4, 17, 2, 100000),    # row-split kernel, 34 rows
    (64, 8, 2, 3, 16, 100000),
    (64, 8, 1, 2, 11, 100000),     # ... two workgroups a kv head
])
def test_attention_of_one_split_writes_the_operand(hd, heads, kv_heads, n_seqs, block, wide_from, monkeypatch):
    """One context split a sequence (many sequences, or short ones): the attention kernels divide by the row sums and write the O
    projection's operand themselves, causal and not.  Ragged contexts around a page and a pair of pages."""
    monkeypatch.setenv("DFLASH_ATTN_TARGET_WGS", "1")
    monkeypatch.setenv("DFLASH_ATTN_WIDE_MIN_CHUNK", str(wide_from))
    w = tiny_workload(seed=hd + heads, n_layers=2, draft_layers=2, vocab=512, block=block, qk_norm=True, kv_heads=kv_heads, dtype="bf16",
                      n_seqs=n_seqs, taps=(0, 1), d=256, heads=heads, hd=hd, ffn=512)
    lens = [(13, 64, 33, 150, 16, 31, 96)[i % 7] for i in range(n_seqs)]
    prompts = [p[:n] for p, n in zip(si.make_prompts(replace(w, ctx_min=150, ctx_max=150)), lens)]
    ls = Lockstep(w, prompts, max_len=150 + 5 * 16)
    ls.prefill()
    for i, plan in enumerate((None, [(3 * s + 1) % block for s in range(n_seqs)], None)):
        ls.step(plan=plan, step_idx=i)
    ls.check_cache([0, 1], [0, 1])
    assert ls.stats["low_margin_flips"] <= 0.02 * ls.stats["rows"] + 2
    assert ls.stats["reseeds"] <= 1


@pytest.mark.parametrize("d,heads,kv_heads,ffn,n_seqs,block,fill,tiles,ranges,blocks", LAST_WORKGROUP)
def test_residual_update_by_the_last_workgroup(d, heads, kv_heads, ffn, n_seqs, block, fill, tiles, ranges, blocks, monkeypatch):
    """The down projection of up to 16 rows, whose K ranges are summed by the last workgroup of a column block, over the numbers of
    ranges, column blocks and weight tiles that its plan can have; an inner and the last layer are tapped.  Several steps on one
    context; the launches that update the residual stream themselves are counted."""
    monkeypatch.setenv("DFLASH_GEMM_FILL", str(fill))
    w = tiny_workload(seed=d + ffn, n_layers=3, draft_layers=2, vocab=512, block=block, qk_norm=True, kv_heads=kv_heads, dtype="bf16",
                      n_seqs=n_seqs, taps=(1, 2), d=d, heads=heads, hd=d // heads, ffn=ffn)
    prompts = [p[:11 + 5 * i] for i, p in enumerate(si.make_prompts(replace(w, ctx_min=64, ctx_max=64)))]
    ls = Lockstep(w, prompts, max_len=64 + 5 * 16)
    ls.prefill()
    for i, plan in enumerate((None, [(3 * s + 1) % block for s in range(n_seqs)], None)):
        ls.g.e.gemm_counts()
        ls.step(plan=plan, step_idx=i)
        # O projections of three and two layers, and the down projections but for the models' last layers
        assert ls.g.e.gemm_counts()[3] == 5 + (3 if tiles >= 4 else 0)
    ls.check_cache([0, 2], [0, 1])
    assert ls.stats["low_margin_flips"] <= 0.02 * ls.stats["rows"] + 2
    assert ls.stats["reseeds"] <= 1


@pytest.mark.parametrize("d,ffn", [
    (4128, 576),      # 258 pieces from the O projection, 43 from the down projection: last groups of two and three
    (4160, 64),       # 260 and 65
    (8192, 64),       # 512: all of them requested ahead
    (8288, 64),       # 518: the last six behind the sweep
])
def test_deferred_norm_of_wide_rows(d, ffn):
    """One band of rows of models wider than 4096: the deferred RMSNorm adds more than 256 pieces of the sums of squares, a number of them
    that is no whole number of groups of four among them.  The last 96 columns of the embedding hold most of a row's energy, so that one of the
    last six pieces lost or doubled is a seventh of the sum (7 % of the norm, some 0.1 in the logits; the bound is 2e-2); the workspace is NaN
    where nothing is written, behind a row's last piece for one."""
    w = tiny_workload(seed=d, n_layers=2, draft_layers=1, vocab=256, block=5, qk_norm=True, kv_heads=1, dtype="bf16", n_seqs=3, taps=(0, 1), d=d,
                      heads=2, hd=64, ffn=ffn)
    wt, wd = si.make_weights(w)
    e = si.bf16_bits_to_f32(wt.t["E"])
    e[:, -96:] *= 256.0
    wt.t["E"] = wd.t["E"] = si.f32_to_bf16_bits(e)
    prompts = [p[:n] for p, n in zip(si.make_prompts(replace(w, ctx_min=33, ctx_max=33)), (7, 33, 16))]
    ls = Lockstep(w, prompts, max_len=64, weights=(wt, wd, W64(wt), W64(wd)))
    ls.g.e.workspace[256:].fill_(255)
    ls.prefill()
    for i, plan in enumerate((None, [2, 0, 4])):
        ls.g.e.workspace[256:].fill_(255)
        ls.step(plan=plan, step_idx=i)
    ls.check_cache([0, 1], [0])
    assert ls.stats["low_margin_flips"] <= 0.02 * ls.stats["rows"] + 2
    assert ls.stats["reseeds"] <= 1


@pytest.mark.parametrize("dtype,hd,heads,kv_heads,n_seqs,block,ctx,wgs,wide_from", [
    ("bf16", 128, 4, 2, 3, 16, 150, 1, 64),         # key-split kernel, whole contexts
    ("bf16", 128, 4, 2, 3, 16, 150, 256, 64),       # ... and split, merged row by row
    ("bf16", 128, 4, 2, 9, 16, 150, 256, 64),       # ... merged in bands of rows
    ("bf16", 64, 8, 2, 3, 16, 150, 1, 100000),      # row-split kernel, whole and split
    ("bf16", 64, 8, 2, 3, 16, 150, 256, 100000),
    ("bf16", 96, 4, 4, 3, 8, 150, 256, 512),        # the plain kernels: one workgroup a row ...
    ("f32", 64, 4, 4, 3, 8, 150, 256, 512),
    ("f32", 64, 4, 4, 3, 8, 300, 256, 512),         # ... splits
    ("f32", 64, 4, 4, 3, 8, 300, 1, 512),
])
@pytest.mark.parametrize("poisoned", ["one key", "all keys"])
def test_nan_scores_make_a_row_nan_however_its_context_is_split(dtype, hd, heads, kv_heads, n_seqs, block, ctx, wgs, wide_from, poisoned, monkeypatch):
    """A cached key (or every one) of sequence 0 is NaN in the first layer: all its logits are NaN, as a softmax over them is; the other sequences keep
    their bits."""
    monkeypatch.setenv("DFLASH_ATTN_TARGET_WGS", str(wgs))
    monkeypatch.setenv("DFLASH_ATTN_WIDE_MIN_CHUNK", str(wide_from))
    import torch
    _gpu()
    import paper_2602_06036_amd as dfl
    from paper_2602_06036_amd import binding as Bd
    from tests.gpu_harness import GpuModel
    w = tiny_workload(seed=ctx + hd, n_layers=2, draft_layers=1, vocab=256, block=block, qk_norm=True, kv_heads=kv_heads, dtype=dtype, n_seqs=n_seqs,
                      taps=(0,), d=256, heads=heads, hd=hd, ffn=256)
    g = GpuModel(w, *si.make_weights(w), ctx + 2 * block)
    lens = [ctx] + [(13, 64, 33, ctx - 1)[i % 4] for i in range(n_seqs - 1)]
    rng = np.random.default_rng(1)
    g.host_lens = np.array(lens, dtype=np.int64)
    g.seq_lens.copy_(torch.tensor(lens, dtype=torch.int32))
    for s, n in enumerate(lens):
        for l in range(2):
            g.write_kv(Bd.DFLASH_POOL_TARGET, l, s, 0, *(rng.standard_normal((n, kv_heads, hd)).astype(np.float32) for _ in range(2)))
    tokens = torch.from_numpy(rng.integers(0, 255, (n_seqs, block)).astype(np.int32)).cuda()

    def logits():
        dfl.dflash_verify(g.e, g.batch(), tokens, None, g.logits_t)
        g.e.device_status()
        return g.logits_t.cpu().numpy().copy()

    sound = logits()
    assert np.isfinite(sound).all()
    at, n = (77, 1) if poisoned == "one key" else (0, ctx)
    bad = np.full((n, kv_heads, hd), np.nan, dtype=np.float32)
    g.write_kv(Bd.DFLASH_POOL_TARGET, 0, 0, at, bad, rng.standard_normal(bad.shape).astype(np.float32))
    got = logits()
    assert np.isnan(got[0]).all()
    assert np.array_equal(got[1:], sound[1:])


@pytest.mark.parametrize("dtype,hd,n_seqs,lens", [
    ("f32", 64, 32, (9, 40, 64, 1)),        # 1024 query rows: a workgroup each
    ("f32", 64, 33, (9, 40, 64, 1)),        # 1056: splits, merged in bands of rows
    ("bf16", 96, 19, (9, 90, 64, 1)),       # 608 of 96 dims: splits
    ("bf16", 96, 19, (9, 150, 64, 1)),      # ... a workgroup each from three tiles of keys on
])
def test_plain_attention_on_both_sides_of_its_row_limit(dtype, hd, n_seqs, lens):
    w = tiny_workload(seed=hd + n_seqs, n_layers=2, draft_layers=1, vocab=256, block=8, qk_norm=True, kv_heads=2, dtype=dtype, n_seqs=n_seqs, taps=(0,), d=256,
                      heads=4, hd=hd, ffn=256)
    prompts = [p[:lens[i % 4]] for i, p in enumerate(si.make_prompts(replace(w, ctx_min=max(lens), ctx_max=max(lens))))]
    ls = Lockstep(w, prompts, max_len=max(lens) + 24)
    ls.prefill()
    for i, plan in enumerate((None, [(3 * s + 1) % 8 for s in range(n_seqs)])):
        ls.step(plan=plan, step_idx=i)
    ls.check_cache([0, 1], [0])
    assert ls.stats["low_margin_flips"] <= 0.02 * ls.stats["rows"] + 2
    assert ls.stats["reseeds"] <= 1


@pytest.mark.parametrize("mt,d_expert,n_seqs", [(4, 256, 14), (4, 320, 14), (8, 192, 30), (8, 256, 30)])
def test_routed_items_with_and_without_the_hint_on_their_weights(mt, d_expert, n_seqs, monkeypatch):
    """Experts with one item and with several in the same launches, 256- and 128-row tiles of four bands and both heights of eight: the same bits whether or not
    the weights of single items are read with the non-temporal hint."""
    import torch
    _gpu()
    import paper_2602_06036_amd as dfl
    from tests.gpu_harness import GpuModel
    monkeypatch.setenv("DFLASH_MOE_MT", str(mt))
    w = si.small_moe_workload(n_seqs=n_seqs, ctx_min=12, ctx_max=40, seed=mt + d_expert, n_experts=16, top_k=4, d_expert=d_expert)
    wts, blobs, got = si.make_weights(w), None, []
    tokens = torch.from_numpy(np.random.default_rng(2).integers(0, 255, (n_seqs, w.block_size)).astype(np.int32)).cuda()
    for kept in ("131072", "1"):
        monkeypatch.setenv("DFLASH_MOE_KEPT_KB", kept)
        g = GpuModel(w, *wts, 64, blobs=blobs)
        blobs = g.blobs()
        g.e.moe_stats()
        dfl.dflash_verify(g.e, g.batch(), tokens, None, g.logits_t)
        g.e.device_status()
        got.append(g.logits_t.cpu().numpy().copy())
        launches, reached, bands, items, per_item = g.e.moe_stats()
        assert per_item == mt and reached < items < 2 * reached, (launches, reached, bands, items)
    assert np.isfinite(got[0]).all() and np.array_equal(got[0], got[1])


@pytest.mark.parametrize("fuse", [1, 2])
def test_deferred_norms_use_the_eps_of_their_own_model(fuse, monkeypatch):
    """A target with an eps of 1e-6 and a draft with one of 5e-3, more than ten times the mean square of an embedding row (4e-4), over one band of rows: any norm
    with the other model's would show in the logits."""
    monkeypatch.setenv("DFLASH_FUSE", str(fuse))
    w = tiny_workload(seed=8, n_layers=3, draft_layers=2, vocab=512, block=5, qk_norm=True, kv_heads=2, dtype="bf16", n_seqs=2, taps=(0, 2), ffn=1024)
    w = replace(w, draft=replace(w.draft, rms_eps=5e-3))
    prompts = [p[:n] for p, n in zip(si.make_prompts(replace(w, ctx_min=33, ctx_max=33)), (7, 33))]
    ls = Lockstep(w, prompts, max_len=64)
    ls.prefill()
    for i, plan in enumerate((None, [2, 0])):
        ls.step(plan=plan, step_idx=i)
    ls.check_cache([0, 2], [0, 1])
    assert ls.stats["reseeds"] == 0


def _open_on(e, workspace):
    """The engine's context anew, over another workspace."""
    import ctypes as C
    e.close()
    e.rt.workspace, e.rt.workspace_bytes = workspace.data_ptr(), workspace.numel()
    h = C.c_void_p()
    assert e.l.dflash_create(C.byref(e.td), e.target_blob.data_ptr(), C.byref(e.dd), e.draft_blob.data_ptr(), C.byref(e.rt), C.byref(h)) == 0
    e.ctx = h


@pytest.mark.parametrize("block", [16, 5])
def test_no_call_relies_on_what_the_workspace_held_before(block):
    """Contexts of one, two and eight sequences of the same models, each by itself and then step by step in turn over one workspace that is
    filled with ones (NaN, counters far from zero) behind the status block before every prefill, draft and verification: the same bits.  One and two
    sequences (of the five-row block) take the launches whose last workgroup finishes the sums."""
    import torch
    _gpu()
    import paper_2602_06036_amd as dfl
    w = tiny_workload(seed=3, n_layers=3, draft_layers=2, vocab=512, block=block, qk_norm=True, kv_heads=2, dtype="bf16", n_seqs=8, taps=(0, 2), ffn=1024)
    from tests.gpu_harness import GpuModel, _with_seqs
    wt, wd = si.make_weights(w)
    prompts = [p[:n] for p, n in zip(si.make_prompts(replace(w, ctx_min=40, ctx_max=40)), (9, 40, 17, 33, 5, 16, 21, 38))]
    models, blobs = [], None
    for n in (1, 2, 8):
        models.append(GpuModel(_with_seqs(w, n), wt, wd, 40 + 6 * block, n_seqs=n, blobs=blobs))
        blobs = blobs or models[0].blobs()

    def turns(models, before):
        out = [[] for _ in models]
        for g, o, n in zip(models, out, (1, 2, 8)):
            g.host_lens[:] = 0
            g.seq_lens.zero_()
            before()
            o.append(g.prefill_entry(prompts[:n]))
        for step in range(3):
            for g, o in zip(models, out):
                b = g.batch()
                before()
                dfl.dflash_draft_block(g.e, b, g.draft_tokens, 0.0, None, g.logits_d)
                before()
                dfl.dflash_verify(g.e, b, g.draft_tokens, g.tgt_argmax, g.logits_t)
                dfl.dflash_accept(g.e, b, g.draft_tokens, g.tgt_argmax, g.accept_len, g.out_tokens)
                dfl.dflash_kv_commit(g.e, b, g.accept_len, g.out_tokens)
                o.append((g.logits_d.cpu().numpy().copy(), g.logits_t.cpu().numpy().copy(), g.out_tokens.cpu().numpy().copy()))
                g.e.device_status()
                g.host_lens = g.seq_lens.cpu().numpy().astype(np.int64)
        return out

    alone = turns(models, lambda: None)
    assert all(np.isfinite(x).all() for o in alone for st in o[1:] for x in st)
    shared = torch.zeros(max(g.e.rt.workspace_bytes for g in models), dtype=torch.uint8, device="cuda:0")
    for g in models:
        _open_on(g.e, shared)
    for got, want in zip(turns(models, lambda: shared[256:].fill_(255)), alone):
        assert np.array_equal(got[0], want[0])
        for a, b in zip(got[1:], want[1:]):
            assert all(np.array_equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("vocab,rows,tiles", STREAM_HEADS)
def test_streaming_heads_with_eight_six_and_four_weight_tiles(vocab, rows, tiles):
    """LM heads of 16, 32 and 48 rows, high enough for the weight tiles per wavefront that a whole vocabulary takes, with their argmax,
    Gumbel-max and softmax-statistics epilogues."""
    n_seqs = rows // 16
    w = tiny_workload(seed=tiles, n_layers=2, draft_layers=1, vocab=vocab, block=16, qk_norm=True, kv_heads=2, dtype="bf16", n_seqs=n_seqs,
                      taps=(0, 1), d=256, heads=4, hd=64, ffn=512)
    prompts = [p[:9 + 4 * i] for i, p in enumerate(si.make_prompts(replace(w, ctx_min=20, ctx_max=20)))]
    ls = Lockstep(w, prompts, max_len=20 + 4 * 16)
    ls.prefill()
    ls.g.e.gemm_counts()
    ls.step(plan=[(5 * s + 3) % 16 for s in range(n_seqs)], step_idx=0)
    ls.step(temperature=0.8, step_idx=1, key=11)
    assert ls.g.e.gemm_counts()[0] > 0
    assert ls.stats["low_margin_flips"] <= 0.02 * ls.stats["rows"] + 2
    assert ls.stats["reseeds"] <= 1


@pytest.mark.parametrize("n_seqs,lens,block", [
    (1, (8500,), 16),           # 33 pairs a wavefront and more: the page ids' second set
    (2, (2300, 33), 10),        # 40 query rows (the last block of 16 half empty), one chunk with a single pair
    (3, (257, 511, 64), 16),    # chunk ends on and off a page, wavefronts without a pair
])
def test_key_split_attention_edges(n_seqs, lens, block, monkeypatch):
    """The key-split attention kernel over chunks from one page pair to more than 32 pairs per wavefront (one split per
    sequence), against the oracle."""
    monkeypatch.setenv("DFLASH_ATTN_WIDE_MIN_CHUNK", "64")
    monkeypatch.setenv("DFLASH_ATTN_TARGET_WGS", "1")
    w = tiny_workload(seed=17 + block, n_layers=2, draft_layers=1, vocab=512, block=block, qk_norm=True, kv_heads=1, dtype="bf16",
                      n_seqs=n_seqs, taps=(0, 1), d=256, heads=4, hd=128, ffn=512)
    top = max(lens)
    prompts = [p[:n] for p, n in zip(si.make_prompts(replace(w, ctx_min=top, ctx_max=top)), lens)]
    ls = Lockstep(w, prompts, max_len=top + 4 * 16)
    ls.prefill()
    for i, plan in enumerate([[3] * n_seqs, None]):
        ls.step(plan=plan, step_idx=i)
    assert ls.stats["low_margin_flips"] <= 0.02 * ls.stats["rows"] + 2
    assert ls.stats["reseeds"] <= 1


@pytest.mark.parametrize("dtype,n_seqs", [("f32", 2), ("bf16", 1), ("bf16", 3), ("bf16", 6)])
def test_logits_reach_buffers_of_any_alignment(dtype, n_seqs):
    """logits_out is written by the LM head's epilogue (fp32, few-row, streaming and LDS-staged kernels) where 16-byte stores
    reach it and copied otherwise: the same values for an aligned buffer, one that is 4 bytes off, and in the workspace."""
    import torch
    from paper_2602_06036_amd import binding as Bd
    GpuModel = _gpu()
    w = tiny_workload(seed=3, n_layers=2, draft_layers=1, vocab=512, block=16, qk_norm=True, kv_heads=2, dtype=dtype, n_seqs=n_seqs,
                      taps=(0,), d=256, heads=4, hd=64, ffn=512)
    wt, wd = si.make_weights(w, 4)
    g = GpuModel(w, wt, wd, 80, n_seqs=n_seqs)
    prompts = si.make_prompts(replace(w, ctx_min=20, ctx_max=40))
    g.prefill(prompts)
    n = n_seqs * 16 * 512
    flat = torch.zeros(2 * n + 4, dtype=torch.float32, device=g.dev)
    for fn, toks in ((Bd.dflash_draft_block, g.draft_tokens), (Bd.dflash_verify, g.draft_tokens)):
        outs = []
        for shift in (0, 1):
            buf = flat[shift:shift + n].view(n_seqs, 16, 512).zero_()
            if fn is Bd.dflash_draft_block:
                fn(g.e, g.batch(), toks, logits_out=buf)
            else:
                fn(g.e, g.batch(), toks, g.tgt_argmax, buf)
            outs.append(buf.clone())
        assert torch.isfinite(outs[0]).all() and outs[0].abs().max() > 0
        assert torch.equal(outs[0], outs[1])
    g.e.close()


@pytest.mark.parametrize("dtype,n_seqs", [("f32", 1), ("bf16", 1), ("bf16", 6)])
def test_logits_reach_host_memory(dtype, n_seqs):
    """A buffer that a copy reaches and a kernel's stores may not: host memory, pinned and pageable, through the C calls."""
    import ctypes as C
    import torch
    from paper_2602_06036_amd import binding as Bd
    GpuModel = _gpu()
    w = tiny_workload(seed=3, n_layers=2, draft_layers=1, vocab=512, block=16, qk_norm=True, kv_heads=2, dtype=dtype, n_seqs=n_seqs,
                      taps=(0,), d=256, heads=4, hd=64, ffn=512)
    wt, wd = si.make_weights(w, 4)
    g = GpuModel(w, wt, wd, 80, n_seqs=n_seqs)
    g.prefill(si.make_prompts(replace(w, ctx_min=20, ctx_max=40)))
    shape = (n_seqs, 16, 512)
    st, b, toks = torch.cuda.current_stream().cuda_stream, g.batch(), g.draft_tokens
    pinned, pageable = torch.empty(shape, pin_memory=True), torch.empty(shape)
    for call in (lambda p: g.e.l.dflash_draft_block(g.e.ctx, C.byref(b), 0.0, None, toks.data_ptr(), p, st),
                 lambda p: g.e.l.dflash_verify(g.e.ctx, C.byref(b), toks.data_ptr(), g.tgt_argmax.data_ptr(), p, st)):
        on_device = torch.zeros(shape, device=g.dev)
        assert call(on_device.data_ptr()) == Bd.DFLASH_OK
        for host in (pinned, pageable):
            host.zero_()
            assert call(host.data_ptr()) == Bd.DFLASH_OK
            torch.cuda.synchronize()
            assert on_device.abs().max() > 0 and torch.equal(host, on_device.cpu())
    g.e.close()


@pytest.mark.parametrize("dtype,n_seqs", [("f32", 1), ("bf16", 1), ("bf16", 6)])
def test_logits_under_capture(dtype, n_seqs):
    """The caller's logits of a captured verification, replayed with eager work in between: the eager call's, each time."""
    import torch
    from paper_2602_06036_amd import binding as Bd
    GpuModel = _gpu()
    w = tiny_workload(seed=4, n_layers=2, draft_layers=1, vocab=512, block=16, qk_norm=True, kv_heads=2, dtype=dtype, n_seqs=n_seqs,
                      taps=(0,), d=256, heads=4, hd=64, ffn=512)
    wt, wd = si.make_weights(w, 4)
    g = GpuModel(w, wt, wd, 80, n_seqs=n_seqs)
    g.prefill(si.make_prompts(replace(w, ctx_min=20, ctx_max=40)))
    b, want = g.batch(), torch.zeros((n_seqs, 16, 512), device=g.dev)
    Bd.dflash_verify(g.e, b, g.draft_tokens, g.tgt_argmax, want)
    out, graph, side = torch.zeros_like(want), torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        Bd.dflash_verify(g.e, b, g.draft_tokens, g.tgt_argmax, out)
    for _ in range(3):
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        Bd.dflash_draft_block(g.e, b, torch.zeros_like(g.draft_tokens))
    g.e.close()


@pytest.mark.parametrize("experts,top_k,n_seqs", [(16, 4, 1), (80, 8, 2), (48, 6, 5), (256, 16, 4), (256, 15, 6)])
def test_equal_router_logits_go_to_the_lowest_expert(experts, top_k, n_seqs):
    """Router rows equal in groups of four give four bitwise equal logits each: every row's choices are whole groups in
    ascending order (the last one cut off where four does not divide top_k), expert counts below, between and at the
    multiples of 64, choices made in the routing kernel (up to 64 rows) and before it."""
    import torch
    from paper_2602_06036_amd import binding as Bd
    GpuModel = _gpu()
    w = si.small_moe_workload(n_seqs=n_seqs, ctx_min=12, ctx_max=20, seed=5, n_experts=experts, top_k=top_k, d_expert=64)
    wt, wd = si.make_weights(w, 8)
    for l in range(w.target.n_layers):
        wt.t[f"L{l}.wr"] = np.ascontiguousarray(np.repeat(wt.t[f"L{l}.wr"][::4], 4, axis=0))
    g = GpuModel(w, wt, wd, 64, n_seqs=n_seqs)
    g.prefill(si.make_prompts(w))
    g.draft_tokens.copy_(torch.arange(n_seqs * 16, device=g.dev).view(n_seqs, 16) * 37 % 4096)
    trace = g.e.moe_trace()
    Bd.dflash_verify(g.e, g.batch(), g.draft_tokens, g.tgt_argmax)
    got = trace.cpu().numpy()[:, : n_seqs * 16].reshape(-1, top_k)
    assert (got >= 0).all() and (got < experts).all()
    assert (got % 4 == np.arange(top_k) % 4).all()
    first = got[:, ::4]
    assert (np.repeat(first, 4, axis=1)[:, :top_k] // 4 == got // 4).all()
    assert all(len(set(r)) == len(r) for r in first)
    assert len(np.unique(first)) > top_k // 4 + 1
    g.e.close()


@pytest.mark.parametrize("d_expert,d_model,seed", [
    (192, 640, 202),      # gate/up 24 bands, down 40: 128-row tiles
    (832, 512, 201),      # gate/up 104 bands: 256-row tiles, the last one half empty; down 32
    (64, 1792, 200),      # gate/up 8 bands: one 128-row tile; down 112: 256-row tiles, the last one half empty
])
def test_four_band_expert_items_of_odd_heights(d_expert, d_model, seed):
    """Routed-expert items of four bands (160 rows, 4 of 16 experts) on matrices that 256-row tiles do not divide."""
    w = si.small_moe_workload(n_seqs=10, ctx_min=12, ctx_max=30, seed=seed, n_experts=16, top_k=4, d_expert=d_expert)
    w = replace(w, target=replace(w.target, d_model=d_model, n_layers=2), draft=replace(w.draft, d_model=d_model, n_layers=1))
    ls = Lockstep(w, si.make_prompts(w), max_len=30 + 3 * 16)
    ls.prefill()
    assert min(ls.route_gaps) > ROUTE_CLEAR
    ls.g.e.moe_stats()
    for i, plan in enumerate([None, list(np.arange(10) % 16)]):
        ls.step(plan=plan, step_idx=i)
    assert ls.g.e.moe_stats()[4] == 4
    ls.check_cache([0, 1], [0])
    assert ls.stats["route_ties"] <= 2 and ls.stats["reseeds"] <= 1 + ls.stats["route_ties"]
