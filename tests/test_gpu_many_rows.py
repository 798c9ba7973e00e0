"""The kernels of launches with many rows give bitwise the rows of the few-row
kernels (whose values the oracle tests judge): teacher-forced logits of a
ragged batch against each sentence alone (its first positions in at most 16
rows, and all of them), at the edges of row tiles, key chunks and column tiles;
decodes that reuse a context's captured iterations."""
import dataclasses

import numpy as np
import pytest

from paper_2305_10427_amd import configs as C, pdec, synth

pytestmark = pytest.mark.gpu


def cfg_of(dtype, d, heads, d_ff, vocab=333, pre_ln=True):
    return dataclasses.replace(C.TINY, name=f"rows_{dtype}_{d}_{heads}", n_enc=1, n_dec=2, d_model=d, n_heads=heads,
                               d_ff=d_ff, vocab=vocab, pre_ln=pre_ln, act_gelu=pre_ln, dtype=dtype)


def logits(ctx, src, lens, tgt):
    import torch
    ctx.encode(torch.from_numpy(src).cuda(), lens)
    return ctx.debug_logits(torch.from_numpy(tgt)).cpu().numpy()


def compare(cfg, B, n, T, seed=1, plant=None):
    """Logits of B sentences of T positions against each sentence alone: its first positions in at most 16 rows, and
    all of them in T rows (attention row by row: T * heads < 2048), so every row tile and key chunk is compared."""
    assert T * cfg.n_heads < 2048
    w = synth.make_weights(cfg, seed=seed, bias_std=0.3, ln_std=0.2)
    if plant is not None:                       # a token whose embedding is not finite
        w.values["emb"][plant] = np.nan
        if w.bf16_bits is not None:
            w.bf16_bits["emb"][plant] = 0x7fc0
    gm = pdec.Model(cfg, w)
    g = np.random.default_rng(seed)
    lens = [int(x) for x in np.linspace(1, n, B).round()]
    src = g.integers(4, cfg.vocab - 1, (B, n)).astype(np.int32)
    tgt = g.integers(4, cfg.vocab - 1, (B, T)).astype(np.int32)
    tgt[:, 0] = C.BOS_ID
    if plant is not None:
        tgt[:, T // 2] = plant                  # positions before it must not see it
    got = logits(pdec.Context(gm, B, n, T), src, lens, tgt)
    one = pdec.Context(gm, 1, n, T)
    t = min(T, 16)
    for b in range(0, B, max(1, B // 7)):
        want = logits(one, src[b:b + 1, :lens[b]], lens[b:b + 1], tgt[b:b + 1, :t])
        np.testing.assert_array_equal(got[b, :t], want[0])
        if T > t:
            np.testing.assert_array_equal(got[b], logits(one, src[b:b + 1, :lens[b]], lens[b:b + 1], tgt[b:b + 1])[0])
    if plant is not None:
        assert np.isfinite(got[:, :T // 2, :plant]).all() and not np.isfinite(got[:, T // 2]).any()
    return got


@pytest.mark.parametrize("dtype,d,heads,d_ff", [("bf16", 256, 8, 512), ("bf16", 256, 4, 2048), ("bf16", 256, 2, 256),
                                                ("f32", 128, 4, 256), ("f32", 256, 4, 2048), ("f32", 256, 2, 256),
                                                ("f32", 64, 4, 256)])
@pytest.mark.parametrize("B,n,T", [(2, 16, 17), (35, 65, 31), (70, 130, 16), (33, 20, 33)])
def test_teacher_forced_rows_are_bitwise_those_of_few_rows(dtype, d, heads, d_ff, B, n, T):
    compare(cfg_of(dtype, d, heads, d_ff), B, n, T)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_a_later_rows_nan_stays_out_of_earlier_rows(dtype):
    cfg = cfg_of(dtype, 128, 2, 256)
    compare(cfg, 45, 20, 24, plant=cfg.vocab - 1)


@pytest.mark.parametrize("dtype,heads", [("bf16", 4), ("bf16", 8), ("f32", 2)])
@pytest.mark.parametrize("mode,block", [("gs_jacobi", 8), ("gs_jacobi", 19), ("jacobi", 1)])
def test_blocks_across_row_tiles_equal_single_decodes(dtype, heads, mode, block):
    """Blocks whose rows straddle 16-row tiles (several sentences a tile, unequal lengths)."""
    import torch
    cfg = cfg_of(dtype, 256, heads, 512, pre_ln=False)
    gm = pdec.Model(cfg, synth.make_weights(cfg, seed=4, bias_std=0.5, ln_std=0.3))
    B, n = 70, 70
    g = np.random.default_rng(2)
    src = g.integers(4, cfg.vocab, (B, n)).astype(np.int32)
    lens = [70, 3, 66, 20, 64, 1, 41] * 10
    ms = [67, 21, 9, 40, 5, 64, 33] * 10
    ctx, one = pdec.Context(gm, B, n, 80), pdec.Context(gm, 1, n, 80)
    ctx.encode(torch.from_numpy(src).cuda(), lens)
    ids, ln, k, fl = [t.cpu().numpy() for t in ctx.decode(mode, ms, block=block)]
    for b in range(0, B, 11):
        one.encode(torch.from_numpy(src[b:b + 1, :lens[b]]).cuda(), lens[b:b + 1])
        i1, l1, k1, f1 = [t.cpu().numpy() for t in one.decode("gs_jacobi", ms[b:b + 1], block=min(block, 7))]
        assert ln[b] == l1[0] and fl[b] == f1[0]
        np.testing.assert_array_equal(ids[b, :ln[b]], i1[0, :l1[0]])


def test_more_sentences_than_a_grid_dimension_holds():
    """70,000 sentences of eight rows (the attention's launches take 65,535): logits and a decode of the first, the
    last and the sentences where the launches meet equal each sentence's own."""
    import torch
    cfg = dataclasses.replace(cfg_of("f32", 64, 2, 64, vocab=40), n_dec=1)
    gm = pdec.Model(cfg, synth.make_weights(cfg, seed=8, bias_std=0.1, ln_std=0.1))
    B, n = 70000, 8
    g = np.random.default_rng(1)
    src = g.integers(4, cfg.vocab, (B, n)).astype(np.int32)
    tgt = g.integers(4, cfg.vocab, (B, n)).astype(np.int32)
    lens = [1 + i % n for i in range(B)]
    ctx, one = pdec.Context(gm, B, n, n), pdec.Context(gm, 1, n, n)
    got = logits(ctx, src, lens, tgt)
    out = [t.cpu().numpy() for t in ctx.decode("gs_jacobi", [n] * B, block=n)]
    for b in (0, 65534, 65535, 65536, B - 1):
        np.testing.assert_array_equal(got[b], logits(one, src[b:b + 1, :lens[b]], lens[b:b + 1], tgt[b:b + 1])[0])
        for x, y in zip(out, one.decode("gs_jacobi", [n], block=n)):
            np.testing.assert_array_equal(x[b], y.cpu().numpy()[0])


def test_more_vocabulary_tiles_than_a_grid_dimension_holds():
    """296,000 rows of V = 58,101: 4.2 million 32 x 128 tiles, more than the 2^22 of the grid's first dimension."""
    import torch
    cfg = dataclasses.replace(cfg_of("f32", 32, 1, 32, vocab=58101), n_dec=1)
    gm = pdec.Model(cfg, synth.make_weights(cfg, seed=8, bias_std=0.1, ln_std=0.1))
    B, n, m = 18500, 3, 16
    src = np.random.default_rng(1).integers(4, cfg.vocab, (B, n)).astype(np.int32)
    ctx, one = pdec.Context(gm, B, n, m), pdec.Context(gm, 1, n, m)
    ctx.encode(torch.from_numpy(src).cuda(), [n] * B)
    out = [t.cpu().numpy() for t in ctx.decode("jacobi", [m] * B, max_iters=2)]
    for b in list(range(0, B, 1999)) + [B - 1]:
        one.encode(torch.from_numpy(src[b:b + 1]).cuda(), [n])
        for x, y in zip(out, one.decode("jacobi", [m], max_iters=2)):
            np.testing.assert_array_equal(x[b], y.cpu().numpy()[0])


def launch_bound(rows, full):
    """Rows an iteration of `rows` rows is launched (and its graph captured) for."""
    b = 1
    while b < min(rows, full):
        b *= 2
    return min(b, full)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("mode,block,short,long", [("jacobi", 1, [40] + [20] * 7, [60] + [20] * 7),
                                                   ("jacobi", 1, [70] + [30] * 15, [100] + [30] * 15),
                                                   ("gs_jacobi", 32, [16] + [14] * 15, [32] + [14] * 15),
                                                   ("hybrid", 32, [16] + [14] * 15, [64] + [14] * 15)])
def test_a_context_decodes_longer_targets_after_shorter_ones(monkeypatch, dtype, mode, block, short, long):
    """A graph captured for short blocks (16-row attention tiles of 8 heads) must not serve longer blocks of the
    same launch bound: what a context decodes, and its trace (whose logits show rows that the argmax hides), equal
    a fresh context's, with graphs and without."""
    import torch
    cfg = cfg_of(dtype, 256, 8, 512, pre_ln=False)
    gm = pdec.Model(cfg, synth.make_weights(cfg, seed=6, eos_bias=-128.0))     # whole targets, dozens of iterations
    B, n = len(short), 20
    rows = [[min(x, block if mode != "jacobi" else x) for x in ms] for ms in (short, long)]
    bounds = [launch_bound(sum(r), B * max(r)) for r in rows]
    assert bounds[0] == bounds[1] and bounds[0] * cfg.n_heads >= 2048
    src = torch.from_numpy(np.random.default_rng(3).integers(4, cfg.vocab, (B, n)).astype(np.int32)).cuda()

    def context():
        c = pdec.Context(gm, B, n, 100)
        c.encode(src, [n] * B)
        c.set_trace(200000, B * 100)
        return c

    def decode(c, ms):
        before = c.trace()[1]
        out = [t.cpu().numpy() for t in c.decode(mode, ms, block=block)]
        torch.cuda.synchronize()
        return out + [c.trace()[0][before:]]

    kept = context()
    for ms in (short, long, short):
        got, fresh = decode(kept, ms), decode(context(), ms)
        monkeypatch.setenv("PDEC_GRAPHS", "0")
        direct = decode(context(), ms)
        monkeypatch.delenv("PDEC_GRAPHS")
        assert direct[2].max() >= 16 and len(direct[4]) < 60000
        for g, f, w in zip(got, fresh, direct):
            np.testing.assert_array_equal(g, w)
            np.testing.assert_array_equal(f, w)


@pytest.mark.parametrize("dtype,d,heads,vocab", [("bf16", 640, 10, 1111), ("bf16", 96, 6, 1111), ("f32", 96, 6, 1111)])
@pytest.mark.parametrize("B,T", [(1, 17), (2, 32), (5, 13), (4, 75), (4, 113), (9, 57), (40, 20)])
def test_vocabulary_rows_are_bitwise_those_of_few_rows(dtype, d, heads, vocab, B, T):
    """Row counts around each change of the projection's tile (16, 32, 64, 160, 448, 512 rows), a ragged last column tile."""
    compare(cfg_of(dtype, d, heads, 128, vocab=vocab), B, 7, T)


@pytest.mark.parametrize("dtype,d,heads,vocab,B,T", [
    ("f32", 64, 4, 1000, 1, 33), ("f32", 64, 4, 1000, 7, 33),            # LayerNorm in the product; 16 x 64 tiles
    ("f32", 96, 6, 20011, 5, 30), ("f32", 288, 18, 20011, 34, 60),       # 32 x 128; staged 128 x 256
    ("bf16", 96, 6, 20011, 2, 40), ("bf16", 96, 6, 58001, 2, 32),        # 32 x 128; 32 x 256
    ("bf16", 96, 6, 20011, 10, 30), ("bf16", 96, 6, 20011, 10, 80),      # staged 128 x 128; 256 x 256
    ("bf16", 640, 10, 20011, 3, 16), ("bf16", 640, 10, 20011, 5, 26),    # 32 x 128; staged 128 x 128
    ("bf16", 640, 10, 58001, 7, 64), ("bf16", 544, 17, 131200, 3, 21)])  # staged 128 x 256; 64 x 256
def test_each_vocabulary_tile_gives_the_rows_of_few_rows(dtype, d, heads, vocab, B, T):
    """Stored logits on every tile that the vocabulary's size, the width and the rows select, ragged columns and rows."""
    compare(dataclasses.replace(cfg_of(dtype, d, heads, 64, vocab=vocab), n_dec=1), B, 5, T)


@pytest.mark.parametrize("dtype,d,heads,vocab,B,m", [
    ("f32", 128, 2, 20011, 9, 28), ("f32", 288, 18, 20011, 34, 60),      # 32 x 128; staged 128 x 256
    ("bf16", 128, 2, 20011, 5, 13), ("bf16", 128, 2, 20011, 9, 16),      # 32 x 128; 32 x 256
    ("bf16", 128, 2, 20011, 9, 28), ("bf16", 640, 10, 20011, 9, 60),     # staged 128 x 128; 128 x 256
    ("bf16", 544, 17, 131200, 3, 13)])                                   # staged 64 x 256
def test_argmax_of_planted_logits_on_each_vocabulary_tile(dtype, d, heads, vocab, B, m):
    cfg = dataclasses.replace(cfg_of(dtype, d, heads, 64, vocab=vocab), n_dec=1, logit_scale=0.0)
    v = vocab
    planted(cfg, B, m, [(2.5, (v - 300, v - 299, v - 1), None), (0.0, (300, 5555, v - 81), None), (1.0, (v - 1,), None),
                        (0.5, (513,), v - 20)])


@pytest.mark.parametrize("dtype,d,heads", [("bf16", 640, 10), ("bf16", 128, 2), ("f32", 128, 2)])
@pytest.mark.parametrize("B,m", [(1, 17), (3, 16), (5, 13), (9, 28), (9, 60)])
def test_argmax_of_planted_logits(dtype, d, heads, B, m):
    """Logits that are the output bias alone (scale 0): the largest, the lowest index among equals (at zero too,
    where the order of +0 and -0 must not matter), and the flag of a non-finite one."""
    cfg = dataclasses.replace(cfg_of(dtype, d, heads, 128, vocab=1111), logit_scale=0.0)
    planted(cfg, B, m, [(2.5, (700, 701, 1110), None), (0.0, (300, 555, 1030), None), (1.0, (1110,), None),
                        (0.5, (513,), 20)])


def planted(cfg, B, m, cases):
    import torch
    w = synth.make_weights(cfg, seed=3)
    for best, at, bad in cases:
        bias = np.full(cfg.vocab, -1.0, np.float32)
        bias[list(at)] = best
        if bad is not None:
            bias[bad] = np.nan
        w.values["out_bias"] = bias
        if w.bf16_bits is not None:
            w.bf16_bits["out_bias"] = (bias.view(np.uint32) >> 16).astype(np.uint16)
        ctx = pdec.Context(pdec.Model(cfg, w), B, 5, m)
        ctx.encode(torch.full((B, 5), 9, dtype=torch.int32, device="cuda"), [5] * B)
        ids, ln, k, fl = [t.cpu().numpy() for t in ctx.decode("jacobi", [m] * B)]
        assert (ids == at[0]).all() and (ln == m).all() and (k == min(2, m)).all()
        assert ((fl & pdec.FLAG_NONFINITE != 0) == (bad is not None)).all()


@pytest.mark.parametrize("d,heads,d_ff,B,T", [(512, 8, 2048, 48, 65), (544, 17, 2080, 50, 63)])
def test_staged_products_are_bitwise_those_of_few_rows(d, heads, d_ff, B, T):
    """Enough rows for every layer product to run on staged tiles: ragged row and column tiles, K of four and eight ranges."""
    compare(dataclasses.replace(cfg_of("bf16", d, heads, d_ff), n_dec=1), B, 64, T)


def test_an_ffn_wider_than_a_tiles_offsets():
    """d_ff of 2^22, whose rows a many-row tile cannot address: the product goes to the kernel that can."""
    cfg = dataclasses.replace(cfg_of("bf16", 32, 1, 64), n_dec=1)
    small, wide = synth.make_weights(cfg, seed=2, bias_std=0.1), dataclasses.replace(cfg, d_ff=1 << 22)
    bits = {n: np.resize(small.bf16_bits[n], s) for n, s in C.param_shapes(wide)}
    shapes = {n: np.broadcast_to(np.float32(0), s) for n, s in C.param_shapes(wide)}
    gm = pdec.Model(wide, synth.Weights(wide, shapes, bits))
    g = np.random.default_rng(5)
    B, T = 9, 16
    src, tgt = (g.integers(4, cfg.vocab, (B, x)).astype(np.int32) for x in (3, T))
    got = logits(pdec.Context(gm, B, 3, T), src, [3] * B, tgt)
    one = pdec.Context(gm, 1, 3, T)
    assert np.isfinite(got).all()
    for b in (0, B - 1):
        np.testing.assert_array_equal(got[b], logits(one, src[b:b + 1], [3], tgt[b:b + 1])[0])


@pytest.mark.parametrize("pre_ln", [True, False])
@pytest.mark.parametrize("d,d_ff,B,T", [(128, 2048, 3, 43), (128, 512, 3, 43), (64, 96, 9, 29), (128, 2048, 23, 32),
                                        (128, 512, 24, 32)])
def test_float32_products_of_few_tiles_are_bitwise_those_of_few_rows(pre_ln, d, d_ff, B, T):
    """More rows than the streaming products take, fewer than 96 tiles of 32 x 32 (the last two: 92 and 96 for N = 128)."""
    compare(cfg_of("f32", d, 4, d_ff, pre_ln=pre_ln), B, 20, T)


@pytest.mark.parametrize("dtype,d,heads,d_ff", [("bf16", 256, 4, 2048), ("f32", 128, 4, 4096), ("bf16", 128, 2, 512),
                                                ("f32", 256, 4, 1024), ("bf16", 1024, 16, 4096)])
@pytest.mark.parametrize("T", [1, 2, 7, 8, 9, 16])
def test_few_rows_are_bitwise_those_of_a_longer_call(dtype, d, heads, d_ff, T):
    """Launches of 1 to 8 rows (input rows through LDS) and of 9 and more (feed order), each whole K range in flight."""
    compare_prefix(cfg_of(dtype, d, heads, d_ff), T)


def compare_prefix(cfg, T):
    gm = pdec.Model(cfg, synth.make_weights(cfg, seed=7, bias_std=0.3, ln_std=0.2))
    g = np.random.default_rng(T)
    src = g.integers(4, cfg.vocab, (1, 5)).astype(np.int32)
    tgt = g.integers(4, cfg.vocab, (1, 40)).astype(np.int32)
    ctx = pdec.Context(gm, 1, 5, 40)
    want = logits(ctx, src, [5], tgt)
    np.testing.assert_array_equal(logits(ctx, src, [5], tgt[:, :T]), want[:, :T])
