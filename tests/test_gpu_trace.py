"""Decoding trace (the data of DDGviz, Section 3.5 and Figure 3) through the
C ABI, against the oracle's argmax records.

For every evaluated row the oracle keeps (position, token, top1, lse) in
evaluation order; its iterates give the iteration that produced each block.
The GPU trace must list the same rows in the same order, with the same token
and iteration, and top1 / lse within the measured logit error bound
(EPS * max|logit|).  A token that differs ends the comparison there only if
the oracle's logit of the GPU's token is within the near-tie threshold of its
top-1 (tests/parity.py); past it both trajectories are valid but may differ."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2305_10427_amd import configs as C, pdec, synth
from tests.parity import EPS, gpu_decode_batch, judge_row, oracle_rows

pytestmark = pytest.mark.gpu

TINY = C.TINY
CHAIN = dataclasses.replace(C.TINY, name="chain", logit_scale=-3.0)
SMALL_PRE_BF16 = dataclasses.replace(C.TINY, name="small_pre", pre_ln=True, act_gelu=True, dtype=C.BF16)
MODES = [("ar", 1), ("jacobi", 0), ("gs_jacobi", 3), ("hybrid", 4)]


def say(*a):
    print(*a, flush=True)


def build(cfg, seed=0, max_batch=4, max_src=32, max_tgt=32, **wkw):
    w = synth.make_weights(cfg, seed=seed, **wkw)
    gm = pdec.Model(cfg, w)
    return gm, pdec.Context(gm, max_batch, max_src, max_tgt), oracle.Model(cfg, w.values)


def sources(vocab, count, n=16, seed=1):
    g = np.random.default_rng(seed)
    return [g.integers(4, vocab, n).astype(np.int32) for _ in range(count)]


def compare(got, want: oracle.Result, mode, m, M, enc, dtype, sentence=0):
    """Compares the GPU records with the oracle's evaluated rows in order
    (iteration, sentence, position and token exactly; top-1 logit and
    log-sum-exp within EPS * max|logit|) until the end, or until a token
    differs where the oracle's logit of the GPU's token is within the
    near-tie threshold of its top-1 (past that point both trajectories are
    valid but may differ; any other difference fails).  Returns the rows
    compared."""
    rows = oracle_rows(want, mode, m)
    assert len(rows) == len(want.records)
    eps = EPS[dtype]
    n = 0
    for g, (it, pos, tok, draft), rec in zip(got, rows, want.records):
        assert (int(g["iteration"]), int(g["sentence"]), int(g["position"])) == (it, sentence, pos), (g, it, pos)
        if int(g["token"]) != tok:
            lab = judge_row(M, enc, draft, pos, int(g["token"]), dtype, "trace")
            assert not lab.startswith("FAIL"), lab
            return n
        assert abs(float(g["top1"]) - rec.top1) <= eps * rec.linf, (g, rec.top1)
        assert abs(float(g["lse"]) - rec.lse) <= eps * rec.linf, (g, rec.lse)
        n += 1
    assert len(got) == len(want.records)
    return n


@pytest.mark.parametrize("cfg,wkw", [(TINY, {}), (CHAIN, dict(bias_std=0.5, ln_std=0.3)),
                                     (SMALL_PRE_BF16, dict(bias_std=0.3, ln_std=0.2))],
                         ids=["tiny", "chain", "small_pre_bf16"])
def test_trace_matches_oracle_records(cfg, wkw):
    gm, ctx, M = build(cfg, seed=3, **wkw)
    rows = compared = 0
    for src in sources(cfg.vocab, 2, seed=21):
        enc = M.encode(src)
        for mode, b in MODES:
            for m in (9, 16):
                say(f"case trace cfg={cfg.name} mode={mode} b={b} m={m}")
                want = oracle.decode(M, enc, m, mode, b)
                ctx.set_trace(4096, m)
                ctx.set_timing(False)                 # resets the row counter
                g = gpu_decode_batch(ctx, [src], [m], mode, b)[0]
                rec, count = ctx.trace()
                assert count == ctx.rows_processed()
                assert count == len(rec)
                rows += len(want.records)
                compared += compare(rec, want, mode, m, M, enc, cfg.dtype)
    say(f"case trace cfg={cfg.name}: {compared} of {rows} rows compared")
    assert compared >= 0.9 * rows
    ctx.set_trace(0, 0)


@pytest.mark.parametrize("cfg,wkw", [(CHAIN, dict(bias_std=0.5, ln_std=0.3)),
                                     (SMALL_PRE_BF16, dict(bias_std=0.3, ln_std=0.2))],
                         ids=["chain_f32", "small_pre_bf16"])
def test_batched_trace_matches_oracle_per_sentence(cfg, wkw):
    """Iterations of more than one 16-row tile: the many-row argmax also returns
    the log-sum-exp partials; each sentence's records equal the oracle's."""
    gm, ctx, M = build(cfg, seed=7, **wkw)
    srcs = sources(cfg.vocab, 4, seed=24)
    ms = [24, 19, 24, 22]
    rows = compared = 0
    for B, mode, b in [(1, "jacobi", 0), (4, "jacobi", 0), (4, "gs_jacobi", 8), (4, "hybrid", 6)]:
        say(f"case trace rows cfg={cfg.name} B={B} mode={mode} b={b}")
        ctx.set_trace(16384, B * 24)
        gpu_decode_batch(ctx, srcs[:B], ms[:B], mode, b)
        rec, count = ctx.trace()
        assert count == len(rec)
        for s in range(B):
            enc = M.encode(srcs[s])
            want = oracle.decode(M, enc, ms[s], mode, b)
            rows += len(want.records)
            compared += compare(rec[rec["sentence"] == s], want, mode, ms[s], M, enc, cfg.dtype, sentence=s)
    say(f"case trace rows cfg={cfg.name}: {compared} of {rows} rows compared")
    assert compared >= 0.9 * rows
    ctx.set_trace(0, 0)


def test_trace_changes_no_result_and_batches_agree():
    """Traced decodes return the untraced ids, k and flags; the records of a
    batch, sentence by sentence, equal those of single-sentence decodes
    (top1 bitwise; lse to float rounding, its summation order following the
    kernel that ran)."""
    gm, ctx, M = build(CHAIN, seed=4, bias_std=0.5, ln_std=0.3)
    srcs = sources(CHAIN.vocab, 3, seed=22)
    ms = [16, 11, 14]
    for mode, b in MODES:
        say(f"case trace batch mode={mode} b={b}")
        ctx.set_trace(0, 0)
        plain = gpu_decode_batch(ctx, srcs, ms, mode, b)
        ctx.set_trace(8192, 3 * 16)
        traced = gpu_decode_batch(ctx, srcs, ms, mode, b)
        rec, count = ctx.trace()
        assert count == len(rec)
        for p, t in zip(plain, traced):
            np.testing.assert_array_equal(p.ids, t.ids)
            assert (p.k, p.flags) == (t.k, t.flags)
        for s in range(3):
            mine = rec[rec["sentence"] == s]
            assert np.all(np.diff(mine["iteration"]) >= 0)
            assert mine["iteration"].max() == traced[s].k
            ctx.set_trace(4096, 16)
            gpu_decode_batch(ctx, [srcs[s]], [ms[s]], mode, b)
            one, _ = ctx.trace()
            cols = ["iteration", "position", "token"]
            for c in cols:
                np.testing.assert_array_equal(mine[c], one[c])
            np.testing.assert_array_equal(mine["top1"].view(np.uint32), one["top1"].view(np.uint32))
            np.testing.assert_allclose(mine["lse"], one["lse"], rtol=1e-6, atol=1e-6)
    ctx.set_trace(0, 0)


def test_trace_capacity_and_scratch_limits():
    """The buffer keeps the first `capacity` records while the count keeps
    growing; a scratch too small for the iteration's rows is refused before
    anything runs, and the context stays usable."""
    gm, ctx, M = build(TINY, seed=5)
    src = sources(TINY.vocab, 1, seed=23)[0]
    ctx.set_trace(4096, 16)
    gpu_decode_batch(ctx, [src], [16], "jacobi")
    full, n_full = ctx.trace()
    ctx.set_trace(5, 16)
    gpu_decode_batch(ctx, [src], [16], "jacobi")
    head, n = ctx.trace()
    assert n == n_full and len(head) == 5
    np.testing.assert_array_equal(head, full[:5])
    ctx.set_trace(16, 4)                              # 4 rows of scratch, Jacobi needs 16
    with pytest.raises(pdec.PdError) as ei:
        gpu_decode_batch(ctx, [src], [16], "jacobi")
    assert ei.value.status == 3
    ctx.set_trace(0, 0)
    want = oracle.decode(M, M.encode(src), 16, "jacobi")
    g = gpu_decode_batch(ctx, [src], [16], "jacobi")[0]
    np.testing.assert_array_equal(g.ids, want.out)


MID_F32 = dataclasses.replace(C.TINY, name="mid_f32", d_model=128, n_heads=2, d_ff=256, vocab=700)
WIDE_PRE_BF16 = dataclasses.replace(C.TINY, name="wide_pre", n_dec=1, n_enc=1, d_model=640, n_heads=10, d_ff=640,
                                    vocab=500, pre_ln=True, act_gelu=True, dtype=C.BF16)


@pytest.mark.parametrize("cfg,wkw", [(CHAIN, dict(bias_std=0.5, ln_std=0.3)), (MID_F32, {}),
                                     (WIDE_PRE_BF16, dict(bias_std=0.3, ln_std=0.2))],
                         ids=["chain_f32_dh16", "mid_f32_dh64", "wide_pre_bf16_dh64"])
def test_rows_of_several_key_chunks_agree_across_launch_shapes(cfg, wkw):
    """Launches whose rows may see more than 64 keys (by the host's bound on
    the key counts) evaluate a row's 64-key chunks on several waves side by
    side and fold them in key order; the others fold one chunk after another
    on one wave.  A row is bitwise the same either way, and whatever the
    launch's row count.  Cross-attention: a 40-token source's teacher-forced
    logits in a batch with a 200-token one (several-wave launch) against the
    same source encoded alone (one-wave launch), and 8 against 30 positions.
    Self- and cross-attention with up to 200 keys (four chunks, more than the
    waves of a row, so a wave also folds a later chunk): greedy steps (one
    row, m = 200) against the last evaluation of each position in a Jacobi
    decode (200 rows per iteration), whose prefix is the same greedy output:
    same tokens, top-1 logits bitwise."""
    import torch
    gm, ctx, M = build(cfg, seed=9, max_batch=3, max_src=256, max_tgt=256, **wkw)
    lens = (200, 40, 70)
    srcs = [np.random.default_rng(31 + i).integers(4, cfg.vocab, n).astype(np.int32) for i, n in enumerate(lens)]
    src = np.zeros((3, 200), np.int32)
    for r, s in enumerate(srcs):
        src[r, :len(s)] = s
    tgt = np.concatenate([np.ones((3, 1), np.int32),
                          np.random.default_rng(32).integers(0, cfg.vocab, (3, 29)).astype(np.int32)], 1)
    say(f"case several chunks cfg={cfg.name}: teacher-forced, batch of sources {lens} and the 40-token one alone")
    ctx.encode(torch.from_numpy(src).cuda(), list(lens))
    full = ctx.debug_logits(torch.from_numpy(tgt)).cpu().numpy()
    part = ctx.debug_logits(torch.from_numpy(np.ascontiguousarray(tgt[:, :8]))).cpu().numpy()
    np.testing.assert_array_equal(part, full[:, :8])
    ctx.encode(torch.from_numpy(np.ascontiguousarray(src[1:2, :40])).cuda(), [40])
    alone = ctx.debug_logits(torch.from_numpy(np.ascontiguousarray(tgt[1:2]))).cpu().numpy()
    np.testing.assert_array_equal(alone[0], full[1])

    m = 200
    say(f"case several chunks cfg={cfg.name}: greedy vs Jacobi, m={m}")
    ctx.set_trace(65536, m)
    ar = gpu_decode_batch(ctx, srcs[:1], [m], "ar")[0]
    rec_ar, n_ar = ctx.trace()
    assert n_ar == len(rec_ar)
    jac = gpu_decode_batch(ctx, srcs[:1], [m], "jacobi")[0]
    rec_j, n_j = ctx.trace()
    assert n_j == len(rec_j)
    ctx.set_trace(0, 0)
    np.testing.assert_array_equal(jac.ids, ar.ids)
    last = {}
    for r in rec_j:                                   # evaluation order: the last record of a position wins
        last[int(r["position"])] = r
    assert len(rec_ar) == len(ar.ids) >= 129, (len(rec_ar), len(ar.ids))
    for r in rec_ar:
        j = last[int(r["position"])]
        assert int(j["token"]) == int(r["token"])
        assert np.float32(j["top1"]).view(np.uint32) == np.float32(r["top1"]).view(np.uint32), (r, j)


@pytest.mark.parametrize("cfg,wkw", [(CHAIN, dict(bias_std=0.5, ln_std=0.3)), (MID_F32, {}),
                                     (WIDE_PRE_BF16, dict(bias_std=0.3, ln_std=0.2))],
                         ids=["chain_f32_dh16", "mid_f32_dh64", "wide_pre_bf16_dh64"])
def test_one_source_padding_changes_no_row(cfg, wkw):
    """A batch of one source (its key slots loaded before its length arrives)
    encoded with padding past its length, and as the first of a batch of two:
    the teacher-forced logits equal those of the unpadded encode bitwise, for
    sources of one and of several key chunks."""
    import torch
    gm, ctx, M = build(cfg, seed=10, max_batch=2, max_src=256, max_tgt=32, **wkw)
    tgt = np.concatenate([np.ones((1, 1), np.int32),
                          np.random.default_rng(33).integers(0, cfg.vocab, (1, 15)).astype(np.int32)], 1)
    for n in (10, 100):
        say(f"case one source cfg={cfg.name} n={n}")
        src = np.random.default_rng(34 + n).integers(4, cfg.vocab, n).astype(np.int32)
        ctx.encode(torch.from_numpy(src[None, :]).cuda(), [n])
        plain = ctx.debug_logits(torch.from_numpy(tgt)).cpu().numpy()
        padded = np.zeros((1, n + 37), np.int32)
        padded[0, :n] = src
        ctx.encode(torch.from_numpy(padded).cuda(), [n])
        np.testing.assert_array_equal(ctx.debug_logits(torch.from_numpy(tgt)).cpu().numpy(), plain)
        pair = np.zeros((2, n + 5), np.int32)
        pair[0, :n] = src
        pair[1, :] = np.random.default_rng(35).integers(4, cfg.vocab, n + 5)
        ctx.encode(torch.from_numpy(pair).cuda(), [n, n + 5])
        two = ctx.debug_logits(torch.from_numpy(np.repeat(tgt, 2, axis=0))).cpu().numpy()
        np.testing.assert_array_equal(two[0], plain[0])

