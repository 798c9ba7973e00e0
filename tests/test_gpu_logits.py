"""Teacher-forced logits at the workload shapes (pd_debug_logits, through the
C ABI) against the oracle: the measured error, relative to each row's max
|logit|, must stay below EPS of tests/parity.py, the bound the token rule's
near-tie threshold (2 EPS) is derived from, and below the north-star
tolerance (1e-3 float32, 5e-2 bfloat16).

The rows are the ones decoding evaluates: inputs BOS followed by the oracle's
greedy tokens, plus rows of random tokens (drafts that have not converged), in
batches of one and of several sentences (the streaming and the many-row
vocabulary kernels)."""
import numpy as np
import pytest

import oracle
from paper_2305_10427_amd import configs as C, pdec, synth
from tests.parity import EPS, TOL, workload_model

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)


def measure(wl_name, n_sent, T, batch):
    import torch
    wl = C.WORKLOADS[wl_name]
    cfg = wl.model
    _, gm, M = workload_model(cfg)
    sents = synth.make_sentences(wl, seed=1, count=n_sent)
    ctx = pdec.Context(gm, batch, max(len(s) for s, _ in sents), max(T, 16))
    g = np.random.default_rng(5)
    worst = 0.0
    for s0 in range(0, n_sent, batch):
        chunk = sents[s0:s0 + batch]
        n_max = max(len(s) for s, _ in chunk)
        src = np.zeros((len(chunk), n_max), np.int32)
        tgts, refs = [], []
        for r, (ids, _) in enumerate(chunk):
            src[r, :len(ids)] = ids
            enc = M.encode(ids)
            y = oracle.greedy(M, enc, T - 1, stop_at_eos=False).y
            tgt = np.concatenate([[C.BOS_ID], y]).astype(np.int32)
            if r % 2 == 1:                         # a draft that has not converged
                tgt[1 + T // 2:] = g.integers(4, cfg.vocab, T - 1 - T // 2)
            tgts.append(tgt)
            refs.append(M.teacher_forced_logits(enc, tgt))
        ctx.encode(torch.from_numpy(src).cuda(), [len(s) for s, _ in chunk])
        got = ctx.debug_logits(torch.from_numpy(np.stack(tgts))).cpu().numpy()
        for r in range(len(chunk)):
            rel = np.abs(got[r] - refs[r]).max(-1) / np.abs(refs[r]).max(-1)
            worst = max(worst, float(rel.max()))
    say(f"case logits {wl_name} sentences={n_sent} T={T} batch={batch}: max rel err {worst:.3g} "
        f"(EPS {EPS[cfg.dtype]:.1e})")
    assert worst <= EPS[cfg.dtype] <= TOL[cfg.dtype]
    return worst


@pytest.mark.parametrize("wl", ["tiny", "mt_base_f32", "mt_base_bf16"])
def test_teacher_forced_logits_mt_shapes(wl):
    measure(wl, 4, 16, 1)                          # 16-row iterations, streaming kernels
    measure(wl, 4, 24, 4)                          # 96 rows


def test_teacher_forced_logits_large_shape():
    measure("large", 2, 16, 1)
    measure("large", 2, 16, 2)                     # 32 rows: many-row vocabulary
