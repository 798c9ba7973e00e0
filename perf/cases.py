"""Performance cases: translation and scoring through the Python entry points.

A case is one call pattern of a serving program that keeps a model and a
context (pdec.Model, pdec.Context) and feeds them source after source:

  kind "translate"  encode a batch of sources, decode it, and score a given
                    reference translation of the same length under the model
                    (teacher-forced logits, as an evaluation pass does);
  kind "trace"      the same with the decoding trace on (per evaluated row:
                    iteration, position, token, its logit and log-sum-exp);
  kind "score"      encode a batch and score reference translations only.

Weights are seeded random ones of the shape (biases and LayerNorm affines
non-zero), made once per process and kept, as a program keeps its model;
sources and references come from the seed.  Sentence lengths of a batch are
spread evenly over [n_lo, n_hi] and m = n + extra, the workloads' rule.
"""
from __future__ import annotations

import dataclasses
import math

import numpy as np
import torch

from paper_2305_10427_amd import configs as C, pdec, synth

MODELS = {
    "tiny": C.TINY,
    "mt_base": C.MT_BASE,
    "large": C.LARGE,
    # a small pre-LN / GELU model of odd widths: 10 heads of 64, a vocabulary
    # that is no multiple of any tile
    "wide": dataclasses.replace(C.TINY, name="wide", n_enc=2, n_dec=2, d_model=640, n_heads=10, d_ff=1280,
                                vocab=7001, pre_ln=True, act_gelu=True, dtype=C.BF16),
    # head width 32, float32, pre-LN
    "mid": dataclasses.replace(C.TINY, name="mid", n_enc=3, n_dec=3, d_model=256, n_heads=8, d_ff=1024,
                               vocab=4003, pre_ln=True, act_gelu=True, dtype=C.F32),
}

# iterations per target position (k/m) that the random models of these shapes
# take in the block modes; greedy decoding takes one per position
K_OVER_M = {"tiny": 0.95, "mt_base": 0.5, "large": 1.0, "wide": 0.9, "mid": 0.9}


def _case(name, kind, model, dtype, batch, n_lo, n_hi, mode="none", block=1, stop="block", extra=10):
    return {"name": name, "kind": kind, "model": model, "dtype": dtype, "batch": batch, "n_lo": n_lo, "n_hi": n_hi,
            "extra": extra, "mode": mode, "block": block, "stop": stop}


def listed():
    return [
        # the smallest call: a 16-token sentence on the tiny model, all launches and latency
        _case("tiny_f32_gs4", "translate", "tiny", "f32", 1, 16, 16, "gs_jacobi", 4, extra=0),
        # interactive translation of one sentence, Transformer-base shape: float32 hybrid b = 5 (the paper's setting)
        _case("base_f32_hybrid5", "translate", "mt_base", "f32", 1, 35, 35, "hybrid", 5),
        # the same in bfloat16: greedy decoding, the baseline of every comparison
        _case("base_bf16_ar", "translate", "mt_base", "bf16", 1, 27, 27, "ar"),
        # bfloat16 GS-Jacobi b = 5 with the decoding trace on (token probabilities for a viewer)
        _case("base_bf16_gs5_trace", "trace", "mt_base", "bf16", 1, 52, 52, "gs_jacobi", 5),
        # one Jacobi block of the whole target (m rows an iteration), prefix stopping condition
        _case("base_bf16_jacobi", "translate", "mt_base", "bf16", 1, 43, 43, "jacobi", 1, "prefix"),
        # offline translation in batches of 64 sentences of mixed length
        _case("base_bf16_b64_hybrid5", "translate", "mt_base", "bf16", 64, 5, 71, "hybrid", 5),
        # validation loss of a float32 model: encode and score references only
        _case("base_f32_b16_score", "score", "mt_base", "f32", 16, 9, 60),
        # interactive translation with the large multilingual shape: greedy, and GS-Jacobi b = 16 (long sentence)
        _case("large_bf16_ar", "translate", "large", "bf16", 1, 38, 38, "ar"),
        _case("large_bf16_gs16", "translate", "large", "bf16", 1, 101, 101, "gs_jacobi", 16),
        # batched serving of the large model: greedy, and GS-Jacobi b = 16 (the largest case)
        _case("large_bf16_b32_ar", "translate", "large", "bf16", 32, 20, 120, "ar"),
        _case("large_bf16_b32_gs16", "translate", "large", "bf16", 32, 20, 120, "gs_jacobi", 16),
        # scoring candidate translations with the large model
        _case("large_bf16_b8_score", "score", "large", "bf16", 8, 30, 119),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    model = rng.choice(["tiny", "mid", "wide", "mt_base", "mt_base", "mt_base", "large", "large"])
    dtype = {"tiny": "f32", "mid": "f32", "wide": "bf16", "large": "bf16"}.get(model) or rng.choice(["f32", "bf16"])
    kind = rng.choice(["translate"] * 7 + ["score"] * 2 + ["trace"])
    batch = _log_int(rng, 1, {"large": 24, "mt_base": 64}.get(model, 40)) if rng.random() < 0.6 else 1
    if kind == "trace":
        batch = min(batch, 2)                        # the static trace scratch bounds an iteration's rows
    n_hi = _log_int(rng, 5, 120 if model != "tiny" else 30)
    n_lo = n_hi if batch == 1 else rng.randint(max(1, n_hi // 6), n_hi)
    mode, block, stop = "none", 1, "block"
    if kind != "score":
        mode = rng.choice(["ar", "gs_jacobi", "gs_jacobi", "hybrid", "jacobi"])
        if mode in ("gs_jacobi", "hybrid"):
            block = _log_int(rng, 2, 32 if batch == 1 else 16)
        if mode == "jacobi" and batch > (2 if model == "large" else 8):
            mode, block = "gs_jacobi", 3
        if mode != "ar" and rng.random() < 0.3:
            stop = "prefix"
    c = _case("", kind, model, dtype, batch, n_lo, n_hi, mode, block, stop, rng.randint(0, 12))
    del c["name"]
    return c


# --- models and contexts a serving program keeps -----------------------------

_KEPT = {}


def _cfg(case):
    return MODELS[case["model"]].with_dtype(case["dtype"])


def _weights(cfg):
    """Seeded weights on the GPU in canonical order, as {name: float32 tensor} (bf16-exact for bf16 models)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(1234 + cfg.d_model + cfg.vocab)
    out = {}
    for name, shape in C.param_shapes(cfg):
        t = torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)
        if len(shape) == 2:
            t = t / math.sqrt(shape[1])              # linear weights and the embedding
        elif name.endswith(".g"):
            t = 1.0 + 0.05 * t
        else:
            t = 0.02 * t
        out[name] = t.to(torch.bfloat16).float() if cfg.dtype == C.BF16 else t
    return out


def _model(cfg):
    key = ("model", cfg)
    if key not in _KEPT:
        w = _weights(cfg)
        bits = None
        if cfg.dtype == C.BF16:
            bits = {k: v.to(torch.bfloat16).view(torch.int16).cpu().numpy().view(np.uint16) for k, v in w.items()}
        values = {k: v.cpu().numpy() for k, v in w.items()}
        del w
        _KEPT[key] = pdec.Model(cfg, synth.Weights(cfg, values, bits))
    return _KEPT[key]


def _context(case, cfg, T):
    key = ("context", cfg, case["batch"], case["n_hi"], T)
    if key not in _KEPT:
        _KEPT[key] = pdec.Context(_model(cfg), case["batch"], case["n_hi"], T)
    return _KEPT[key]


# --- inputs ------------------------------------------------------------------

def _lengths(case):
    B, lo, hi = case["batch"], case["n_lo"], case["n_hi"]
    n = [hi] if B == 1 else [lo + round((hi - lo) * i / (B - 1)) for i in range(B)]
    return n, [max(1, k + case["extra"]) for k in n]


def _inputs(case, seed):
    """Sources [B, n_hi] (PAD after each length), lengths, targets m and reference inputs [B, T] (BOS first)."""
    cfg = _cfg(case)
    g = np.random.Generator(np.random.PCG64(seed))
    n, m = _lengths(case)
    order = g.permutation(len(n))
    n, m = [n[i] for i in order], [m[i] for i in order]
    T = max(m)
    src = np.full((len(n), case["n_hi"]), C.PAD_ID, np.int32)
    ref = np.full((len(n), T), C.PAD_ID, np.int32)
    for b in range(len(n)):
        src[b, :n[b]] = g.integers(C.FIRST_WORD_ID, cfg.vocab, n[b])
        ref[b, 0] = C.BOS_ID
        ref[b, 1:m[b]] = g.integers(C.FIRST_WORD_ID, cfg.vocab, m[b] - 1)
    return src, n, m, ref


def prepare(case, seed):
    cfg = _cfg(case)
    src, n, m, ref = _inputs(case, seed)
    B, T = ref.shape
    state = {"case": case, "ctx": _context(case, cfg, T), "src": torch.from_numpy(src).cuda(), "n": n, "m": m,
             "ref": torch.from_numpy(ref).cuda()}
    state["out"] = tuple(torch.empty(s, dtype=torch.int32, device="cuda") for s in ((B, T), (B,), (B,), (B,)))
    return state


def run(state):
    case, ctx = state["case"], state["ctx"]
    ctx.encode(state["src"], state["n"])
    res = {}
    if case["kind"] == "translate":
        res["ids"], res["len"], res["k"], res["flags"] = ctx.decode(
            case["mode"], state["m"], block=case["block"], stop=case["stop"], out=state["out"])
    elif case["kind"] == "trace":
        rows = {"ar": 1, "jacobi": max(state["m"])}.get(case["mode"], case["block"]) * case["batch"]
        cap = rows * max(state["m"])
        ids, ln, k, fl, rec, count = ctx.decode_traced_static(case["mode"], state["m"], cap, block=case["block"],
                                                              stop=case["stop"])
        res = {"ids": ids, "len": ln, "k": k, "flags": fl, "count": count}
        full = np.zeros(cap, rec.dtype)              # the viewer's buffer: records, then zeros
        full[:len(rec)] = rec
        for f in ("iteration", "sentence", "position", "token", "top1", "lse"):
            res["rec_" + f] = full[f]
    res["logits"] = ctx.debug_logits(state["ref"])
    return res


# --- floors and tolerances ----------------------------------------------------

def work(case):
    cfg = _cfg(case)
    d, f, V, es = cfg.d_model, cfg.d_ff, cfg.vocab, 2 if cfg.dtype == C.BF16 else 4
    n, m = _lengths(case)
    T = max(m)
    enc_w = cfg.n_enc * (4 * d * d + 2 * d * f) + cfg.n_dec * 2 * d * d
    dec_w = cfg.n_dec * (6 * d * d + 2 * d * f)
    # scoring: every weight once, the logits written once
    rows = len(m) * T
    nbytes = (enc_w + dec_w + V * d) * es + rows * V * 4
    flops = 2 * sum(n) * enc_w + 2 * rows * (dec_w + V * d)
    if case["kind"] != "score":
        mode = case["mode"]
        ratio = 1.0 if mode == "ar" else K_OVER_M[case["model"]] * (0.3 if mode == "jacobi" else 1.0)
        if case["model"] == "large" and mode == "jacobi":
            ratio = 1.0
        L = {"ar": 1, "jacobi": T}.get(mode, case["block"])
        iters = max(1, math.ceil(ratio * T))
        done = sum(max(1, math.ceil(ratio * x)) * min(L, x) for x in m)   # rows over all iterations
        nbytes += iters * (dec_w + V * d) * es        # an iteration streams the decoder and the embedding
        flops += 2 * done * (dec_w + V * d)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # logits against float64, 2-norm: 2.5e-7 to 6.1e-7 (f32), 4.3e-3 to 8.8e-3 (bf16) measured over
    # the listed and some drawn cases; about four (bf16: two to four) times that.  Tokens and counts: ties only.
    if _cfg(case).dtype == C.BF16:
        return {"rel": 2e-2, "max": 0.2, "differ": 0.01}
    return {"rel": 2.5e-6, "max": 2.5e-5, "differ": 0.01}


# --- the same logits in float64 by plain torch ---------------------------------

def _attend(q, k, v, H, mask):
    B, T, d = q.shape
    S = k.shape[1]
    sp = lambda x, L: x.view(B, L, H, d // H).transpose(1, 2)  # noqa: E731
    s = sp(q, T) @ sp(k, S).transpose(2, 3) / math.sqrt(d // H)
    p = torch.softmax(s.masked_fill(~mask, float("-inf")), -1)
    return (p @ sp(v, S)).transpose(1, 2).reshape(B, T, d)


def exact(case, seed):
    cfg = _cfg(case)
    W = _weights(cfg)
    src, n, m, ref = _inputs(case, seed)
    d, H = cfg.d_model, cfg.n_heads
    F = torch.nn.functional
    w = lambda name: W[name].double()  # noqa: E731
    lin = lambda x, p, leaf: F.linear(x, w(p + "w" + leaf), w(p + "b" + leaf))  # noqa: E731
    ln = lambda x, p: F.layer_norm(x, (d,), w(p + ".g"), w(p + ".b"), cfg.ln_eps)  # noqa: E731
    act = F.gelu if cfg.act_gelu else F.relu
    pos = torch.arange(1024, device="cuda", dtype=torch.float64)[:, None]
    freq = 10000.0 ** (-torch.arange(0, d, 2, device="cuda", dtype=torch.float64) / d)
    pe = torch.stack([torch.sin(pos * freq), torch.cos(pos * freq)], -1).reshape(1024, d)
    embed = lambda ids: W["emb"][ids].double() * math.sqrt(d) + pe[: ids.shape[1]]  # noqa: E731

    def sub(x, p, norm, fn):
        return x + fn(ln(x, p + norm)) if cfg.pre_ln else ln(x + fn(x), p + norm)

    src_t = torch.from_numpy(src).cuda().long()
    ref_t = torch.from_numpy(ref).cuda().long()
    keys = torch.arange(src.shape[1], device="cuda")[None, :] < torch.tensor(n, device="cuda")[:, None]
    kmask = keys[:, None, None, :]
    T = ref.shape[1]
    causal = torch.ones(T, T, dtype=torch.bool, device="cuda").tril()[None, None]

    def self_attn(p, mask):
        def fn(h):
            q, k, v = F.linear(h, w(p + "sa.w_qkv"), w(p + "sa.b_qkv")).chunk(3, -1)
            return lin(_attend(q, k, v, H, mask), p + "sa.", "_o")
        return fn

    def cross_attn(p, mem):
        def fn(h):
            k, v = lin(mem, p + "ca.", "_kv").chunk(2, -1)
            return lin(_attend(lin(h, p + "ca.", "_q"), k, v, H, kmask), p + "ca.", "_o")
        return fn

    def ffn(p):
        return lambda h: lin(act(lin(h, p + "ff.", "1")), p + "ff.", "2")

    x = embed(src_t)
    for l in range(cfg.n_enc):
        p = f"enc.{l}."
        x = sub(x, p, "ln1", self_attn(p, kmask))
        x = sub(x, p, "ln2", ffn(p))
    mem = ln(x, "enc.ln") if cfg.pre_ln else x
    y = embed(ref_t)
    for l in range(cfg.n_dec):
        p = f"dec.{l}."
        y = sub(y, p, "ln1", self_attn(p, causal))
        y = sub(y, p, "ln2", cross_attn(p, mem))
        y = sub(y, p, "ln3", ffn(p))
    if cfg.pre_ln:
        y = ln(y, "dec.ln")
    res = {"logits": cfg.logit_scale * (y @ w("emb").T) + w("out_bias")}
    names = {"score": [], "translate": ["ids", "len", "k", "flags"],
             "trace": ["ids", "len", "k", "flags", "count", "rec_iteration", "rec_sentence", "rec_position",
                       "rec_token", "rec_top1", "rec_lse"]}[case["kind"]]
    return {**{k: None for k in names}, **res}
