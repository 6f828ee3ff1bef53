"""The work whose speed counts: one call, or one training pass, through the public entry
points of paper_2208_08124_amd.fmha, at the sizes users of the library bring.

An attention case is one layer's attention of an unpadded batch: the forward call alone
(serving), or forward and backward with the tile list shared between them (training).  The
other kinds are the steps around it: Dropout + Add + LayerNorm, the padded <-> unpadded
conversions, and the embedding's backward.  A case fixes the multiset of sequence lengths;
the seed decides in which order the sequences are packed, and all values.
"""
import math

import numpy as np
import torch

from paper_2208_08124_amd import fmha

DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16}
HEAD_DIM = 64
VOCAB = 30522        # word pieces of the BERT models
DROP_SEED = 220808124


def listed():
    return [
        # --- serving: forward only ---
        # the smallest call: four short sequences, two heads (one tensor-parallel slice); latency
        dict(name="serve_tiny", kind="attention", mixture="ladder", batch=4, max_len=128, heads=2,
             dtype="f16", train=False, drop=0.0, interleaved=False, static=False, lengths=1),
        # a serving batch of ragged requests; no workspace, Q, K, V sliced from one projection
        dict(name="serve_ragged", kind="attention", mixture="uniform", batch=9, max_len=387, heads=12,
             dtype="bf16", train=False, drop=0.0, interleaved=True, static=True, lengths=2),
        # --- training: forward and backward ---
        # a BERT-large micro-batch: 56 sequences, a third of them at the maximum length
        dict(name="train_bert", kind="attention", mixture="bert", batch=56, max_len=512, heads=16,
             dtype="f16", train=True, drop=0.0, interleaved=False, static=False, lengths=3),
        # the same with what BERT pre-training applies: dropout on the probabilities, fused QKV storage
        dict(name="train_bert_dropout", kind="attention", mixture="bert", batch=56, max_len=512, heads=16,
             dtype="f16", train=True, drop=0.1, interleaved=True, static=False, lengths=3),
        # fine-tuning data: mostly very short sequences, a few at the maximum
        dict(name="train_skewed", kind="attention", mixture="skewed", batch=256, max_len=512, heads=16,
             dtype="f16", train=True, drop=0.0, interleaved=False, static=False, lengths=4),
        # long documents
        dict(name="train_long", kind="attention", mixture="full", batch=16, max_len=2048, heads=16,
             dtype="f16", train=True, drop=0.0, interleaved=False, static=False, lengths=5),
        # the largest: a BERT-base batch of half a million tokens
        dict(name="train_large", kind="attention", mixture="uniform", batch=2048, max_len=512, heads=12,
             dtype="bf16", train=True, drop=0.0, interleaved=False, static=False, lengths=6),
        # --- around the attention ---
        # Dropout + Add + LayerNorm, forward and backward, on the rows of a BERT-large micro-batch
        dict(name="layernorm_bert", kind="layernorm", rows=15769, hidden=1024, dtype="f16", drop=0.1),
        # and of the largest batch
        dict(name="layernorm_large", kind="layernorm", rows=527340, hidden=768, dtype="bf16", drop=0.1),
        # input mask -> indices, gather to the packed rows, scatter back, once per model step
        dict(name="unpad_bert", kind="unpad", mixture="bert", batch=56, max_len=512, hidden=1024,
             dtype="f16", lengths=3),
        # weight gradient of the word embedding: in one call, for a micro-batch
        dict(name="embedding_bert", kind="embedding", rows=15769, hidden=1024, vocab=VOCAB, dtype="f16",
             sort=False),
        # and with the positions ordered first, for the largest batch
        dict(name="embedding_large", kind="embedding", rows=527340, hidden=768, vocab=VOCAB, dtype="bf16",
             sort=True),
    ]


# ---------------------------------------------------------------- drawn cases

def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["attention"] * 6 + ["layernorm", "unpad", "embedding"])
    dtype = rng.choice(["f16", "bf16"])
    if kind == "attention":
        while True:
            train = rng.random() < 0.65
            c = dict(kind=kind, mixture=rng.choice(["bert", "skewed", "uniform", "uniform", "full"]),
                     batch=_log_int(rng, 1, 2048), max_len=_log_int(rng, 24, 2048),
                     heads=rng.choice([1, 2, 3, 4, 5, 8, 12, 16]), dtype=dtype, train=train,
                     drop=0.1 if train and rng.random() < 0.4 else 0.0,
                     interleaved=rng.random() < 0.5, static=not train and rng.random() < 0.5,
                     lengths=rng.randrange(1 << 20))
            n = _lengths(c).astype(np.float64)
            # within the largest listed case, in products (dropout costs about half as much
            # again) as in bytes
            cost = float((n * n).sum()) * c["heads"] * (1.5 if c["drop"] else 1.0)
            if cost <= 1.5e9 and n.sum() * c["heads"] <= 6.3e6:
                return c
    if kind == "layernorm":
        hidden = rng.choice([128, 256, 512, 768, 1024, 1040, 1536, 2048, 4096])
        return dict(kind=kind, rows=_log_int(rng, 48, min(527340, 405_000_000 // hidden)), hidden=hidden,
                    dtype=dtype, drop=rng.choice([0.0, 0.1]))
    if kind == "unpad":
        return dict(kind=kind, mixture=rng.choice(["bert", "skewed", "uniform"]), batch=_log_int(rng, 2, 1024),
                    max_len=_log_int(rng, 32, 512), hidden=rng.choice([128, 256, 768, 1024]), dtype=dtype,
                    lengths=rng.randrange(1 << 20))
    sort = rng.random() < 0.5
    hidden = rng.choice([128, 256, 512, 768, 1024])
    return dict(kind=kind, rows=_log_int(rng, 256, 527340 if sort else 32768), hidden=hidden,
                vocab=rng.choice([VOCAB, 8192, 28996]), dtype=dtype if sort else "f16", sort=sort)


def _lengths(case):
    """The case's sequence lengths (int32), in no particular order."""
    n, top = case["batch"], case["max_len"]
    rng = np.random.default_rng(case["lengths"])
    u = rng.random(n)
    if case["mixture"] == "ladder":       # 3, 17, 64, 128 of 128
        x = np.array([top, top // 2, top // 8 + 1, 3])[np.arange(n) % 4]
    elif case["mixture"] == "full":
        x = np.full(n, top)
    elif case["mixture"] == "uniform":
        x = rng.integers(1, top + 1, size=n)
    else:
        a = rng.integers(1, max(top // 4, 1) + 1, size=n)
        if case["mixture"] == "bert":     # 30 % short, 40 % between, 30 % at the maximum
            b = rng.integers(top // 4 + 1, top + 1, size=n)
            x = np.where(u < 0.3, a, np.where(u < 0.7, b, top))
        else:                             # "skewed": 60 % very short, 25 % short, 15 % at the maximum
            x = np.where(u < 0.6, (a + 1) // 2, np.where(u < 0.85, top // 8 + (3 * a) // 2, top))
    return np.clip(x, 1, top).astype(np.int32)


def _packed(case, seed):
    """Lengths in the seed's pack order, and their prefix sums."""
    n = np.random.default_rng([seed, 7]).permutation(_lengths(case))
    cu = np.zeros(len(n) + 1, dtype=np.int32)
    np.cumsum(n, out=cu[1:])
    return n, cu


# ---------------------------------------------------------------- prepare / run

class _State:
    pass


def prepare(case, seed):
    return {"attention": _prepare_attention, "layernorm": _prepare_layernorm, "unpad": _prepare_unpad,
            "embedding": _prepare_embedding}[case["kind"]](case, seed)


def run(state):
    return state.run(state)


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _normal(shape, dtype, gen):
    return torch.randn(shape, dtype=DTYPES[dtype], device="cuda", generator=gen)


def _prepare_attention(case, seed):
    s, gen = _State(), _generator(seed)
    _, cu = _packed(case, seed)
    h, t = case["heads"], int(cu[-1])
    s.cu, s.max_len, s.scale = torch.from_numpy(cu).cuda(), case["max_len"], HEAD_DIM ** -0.5
    if case["interleaved"]:
        s.q, s.k, s.v = _normal((t, 3, h, HEAD_DIM), case["dtype"], gen).unbind(1)
    else:
        s.q, s.k, s.v = (_normal((t, h, HEAD_DIM), case["dtype"], gen) for _ in range(3))
    s.o = torch.empty((t, h, HEAD_DIM), dtype=s.q.dtype, device="cuda")
    s.lse = torch.empty((h, t), dtype=torch.float32, device="cuda")
    if case["static"]:
        s.run = _run_forward_static
        return s
    s.workspace = fmha.alloc_workspace(case["batch"], t, h, case["train"])
    if not case["train"]:
        s.run = _run_forward
        return s
    s.dropout = (case["drop"], DROP_SEED + seed) if case["drop"] else None
    s.d_o = _normal((t, h, HEAD_DIM), case["dtype"], gen)
    if case["interleaved"]:
        s.grads = torch.empty((t, 3, h, HEAD_DIM), dtype=s.q.dtype, device="cuda")
        s.dq, s.dk, s.dv = s.grads.unbind(1)
    else:
        s.dq, s.dk, s.dv = (torch.empty_like(s.q) for _ in range(3))
    s.run = _run_train
    return s


def _run_forward(s):
    fmha.fmha_varlen_fwd(s.q, s.k, s.v, s.cu, s.max_len, s.scale, s.o, s.lse, s.workspace)
    return s.o, s.lse


def _run_forward_static(s):
    fmha.fmha_varlen_fwd_static(s.q, s.k, s.v, s.cu, s.max_len, s.scale, s.o, s.lse)
    return s.o, s.lse


def _run_train(s):
    fmha.fmha_varlen_fwd(s.q, s.k, s.v, s.cu, s.max_len, s.scale, s.o, s.lse, s.workspace, dropout=s.dropout)
    fmha.fmha_varlen_bwd(s.q, s.k, s.v, s.o, s.d_o, s.lse, s.cu, s.max_len, s.scale, s.dq, s.dk, s.dv,
                         s.workspace, reuse_schedule=True, dropout=s.dropout)
    return s.o, s.lse, s.dq, s.dk, s.dv


def _prepare_layernorm(case, seed):
    s, gen = _State(), _generator(seed)
    t, n = case["rows"], case["hidden"]
    s.x, s.residual, s.dy = (_normal((t, n), case["dtype"], gen) for _ in range(3))
    s.gamma = 1.0 + 0.1 * torch.randn(n, device="cuda", generator=gen)
    s.beta = 0.1 * torch.randn(n, device="cuda", generator=gen)
    s.y, s.z, s.dx, s.dresidual = (torch.empty_like(s.x) for _ in range(4))
    s.mu, s.rstd = (torch.empty(t, dtype=torch.float32, device="cuda") for _ in range(2))
    s.dgamma, s.dbeta = (torch.empty(n, dtype=torch.float32, device="cuda") for _ in range(2))
    s.workspace = torch.empty(fmha.fmha_dropout_add_ln_bwd_workspace_size(t, n), dtype=torch.uint8, device="cuda")
    s.dropout = (case["drop"], DROP_SEED + seed) if case["drop"] else None
    s.run = _run_layernorm
    return s


def _run_layernorm(s):
    fmha.fmha_dropout_add_ln_fwd(s.x, s.residual, s.gamma, s.beta, 1e-12, s.y, s.z, s.mu, s.rstd, dropout=s.dropout)
    fmha.fmha_dropout_add_ln_bwd(s.dy, s.z, s.mu, s.rstd, s.gamma, 1e-12, s.dx, s.dresidual, s.dgamma, s.dbeta,
                                 s.workspace, dropout=s.dropout)
    return s.y, s.z, s.mu, s.rstd, s.dx, s.dresidual, s.dgamma, s.dbeta


def _prepare_unpad(case, seed):
    s, gen = _State(), _generator(seed)
    n, _ = _packed(case, seed)
    b, top = case["batch"], case["max_len"]
    s.mask = (torch.arange(top, device="cuda")[None, :] < torch.from_numpy(n).cuda()[:, None]).to(torch.int32)
    s.padded = _normal((b * top, case["hidden"]), case["dtype"], gen)
    s.valid = int(n.sum())                 # only to cut what run() returns to what is written
    s.indices = torch.empty(b * top, dtype=torch.int32, device="cuda")
    s.inverse = torch.empty(b * top, dtype=torch.int32, device="cuda")
    s.cu = torch.empty(b + 1, dtype=torch.int32, device="cuda")
    s.packed = torch.empty_like(s.padded)  # room for the worst case: the host does not know the count
    s.restored = torch.empty_like(s.padded)
    s.run = _run_unpad
    return s


def _run_unpad(s):
    fmha.fmha_unpad_indices(s.mask, s.indices, s.inverse, s.cu)
    fmha.fmha_gather_rows(s.padded, s.indices, s.cu[-1:], s.packed)
    fmha.fmha_scatter_rows(s.packed, s.inverse, s.cu[-1:], s.restored)
    return s.indices[:s.valid], s.inverse, s.cu, s.packed[:s.valid], s.restored


def _prepare_embedding(case, seed):
    s, gen = _State(), _generator(seed)
    t, n, vocab = case["rows"], case["hidden"], case["vocab"]
    # word-piece frequencies follow Zipf's law
    w = 1.0 / torch.arange(1, vocab + 1, device="cuda", dtype=torch.float64)
    cdf = torch.cumsum(w / w.sum(), 0)
    ranks = torch.searchsorted(cdf, torch.rand(t, device="cuda", dtype=torch.float64, generator=gen))
    s.ids = torch.randperm(vocab, device="cuda", generator=gen)[ranks.clamp_(max=vocab - 1)].to(torch.int32)
    s.dy = _normal((t, n), case["dtype"], gen)
    s.dw = torch.zeros((vocab, n), dtype=s.dy.dtype, device="cuda")
    if case["sort"]:
        s.workspace = torch.empty(fmha.fmha_embedding_sort_workspace_size(t, n), dtype=torch.uint8, device="cuda")
        s.run = _run_embedding_sorted
    else:
        s.run = _run_embedding
    return s


def _run_embedding(s):
    fmha.fmha_embedding_bwd(s.dy, s.ids, s.dw, zero_first=True)
    return s.dw


def _run_embedding_sorted(s):
    fmha.fmha_embedding_sort(s.ids, s.dy.shape[1], s.dw.shape[0], s.workspace)
    fmha.fmha_embedding_bwd_sorted(s.dy, s.workspace, s.dw, zero_first=True)
    return s.dw


# ---------------------------------------------------------------- work and tolerance

def work(case):
    if case["kind"] == "attention":
        n = _lengths(case).astype(np.float64)
        rows, s2 = float(n.sum()) * case["heads"], float((n * n).sum()) * case["heads"]
        # forward: Q, K, V -> O, LSE; backward: Q, K, V, O, dO, LSE -> dQ, dK, dV
        nbytes = rows * (4 * 128 + 4 + ((8 * 128 + 4) if case["train"] else 0))
        return {"bytes": nbytes, "flops": (14 if case["train"] else 4) * s2 * HEAD_DIM}
    if case["kind"] == "layernorm":
        rows, n = case["rows"], case["hidden"]
        # forward: x, residual -> y, z, mu, rstd; backward: dy, z, mu, rstd -> dx, dresidual
        return {"bytes": rows * (16.0 * n + 16) + 20.0 * n, "flops": 25.0 * rows * n}
    if case["kind"] == "unpad":
        valid, total = float(_lengths(case).sum()), float(case["batch"]) * case["max_len"]
        row = 2.0 * case["hidden"]
        # indices: mask -> indices, inverse; gather: rows in and out; scatter: rows in, all rows out
        return {"bytes": 8 * total + 4 * valid + 2 * valid * row + 4 * valid + (valid + total) * row + 4 * total,
                "flops": 0.0}
    t, n = case["rows"], case["hidden"]
    # ids and gradient rows in, every weight row out
    return {"bytes": 4.0 * t + 2.0 * t * n + 2.0 * case["vocab"] * n, "flops": float(t) * n}


def tolerance(case):
    # four times the distance from the same operation in float64 on these inputs
    if case["kind"] == "unpad":
        return "exact"
    f16 = case["dtype"] == "f16"
    if case["kind"] == "attention":      # measured 3e-4 / 9e-3 and 2.5e-3 / 6e-2
        return {"rel": 1.2e-3, "max": 4e-2} if f16 else {"rel": 1e-2, "max": 2.5e-1}
    if case["kind"] == "layernorm":      # 2.9e-4 / 1.0e-3 and 2.3e-3 / 8.5e-3
        return {"rel": 1.2e-3, "max": 4e-3} if f16 else {"rel": 1e-2, "max": 3.5e-2}
    if not case["sort"]:                 # every addition is rounded to 16 bits: 1.8e-3 / 0.37
        return {"rel": 7e-3, "max": 0.9}
    # sums in float32, rounded once: 2.1e-4 / 4.9e-4 and 1.7e-3 / 3.9e-3
    return {"rel": 8e-4, "max": 2e-3} if f16 else {"rel": 7e-3, "max": 1.6e-2}
