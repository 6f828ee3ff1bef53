"""The backward kernel that forms every score once, against the two passes it stands in for and
against the oracle.

The library takes it where the batch keeps all compute units busy with whole sequences.  The two
passes run one after the other (`only`) give the same dV bit for bit (same products in the same order),
and with dropout the same dK.  The rest differs by what rounds otherwise: dQ sums over keys in another
order, and without dropout dP - D is summed from -D on, so that a dS = P (dP - D) beside a rounding
boundary of the 16-bit type may fall on its other side.  One such dS moves a gradient by one unit in
the last place of dS times K or Q; the bound allows each of a row's dS to do so on average by a
quarter, in units of the largest gradient of the sequence."""
import numpy as np
import pytest
import torch

from oracle import dropout_mask as dm
from oracle import oracle
from oracle.parity import G_TOL, gradient_errors
from paper_2208_08124_amd import fmha
from paper_2208_08124_amd import workloads as wl

from gpu_util import DeviceBatch, oracle_inputs, to_f64

pytestmark = pytest.mark.gpu

EDGES = [1, 31, 32, 33, 63, 64, 65, 96, 127, 128, 129, 160, 255, 256]
LONG = EDGES + [257, 287, 288, 300, 384, 385, 511, 512]


def fill(some, n):
    return [some[i % len(some)] for i in range(n)]


def both_ways(b, dropout=None):
    """dQ, dK, dV by one call and by the two passes."""
    # the batch is one the library takes the kernel for, with some room: a compute unit's share of the work (in blocks of
    # 256 keys by 32 queries, as if all sequences were as long) is at least 0.6 of the longest sequence's
    # (0.2 up to 256 tokens, 0.9 beyond 1024)
    n = b["max_seqlen"]
    share = b["total_tokens"] ** 2 * b["heads"] / (b["batch"] * 8192.0 * 256)
    assert share >= (0.2 if n <= 256 else 0.6 if n <= 1024 else 0.9) * -(-n // 256) * -(-n // 32)
    assert fmha.fmha_varlen_bwd_passes(b["batch"], b["total_tokens"], b["heads"], n, dropout=dropout,
                                       seqused="seqused" in b) == 1
    db = DeviceBatch(b, True)
    db.fwd(dropout=dropout)
    for x in (db.dq, db.dk, db.dv):
        x.fill_(float("nan"))
    db.bwd(reuse_schedule=True, dropout=dropout)
    one = [x.clone() for x in (db.dq, db.dk, db.dv)]
    for x in (db.dq, db.dk, db.dv):
        x.fill_(float("nan"))
    db.bwd(reuse_schedule=True, dropout=dropout, only="dq")
    db.bwd(reuse_schedule=True, dropout=dropout, only="dkv")
    torch.cuda.synchronize()
    return db, one, [db.dq, db.dk, db.dv]


def compare(b, one, two, dtype, dropout=None):
    assert not any(torch.isnan(x).any() for x in one)
    assert torch.equal(one[2], two[2])
    if dropout:
        assert torch.equal(one[1], two[1])
    for x, y in zip(one[:2], two[:2]):
        rel, _ = gradient_errors(to_f64(x), to_f64(y), b["cu_seqlens"])
        assert rel <= (2.0 ** -9 if dtype == "f16" else 2.0 ** -6), rel


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("lengths,heads,dropout,used", [
    (fill([1, 31, 32, 33, 64], 300), 16, None, False),       # four heads at a time
    (fill([3, 64, 17, 64], 400), 13, None, False),               # and a last group of one
    (fill([65, 96, 97, 128], 150), 15, None, False),         # two at a time, the last alone
    (fill(EDGES, 140), 16, None, False),                      # all kinds, one sweep each
    (fill(LONG, 132), 16, None, False),                      # two sweeps
    (fill(LONG, 110), 16, (0.1, 77), False),
    (fill(EDGES, 140), 13, (0.25, 5), False),
    (fill(LONG, 110), 16, None, True),
    (fill([1025, 700, 1100], 40), 16, None, False),           # up to five
    (fill([5, 130, 256, 64], 24), 16, None, False),           # a few items for some workgroups, none for others
    (fill([5, 33, 63, 64], 300), 3, None, False),             # three heads
    (fill([5, 40, 100, 128], 300), 2, (0.1, 9), False),       # two
])
def test_one_pass_against_the_two(lengths, heads, dropout, used, dtype):
    b = wl.make_batch(lengths, heads, dtype, seed=len(lengths) + heads)
    if used:
        rng = np.random.default_rng(3)
        b["seqused"] = np.array([int(rng.integers(0, n + 1)) for n in lengths], dtype=np.int32)
    db, one, two = both_ways(b, dropout)
    compare(b, one, two, dtype, dropout)
    if dropout is None and not used:
        pick = list(range(0, len(lengths), max(len(lengths) // 7, 1)))
        cu = b["cu_seqlens"]
        rows = np.concatenate([np.arange(cu[i], cu[i + 1]) for i in pick])
        x = {n: v[rows] for n, v in oracle_inputs(b).items() if n in ("q", "k", "v", "do")}
        sub_cu = wl.cu_from_lengths(np.array([lengths[i] for i in pick]))
        ref = oracle.bwd(x["q"], x["k"], x["v"], x["do"], sub_cu, b["scale"])
        for name, got, want in zip(("dq", "dk", "dv"), one, ref):
            rel, fro = gradient_errors(to_f64(got[torch.from_numpy(rows).cuda()]), want, sub_cu)
            assert rel <= G_TOL and fro <= G_TOL, f"{name}: {rel:.3e} {fro:.3e}"


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_sequences_longer_than_stated(dtype):
    """max_seqlen too small: dQ does not fit its buffer, and is formed in sweeps of its own."""
    b = wl.make_batch(fill([40, 256, 64, 129], 130) + [700, 300, 1030], 12, dtype, seed=9)
    b["max_seqlen"] = 256
    db, one, two = both_ways(b)
    compare(b, one, two, dtype)


def test_repeats_itself_and_leaves_the_statistics_of_the_two_passes():
    b = wl.make_batch(fill(LONG, 132), 16, "f16", seed=4)
    db, one, two = both_ways(b)
    two_dk = two[1].clone()
    db.bwd(reuse_schedule=True)
    again = [x.clone() for x in (db.dq, db.dk, db.dv)]
    db.dk.fill_(float("nan"))
    db.bwd(reuse_schedule=True, only="dkv")    # with what the call before left in the workspace
    torch.cuda.synchronize()
    for x, y in zip(one, again):
        assert torch.equal(x, y)
    assert torch.equal(db.dk, two_dk)


def test_key_places_without_a_key_add_nothing():
    """The scores' gradients of a key that does not exist would overflow f16 (every row attends to its sequence's
    last key alone, dP / (1 - p) = 524 288): all dS are 0, in the one pass as in the two."""
    b = wl.make_batch(fill([1, 33, 40, 5, 70, 250], 240), 16, "f16", seed=3)
    value = lambda x: wl.to_bits(np.array([x], np.float32), "f16")[0]
    for name, x in (("q", 2.0), ("k", 0.0), ("v", 64.0), ("do", 64.0)):
        b[name][:] = value(x)
    b["k"][b["cu_seqlens"][1:] - 1] = value(4.0)
    _, one, two = both_ways(b, (0.5, 99))
    for x, y in zip(one, two):
        assert torch.isfinite(x).all() and torch.equal(x, y)
    assert not one[0].any()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_single_token_sequences(dtype):
    """P = 1 and O = V, so dP = D and dQ = dK = 0 but for rounding.  Products of 16-bit numbers are exact in fp32; with
    S = sum_c |dO_c V_c|, D takes at most 8 roundings of sums up to S and dP - D, summed from -D on, at most 64 of sums
    up to 2 S (truncated, 2^-23, if the matrix cores do): |dS| <= 2^-16 S.  dS and the result are rounded to 16 bits."""
    b = wl.make_batch(fill([1, 64, 33, 1, 200], 300), 16, dtype, seed=8)
    db, one, two = both_ways(b)
    compare(b, one, two, dtype)
    rows = b["cu_seqlens"][:-1][b["lengths"] == 1]
    x = {n: v[rows] for n, v in oracle_inputs(b).items()}
    o, dq, dk, dv = (to_f64(t)[rows] for t in [db.o] + one)
    assert np.array_equal(o, x["v"]) and np.array_equal(dv, x["do"])
    tiny = 2.0 ** -25 if dtype == "f16" else 0.0                        # half the smallest f16
    ds = 2.0 ** -16 * np.abs(x["do"] * x["v"]).sum(axis=2, keepdims=True) * (1 + 2.0 ** -7) + tiny
    for got, with_ in ((dq, x["k"]), (dk, x["q"])):
        assert (np.abs(got) <= b["scale"] * ds * np.abs(with_) * (1 + 2.0 ** -8) + tiny).all()


def test_infinite_product_at_a_dropped_score():
    """dO V^T overflows fp32 at one (query, key) pair that the mask drops: no gradient sees the infinity."""
    n, drop = 70, (0.5, 4711)
    b = wl.make_batch([n] + fill([64, 33, 120, 64], 250), 16, "bf16", seed=21)
    keep = dm.keep_masks(np.array([0, n], np.int32), 16, *drop)[0][0]
    q, k = next((q, k) for q in range(33, n - 1) for k in range(5, n) if not keep[q, k])
    for name in ("v", "do"):
        b[name][:n, 0, 0] = 0
    huge = wl.to_bits(np.array([2e20], np.float32), "bf16")[0]
    b["v"][k, 0, 0] = huge
    b["do"][q, 0, 0] = huge
    _, one, two = both_ways(b, drop)
    assert all(torch.isfinite(x).all() for x in one)
    compare(b, one, two, "bf16", drop)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_scaled_product_is_rounded_before_d_is_subtracted(dtype):
    """Single-token sequences with P = 1, dO V^T = 1.5, 1/(1-p) = 4/3 in fp32 (1.33333337), D = 2, among longer ones: the
    product rounds to 2 and a kept element's gradients are exactly zero; a dropped one has dS = -2."""
    p, seed, h = 0.25, 12, 16
    b = wl.make_batch(fill([1, 64, 1, 1], 800), h, dtype, seed=1)
    one = lambda x: wl.to_bits(np.array([x], np.float32), dtype)[0]
    for name, column, value in (("q", 1, 64.0), ("k", 0, 64.0), ("v", 0, 1.5), ("do", 0, 1.0)):
        b[name][:] = 0
        b[name][:, :, column] = one(value)
    b["scale"] = 0.5
    db = DeviceBatch(b, True)
    db.o.zero_()
    db.o[:, :, 0] = 2.0
    db.lse.zero_()                    # the one score is q k = 0, so P = 1
    db.bwd(dropout=(p, seed))
    torch.cuda.synchronize()
    rows = b["cu_seqlens"][:-1][b["lengths"] == 1]
    keep = np.stack([dm.random_bytes(int(r), h, 1, 1, seed)[:, 0, 0] >= dm.threshold(p) for r in rows])
    assert 0 < keep.sum() < keep.size
    dq, dk = to_f64(db.dq)[rows], to_f64(db.dk)[rows]
    assert np.array_equal(dq[:, :, 0], np.where(keep, 0.0, -64.0)) and (dq[:, :, 1:] == 0).all()
    assert np.array_equal(dk[:, :, 1], np.where(keep, 0.0, -64.0)) and (dk[:, :, 0] == 0).all() and (dk[:, :, 2:] == 0).all()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("batch,length,heads,dropout", [
    (16, 2048, 16, None),            # eight sweeps, and the whole of the buffer for dQ between them
    (48, 512, 16, (0.1, 5)),
    (64, 512, 4, None),              # one item for every workgroup
])
def test_equal_lengths(batch, length, heads, dropout, dtype):
    b = wl.make_batch([length] * batch, heads, dtype, seed=length)
    _, one, two = both_ways(b, dropout)
    compare(b, one, two, dtype, dropout)
    if dropout is None:              # one sequence, two heads of it
        rows = slice(length, 2 * length)
        x = {n: v[rows, :2] for n, v in oracle_inputs(b).items() if n in ("q", "k", "v", "do")}
        cu = wl.cu_from_lengths(np.array([length]))
        for name, got, want in zip(("dq", "dk", "dv"), one, oracle.bwd(x["q"], x["k"], x["v"], x["do"], cu, b["scale"])):
            rel, fro = gradient_errors(to_f64(got[rows, :2]), want, cu)
            assert rel <= G_TOL and fro <= G_TOL, f"{name}: {rel:.3e} {fro:.3e}"


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("lengths,heads,dropout", [
    ([2100, 4096, 2049], 16, None),   # keep the two passes: more rows than the buffer for dQ between sweeps holds
    ([2100, 2300], 16, (0.1, 3)),
])
def test_more_rows_than_the_buffer_holds(lengths, heads, dropout, dtype):
    """Against the one pass, which a longest sequence stated too small (512) sends the same batch to."""
    b = wl.make_batch(fill(lengths, 12), heads, dtype, seed=5)
    db = DeviceBatch(b, True)
    assert fmha.fmha_varlen_bwd_passes(b["batch"], b["total_tokens"], heads, b["max_seqlen"], dropout=dropout) == 2
    db.fwd(dropout=dropout)
    db.bwd(reuse_schedule=True, dropout=dropout)
    two = [x.clone() for x in (db.dq, db.dk, db.dv)]
    b["max_seqlen"] = 512
    assert fmha.fmha_varlen_bwd_passes(b["batch"], b["total_tokens"], heads, 512, dropout=dropout) == 1
    for x in (db.dq, db.dk, db.dv):
        x.fill_(float("nan"))
    db.bwd(reuse_schedule=True, dropout=dropout)
    torch.cuda.synchronize()
    compare(b, [db.dq, db.dk, db.dv], two, dtype, dropout)


@pytest.mark.parametrize("dropout", [None, (0.1, 5)])
def test_workspace_without_the_buffer_for_dq(dropout):
    """A backward in the smallest workspace runs as the two passes do, and writes nothing behind it."""
    b = wl.make_batch(fill(LONG, 110), 16, "f16", seed=6)
    db, _, two = both_ways(b, dropout)
    two = [x.clone() for x in two]
    t = b["total_tokens"]
    least = fmha.fmha_varlen_workspace_size(b["batch"], t, 16, False) + 2 * ((4 * (t * 16 + 1) + 255) // 256 * 256)
    whole = db.ws
    whole.fill_(0x5A)
    db.ws = whole[:least]
    for x in (db.dq, db.dk, db.dv):
        x.fill_(float("nan"))
    db.bwd(dropout=dropout)
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip((db.dq, db.dk, db.dv), two))
    assert (whole[least:] == 0x5A).all()
