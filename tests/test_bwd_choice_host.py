"""Which batches the backward takes in one pass: what was measured to lose by it keeps the two passes.
(Sizes alone decide, so this needs no GPU.)"""
import os

import pytest

from paper_2208_08124_amd import fmha

pytestmark = pytest.mark.skipif(not os.path.exists(fmha.LIB_PATH), reason="library not built (run __graft_entry__.build())")

DROP = (0.1, 7)


def passes(batch, mean, heads, longest, **kw):
    return fmha.fmha_varlen_bwd_passes(batch, int(batch * mean), heads, longest, **kw)


@pytest.mark.parametrize("dropout", [None, DROP])
@pytest.mark.parametrize("batch,mean,heads,longest,want", [
    (56, 281, 16, 512, 1), (256, 110, 16, 512, 1), (2048, 257, 12, 512, 1), (16, 2048, 16, 2048, 1),
    # more rows than the fp32 dQ between sweeps has room for
    (16, 2049, 16, 2049, 2), (16, 4096, 16, 4096, 2), (16, 8192, 16, 8192, 2), (64, 2100, 16, 4096, 2),
    (1, 2048, 256, 1 << 20, 1),                   # (rows that the tensors do not have need no room)
    (34, 610, 16, 1024, 2), (33, 466, 16, 768, 2),   # 0.81 and 0.90 of the two passes' speed
    (25, 260, 16, 260, 2), (262, 289, 4, 289, 2),    # few keys in a second sweep, in more than one round
    (67, 1228, 3, 1291, 2),                         # 0.93, rounds 0.79 full
    (1000, 48, 1, 512, 2), (500, 60, 2, 1024, 2),    # few heads and short sequences, whatever the longest is stated to be
    (1226, 75, 3, 295, None),                       # 0.91 without dropout, 0.98 with
])
def test_choice(batch, mean, heads, longest, want, dropout):
    if want is None:
        if dropout:
            return
        want = 2
    assert passes(batch, mean, heads, longest, dropout=dropout) == want


@pytest.mark.parametrize("dropout", [None, DROP])
@pytest.mark.parametrize("batch,rows,heads,longest,want", [
    (1413, 64, 8, 64, 2), (329, 44, 8, 176, 2), (1250, 80, 16, 80, 2), (196, 96, 12, 96, 2), (600, 128, 16, 128, 2),
    (340, 168, 4, 168, 1), (2048, 512, 12, 512, 1),
    (8, 1024, 3, 1024, 2), (67, 889, 5, 889, 2), (411, 330, 2, 330, 2),
])
def test_choice_with_key_counts(batch, rows, heads, longest, want, dropout):
    """With seqused every sequence is taken one head at a time: rows of up to 128 tokens leave most key places empty."""
    assert passes(batch, rows, heads, longest, dropout=dropout, seqused=True) == want


def test_halves_by_themselves_and_an_unknown_longest_sequence_take_two():
    assert passes(256, 512, 16, 512) == 1
    assert passes(256, 512, 16, 0) == 2
    for only in ("dq", "dkv"):
        assert passes(256, 512, 16, 512, only=only) == 2
    with pytest.raises(fmha.FmhaError):
        passes(256, 512, 16, 512, dropout=(1.5, 0))
    with pytest.raises(fmha.FmhaError):
        passes(256, 512, 16, 512, workspace_bytes=4096)


def without_dq_buffer(batch, total_tokens, heads):
    stats = (4 * (total_tokens * heads + 1) + 255) // 256 * 256
    return fmha.fmha_varlen_workspace_size(batch, total_tokens, heads, False) + 2 * stats


@pytest.mark.parametrize("batch,mean,heads,longest", [(56, 281, 16, 512), (256, 200, 16, 256), (16, 2048, 16, 2048),
                                                      (3, 20, 5, 64)])
def test_workspace_without_the_buffer_for_dq(batch, mean, heads, longest):
    """The two passes use no fp32 dQ between sweeps: they run in a workspace without it."""
    least, full = without_dq_buffer(batch, batch * mean, heads), fmha.fmha_varlen_workspace_size(batch, batch * mean, heads, True)
    want = passes(batch, mean, heads, longest)
    assert passes(batch, mean, heads, longest, workspace_bytes=full) == want
    assert passes(batch, mean, heads, longest, workspace_bytes=full + (1 << 30)) == want
    assert passes(batch, mean, heads, longest, workspace_bytes=least) == 2
    for kw in (dict(only="dq"), dict(only="dkv"), dict(dropout=DROP)):
        assert passes(batch, mean, heads, longest, workspace_bytes=least, **kw) == 2
    assert passes(batch, mean, heads, 0, workspace_bytes=least) == 2
    with pytest.raises(fmha.FmhaError):
        passes(batch, mean, heads, longest, workspace_bytes=least - 1)
