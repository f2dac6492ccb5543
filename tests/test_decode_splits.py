"""Launch policy of the decode on the host: sizes and orders that the kernel's merge and its workgroups rely on.  No launch is made."""
import ctypes

import pytest

from tests.test_library_abi import fake_struct, kb

SPLITS_OF_THE_MERGE = 32  # rows of partial results that the merge of a query head holds


def most_splits(c, context):
    """The most splits a sequence may take, from the workspace: B * H_q * (splits + 4 correction parts) rows of 132 floats."""
    per_row, rest = divmod(kb.kvlinc_decode_workspace_bytes(c, context), c.B * c.H_q * 132 * 4)
    assert rest == 0
    return per_row - 4


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("corr", [True, False])
def test_no_sequence_takes_more_splits_than_the_merge_holds(bits, corr):
    off = {} if corr else dict(S=0, S16=0, P=0, Wq=0, Wk=0)
    for H_kv in (1, 2, 3, 4, 5, 6, 7, 8, 16, 32):
        for gq in range(1, 9):
            for B in list(range(1, 41)) + [64, 144, 257]:
                c = fake_struct(B=B, H_q=H_kv * gq, H_kv=H_kv, bits=bits, max_groups=1025, **off)
                for context in (1, 128, 700, 1281, 4096, 9000, 17000, 20000, 32768, 70000, 131072):
                    splits = most_splits(c, context)
                    assert 1 <= splits <= SPLITS_OF_THE_MERGE, (B, H_kv, gq, context, splits)


class Splits(ctypes.Structure):
    _fields_ = [("avg", ctypes.c_int), ("most", ctypes.c_int), ("corr_first", ctypes.c_int), ("corr_seqs", ctypes.c_int)]


def splits_of(B, H_q, H_kv, context, **over):
    """The launch policy itself: an internal function of the library, by its symbol."""
    f = kb.lib._ZN6kvlinc13decode_splitsERK12kvlinc_cachei
    f.restype, f.argtypes = Splits, [ctypes.POINTER(kb.CacheStruct), ctypes.c_int]
    c = fake_struct(B=B, H_q=H_q, H_kv=H_kv, max_groups=1025, **over)
    s = f(ctypes.byref(c), context)
    assert s.most == most_splits(c, context)
    return s


@pytest.mark.parametrize("gq", range(1, 9))
def test_the_correction_leads_short_contexts(gq):
    """Its chain is the longest part of a launch over short contexts: it must not start behind the streaming workgroups there,
    whatever the number of sequences and heads."""
    for H_kv in (1, 2, 4, 8, 16, 32):
        for B in range(2, 65):
            for context in (1, 140, 300, 512):
                s = splits_of(B, H_kv * gq, H_kv, context)
                assert s.avg == 1 and s.corr_first >= 1, (B, H_kv, context)


@pytest.mark.parametrize("B,H_q,H_kv,context,first", [
    (24, 32, 8, 500, 1), (32, 32, 8, 1000, 1), (32, 32, 8, 1500, 1), (32, 32, 8, 4000, 0), (16, 16, 16, 1000, 1), (8, 32, 32, 4000, 1),  # one split
    (5, 16, 16, 1000, 0), (8, 16, 16, 1000, 0), (16, 32, 8, 1000, 1), (12, 64, 8, 1000, 2), (17, 28, 4, 1400, 2),  # two and three
    (8, 32, 8, 1800, 0), (12, 28, 4, 2500, 0), (4, 64, 8, 4000, 0), (2, 32, 8, 8000, 0)])
def test_order_between_one_and_two_workgroups_per_unit(B, H_q, H_kv, context, first):
    """First (1), on compute units of its own (2) or last (0), from one, two, four splits of a sequence on."""
    assert splits_of(B, H_q, H_kv, context).corr_first == first
    if first == 0 and context >= 1800:  # a compute unit holds two workgroups at 4 bits: never last beside so few
        assert splits_of(B, H_q, H_kv, context, bits=4).corr_first >= 1


def test_a_single_sequence_leads_with_the_correction():
    for context in (1, 300, 5000, 131072):
        assert splits_of(1, 32, 8, context).corr_first >= 1


@pytest.mark.parametrize("B,H_q,H_kv,bits,seqs", [
    (12, 32, 32, 2, 4), (13, 32, 32, 2, 8), (16, 32, 32, 2, 8), (17, 32, 32, 2, 4), (8, 64, 64, 2, 8), (8, 128, 64, 2, 8), (53, 16, 8, 2, 8),  # 768 places
    (8, 192, 64, 2, 4), (13, 32, 32, 4, 4), (32, 32, 32, 2, 8), (32, 32, 32, 4, 8), (28, 32, 32, 2, 4), (32, 64, 32, 2, 4)])
def test_sequences_of_a_correction_workgroup(B, H_q, H_kv, bits, seqs):
    for context in (1500, 8064):
        assert splits_of(B, H_q, H_kv, context, bits=bits).corr_seqs == seqs
    if B * H_kv < 1000:
        for context in (300, 1408, 8065, 131072):
            assert splits_of(B, H_q, H_kv, context, bits=bits).corr_seqs == 4


@pytest.mark.parametrize("B,H_q,H_kv,context,bits,seqs", [
    (1, 4, 1, 300, 2, 2), (9, 32, 8, 300, 2, 2), (7, 64, 16, 300, 2, 4), (16, 32, 8, 300, 2, 4),  # one split: 2 where all have a unit of their own
    (1, 32, 8, 131072, 2, 1), (5, 32, 8, 818, 2, 1), (6, 32, 8, 818, 2, 2), (16, 32, 8, 8320, 2, 4), (9, 64, 8, 2875, 2, 1),  # several, up to three a unit
    (16, 32, 8, 8320, 4, 4), (5, 64, 16, 818, 2, 1), (5, 64, 16, 818, 4, 2)])  # two a unit at 4 bits: never 1 there
def test_few_sequences_of_a_correction_workgroup(B, H_q, H_kv, context, bits, seqs):
    assert splits_of(B, H_q, H_kv, context, bits=bits).corr_seqs == seqs


class Launch(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("avg", "splits", "corr_seqs", "corr_first", "awaited", "workgroups", "skip")]


def launch_of(B, H_q, H_kv, context, **over):
    f = kb.lib._ZN6kvlinc13decode_launchERK12kvlinc_cachei
    f.restype, f.argtypes = Launch, [ctypes.POINTER(kb.CacheStruct), ctypes.c_int]
    return f(ctypes.byref(fake_struct(B=B, H_q=H_q, H_kv=H_kv, max_groups=1025, **over)), context)


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("gq", [1, 2, 4, 7])
def test_the_correction_is_awaited_only_where_all_of_it_goes_first(gq, bits):
    """Streaming workgroups that wait for correction workgroups behind them in the grid hold the places that these need as soon as
    another stream's launch shares the chip."""
    seen = set()
    for H_kv in (1, 2, 3, 4, 8, 16, 32):
        for B in list(range(1, 41)) + [64, 144]:
            for context in (1, 300, 500, 1281, 4096, 9000, 20000, 131072):
                l = launch_of(B, H_kv * gq, H_kv, context, bits=bits)
                s = splits_of(B, H_kv * gq, H_kv, context, bits=bits)
                n_corr = H_kv * 4 * -(-B // s.corr_seqs)
                assert (l.avg, l.corr_seqs) == (s.avg, s.corr_seqs) and l.workgroups == B * H_kv * l.splits + n_corr and l.splits in (1, s.most)
                assert not l.awaited or l.corr_first == 1, (B, H_kv, context)
                # (a correction workgroup of one sequence has no more to merge than the streaming workgroup that would wait for it)
                assert not l.awaited or l.avg == 1 or min(l.corr_seqs, B) > 1, (B, H_kv, context)
                seen.add((l.corr_first, l.awaited))
    assert {(1, 1), (2, 0)} <= seen and (bits == 4 or (0, 0) in seen)


@pytest.mark.parametrize("bits", [2, 4])
def test_rounds_that_split_0_sits_out(bits):
    """One where two would make a context of the bound itself a round longer, for the splits that such a sequence takes."""
    seen = set()
    for B, H_kv, gq in ((1, 8, 4), (2, 1, 1), (16, 8, 4), (15, 8, 1), (32, 4, 7), (40, 8, 4), (144, 8, 4)):
        for context in range(1, 12000, 127):
            l = launch_of(B, H_kv * gq, H_kv, context, bits=bits)
            groups = -(-max(context, 1) // 128) - 1
            n = min(l.avg, -(-groups // 4))
            longer = n > 1 and -(-(groups + 8) // (4 * n)) > -(-(groups + 4) // (4 * n))
            assert l.skip == (1 if bits == 4 or longer else 2), (B, H_kv, gq, context)
            seen.add(l.skip)
    assert seen == ({1} if bits == 4 else {1, 2})


@pytest.mark.parametrize("bits,sliding,held", [(2, False, 3), (4, False, 2), (2, True, 3), (4, True, 2)])
def test_small_correction_workgroups_only_where_all_workgroups_fit_the_chip(bits, sliding, held):
    """`held`: workgroups that a compute unit holds; the kernel of the sliding window for more than 4 heads holds two."""
    seen = set()
    for gq in (1, 2, 4, 5, 8):
        places = 256 * (2 if sliding and gq > 4 else held)
        for H_kv in (1, 2, 3, 4, 8, 16, 32):
            for B in list(range(1, 41)) + [64, 144]:
                for context in (1, 300, 900, 1500, 3000, 4500, 9000, 20000):
                    s = splits_of(B, H_kv * gq, H_kv, context, bits=bits, flags=kb.KVLINC_FLAG_SLIDING_VALUES if sliding else 0)
                    seen.add(s.corr_seqs)
                    if s.corr_seqs < 4:
                        assert B * H_kv * s.avg + H_kv * 4 * -(-B // s.corr_seqs) <= places, (B, H_kv, gq, context)
    assert {1, 2, 4} <= seen


@pytest.mark.parametrize("bits", [2, 4])
def test_two_runs_lead_only_where_units_are_shared(bits):
    seen = set()
    for gq in (1, 2, 4, 7):
        for H_kv in (1, 2, 3, 4, 8, 16, 32):
            for B in list(range(1, 41)) + [64, 144]:
                for context in (300, 900, 1500, 3000, 4500, 9000, 20000, 131072):
                    s = splits_of(B, H_kv * gq, H_kv, context, bits=bits)
                    seen.add(s.corr_first)
                    assert s.corr_first < 2 or B * H_kv * s.avg + H_kv * 4 * -(-B // 4) > 256, (B, H_kv, gq, context)
    assert {1, 2} <= seen
