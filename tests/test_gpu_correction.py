"""GPU parity of the linear correction over the ways in which its workgroups are filled: 1 to 8 query heads per kv head (fewer
than 4 share their channels out among the waves, more than 4 are two head blocks), numbers of sequences around the 1, 2, 4 and 8
that a workgroup serves (one and two sequences are shared by the waves, of more every wave takes whole ones).  Short contexts and
small queries, so that the correction is a large part of the result."""
import numpy as np
import pytest

import kvlinc_synth as synth
from tests import kvlinc_testlib as tl
from tests.test_decode_splits import launch_of

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kv():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2510_05373_amd as kvmod
    return kvmod


def _check(kv, B, H_kv, gq, bits, pairs, n=150, sliding=False, bound=0, seqs=None):
    from oracle import attention as o_attn
    from oracle import kvcache as o_cache
    H_q = H_kv * gq
    if seqs is not None:
        capacity = 128 * -(-max(n + 128, bound) // 128) + 128
        assert launch_of(B, H_q, H_kv, bound or capacity, bits=bits, flags=kv.KVLINC_FLAG_SLIDING_VALUES if sliding else 0).corr_seqs == seqs
    K, V = tl.gen_kv(95, B, H_kv, [n] * B)
    q = (np.random.default_rng(95).standard_normal((B, H_q, 128)) * 0.05).astype(np.float16)
    Wq, Wk = synth.adapters_q(95, H_q), synth.adapters_k(95, H_kv)
    Wq = (Wq.astype(np.float32) * 64.0).astype(np.float16)  # peaked feature maps, of small queries too
    Wk = (Wk.astype(np.float32) * (8.0 if bits == 2 else 40.0)).astype(np.float16)  # (the key error is a fifth at 4 bits)
    cache = kv.KVLincCache(B, H_q, H_kv, max(n + 128, bound), Wq=tl.to_dev(Wq), Wk=tl.to_dev(Wk), bits=bits,
                           flags=kv.KVLINC_FLAG_SLIDING_VALUES if sliding else 0)
    cache.append(tl.to_dev(K), tl.to_dev(V))
    got = [cache.decode(tl.to_dev(q), max_context=bound).cpu().numpy() for _ in range(2)]
    assert np.array_equal(tl.u16(got[0]), tl.u16(got[1]))
    assert int(cache.split_done.abs().sum().item()) == 0
    nq = int(cache.n_quant[0].item())
    assert nq == (n - 1) // 128 * 128
    want = {}
    window = "sliding" if sliding else "block"
    for b, g in pairs:
        ref = o_cache.build_cache(K[b, g], V[b, g], nq, Wk=Wk[g], bits=bits)
        for h in range(g * gq, (g + 1) * gq):
            want[b, h] = o_attn.decode(q[b, h], ref, Wq[h], value_window=window)
    tl.check_outputs(got[0], want)
    # the correction is five times what the tolerance lets pass, or more
    without = {k: o_attn.decode(q[k[0], k[1]], o_cache.build_cache(K[k[0], k[1] // gq], V[k[0], k[1] // gq], nq, Wk=None, bits=bits), None, value_window=window) for k in list(want)[:1]}
    for k, y in without.items():
        assert np.linalg.norm(y - want[k]) > 5 * tl.OUT_REL_L2 * np.linalg.norm(want[k])


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("gq", [1, 2, 3, 4, 5, 7, 8])
@pytest.mark.parametrize("B,H_kv", [(1, 1), (3, 2), (4, 1), (5, 3), (9, 1)])
def test_heads_and_sequences(kv, B, H_kv, gq, bits):
    _check(kv, B, H_kv, gq, bits, [(b, g) for b in range(B) for g in range(H_kv)], seqs=2)


# 4 sequences a workgroup, and 1, 2 and 3 in the last one
@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("gq", [1, 2, 3, 4, 5, 7, 8])
@pytest.mark.parametrize("B", [13, 14, 15, 16])
def test_four_sequences(kv, B, gq, bits):
    _check(kv, B, 16, gq, bits, sorted({(b, g) for b in (0, 3, 4, 12, B - 1) for g in (0, 15)}), seqs=4)


# two splits: one sequence a workgroup, and two (one in the last, and none left over)
@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("gq", [1, 2, 3, 4, 5, 7, 8])
@pytest.mark.parametrize("B,H_kv,seqs", [(1, 2, 1), (3, 2, 1), (5, 8, 1), (5, 9, 2), (6, 8, 2)])
def test_one_and_two_sequences_of_two_splits(kv, B, H_kv, seqs, gq, bits):
    _check(kv, B, H_kv, gq, bits, sorted({(b, g) for b in (0, B // 2, B - 1) for g in (0, H_kv - 1)}), n=690, seqs=seqs)


@pytest.mark.parametrize("B,H_kv", [(12, 64), (13, 64), (16, 64), (17, 64)])  # 8 sequences a workgroup from 13 on
def test_many_single_heads(kv, B, H_kv):
    _check(kv, B, H_kv, 1, 2, sorted({(b, g) for b in (0, 3, 4, 7, 8, 11, B - 1) for g in (0, 31, 63)}))


@pytest.mark.parametrize("bits,sliding", [(4, False), (2, True), (4, True)])
@pytest.mark.parametrize("B", [13, 16, 17])
def test_many_single_heads_of_the_variants(kv, B, bits, sliding):
    _check(kv, B, 64, 1, bits, sorted({(b, g) for b in (0, 4, 7, 8, B - 1) for g in (0, 63)}), sliding=sliding)


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("gq", [1, 2, 3, 5])
def test_sliding_values(kv, gq, bits):
    _check(kv, 5, 2, gq, bits, [(b, g) for b in (0, 3, 4) for g in (0, 1)], sliding=True)


# 8 sequences a workgroup where workgroups of 4 do not fit the chip at once (of a bound of 12 groups or more: the sequences are short)
@pytest.mark.parametrize("sliding", [False, True])
@pytest.mark.parametrize("gq", [1, 2])
@pytest.mark.parametrize("B,H_kv", [(5, 64), (8, 64), (13, 32), (27, 16), (53, 8)])
def test_eight_sequences_where_four_do_not_fit(kv, B, H_kv, gq, sliding):
    _check(kv, B, H_kv, gq, 2, sorted({(b, g) for b in (0, min(3, B - 1), 4, min(7, B - 1), min(8, B - 1), B - 1) for g in (0, H_kv - 1)}), sliding=sliding, bound=1500)
