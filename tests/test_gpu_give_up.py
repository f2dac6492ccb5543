"""GPU parity of decodes whose streaming workgroups do not get to wait for the correction: the library built with no looks at the
counter, in which every wait runs out at once.  A single split then writes the result it has kept to memory after all, and the
correction workgroup that arrives last merges.  Against the ordinary library (same bits) and the oracle."""
import ctypes

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


@pytest.fixture(scope="module")
def no_looks(kv):
    from paper_2510_05373_amd import build
    f = ctypes.CDLL(build.NOLOOKS_PATH).kvlinc_decode_attention
    f.restype, f.argtypes = ctypes.c_int, kv.binding.lib.kvlinc_decode_attention.argtypes
    return f


# (sequences, kv heads, heads per kv head, longest context, sequences of a correction workgroup, splits): one split and several -- up
# to 4 and 12 (merge_pair, merge_row) and more --, one head block and two, workgroups of 2 and 4 sequences, whole and ragged.
@pytest.mark.parametrize("bits,sliding", [(2, False), (4, False), (2, True)])
@pytest.mark.parametrize("B,H_kv,gq,n,seqs,splits", [
    (1, 1, 4, 150, 2, 1), (3, 2, 7, 300, 2, 1), (5, 3, 1, 150, 2, 1), (7, 16, 4, 300, 4, 1), (7, 16, 8, 300, 4, 1), (27, 4, 2, 300, 4, 1),
    (24, 2, 2, 1500, 2, 3), (13, 2, 7, 3000, 2, 6), (3, 16, 3, 1500, 4, 3), (13, 4, 8, 1500, 4, 3), (12, 1, 4, 9000, 2, 18)])
def test_every_wait_runs_out(kv, no_looks, B, H_kv, gq, n, seqs, splits, bits, sliding):
    import torch
    H_q = H_kv * gq
    over = dict(bits=bits, flags=kv.KVLINC_FLAG_SLIDING_VALUES if sliding else 0)
    l = launch_of(B, H_q, H_kv, n, **over)
    assert (l.awaited, l.corr_seqs, l.avg) == (1, seqs, splits)
    lengths = [n] + [n - (17 * b) % (n // 2) for b in range(1, B)]
    lengths[-1] = n if B < 3 else 100  # (no group yet: nothing to add)
    K, V = tl.gen_kv(89, B, H_kv, lengths)
    q = tl.gen_q(89, B, H_q)
    Wq, Wk = synth.adapters_q(89, H_q), synth.adapters_k(89, H_kv)
    cache = kv.KVLincCache(B, H_q, H_kv, n + 128, Wq=tl.to_dev(Wq), Wk=tl.to_dev(Wk), **over)
    cache.append(tl.to_dev(K), tl.to_dev(V), n_new=tl.to_dev(np.asarray(lengths, dtype=np.int32)))
    qd = tl.to_dev(q)
    want = cache.decode(qd, max_context=n)
    ws = cache.workspace(n)
    stream = torch.cuda.current_stream().cuda_stream
    for _ in range(8):
        got = torch.full_like(qd, float("nan"))
        assert no_looks(ctypes.byref(cache.struct), qd.data_ptr(), got.data_ptr(), ws.data_ptr(), ws.numel() * 4, n, stream) == 0
        torch.cuda.synchronize()
        assert not cache.split_done.any()
        assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    if not sliding:
        pairs = sorted({(0, 0), (B - 1, H_kv - 1), (B // 2, 0)})
        tl.check_outputs(got.cpu().numpy(), tl.oracle_decode(K, V, q, lengths, cache.n_quant.cpu().numpy(), pairs, H_q, H_kv, Wq, Wk, bits))
