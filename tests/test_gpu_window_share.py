"""GPU parity of the decode's window part: numbers of window tokens around the shares of the four waves and their tiles (a share is a
multiple of 4 tokens, 32 at most; with one split, of the waves without a group in the last round), one split and several.
Slots behind the window hold large numbers, which must not show."""
import numpy as np
import pytest

import kvlinc_synth as synth
from tests import kvlinc_testlib as tl

pytestmark = pytest.mark.gpu

TOKENS = [1, 3, 4, 5, 15, 16, 17, 20, 33, 64, 65, 100, 113, 127, 128]


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("gq", [1, 4, 7])
@pytest.mark.parametrize("H_kv,groups", [(1, 0), (1, 1), (1, 2), (1, 3), (16, 1), (1, 17), (4, 17), (8, 18)])  # (8, 18): one round for the window (up to 4 heads)
def test_window_tokens(H_kv, groups, gq, bits):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2510_05373_amd as kv
    B, H_q = len(TOKENS), H_kv * gq
    lengths = [128 * groups + t for t in TOKENS]
    K, V = tl.gen_kv(98, B, H_kv, lengths)
    q = tl.gen_q(98, B, H_q)
    Wq, Wk = synth.adapters_q(98, H_q), synth.adapters_k(98, H_kv)
    cache = kv.KVLincCache(B, H_q, H_kv, max(lengths) + 128, Wq=tl.to_dev(Wq), Wk=tl.to_dev(Wk), bits=bits)
    cache.append(tl.to_dev(K), tl.to_dev(V), n_new=tl.to_dev(np.asarray(lengths, dtype=np.int32)))
    n_quant, n_res = tl.check_counters(cache, lengths)
    for b in range(B):
        nr = int(n_res[b])
        cache.k_res[b, :, nr:] = 60000.0
        window = cache.v_res[b].permute(0, 1, 3, 2).reshape(H_kv, 128, 128).clone()  # [head][slot][channel]
        window[:, nr:] = 60000.0
        cache.v_res[b] = window.reshape(H_kv, 32, 4, 128).permute(0, 1, 3, 2)
    got = cache.decode(tl.to_dev(q), max_context=max(lengths)).cpu().numpy()
    pairs = [(b, H_kv - 1) for b in range(B)]
    tl.check_outputs(got, tl.oracle_decode(K, V, q, lengths, n_quant, pairs, H_q, H_kv, Wq, Wk, bits))
    assert int(cache.split_done.abs().sum().item()) == 0
