"""GPU parity where every logit of a row lies far below zero: 2^M, M the largest one in the log2 domain, leaves the normal range of
binary32 at -87.3 and all of it at -103.3, but a softmax with nothing added does not hang on it, nor does one to which the
correction adds as little."""
import numpy as np
import pytest

import kvlinc_synth as synth
from tests import kvlinc_testlib as tl

pytestmark = pytest.mark.gpu

# All keys alike, all queries 2: the logits are -128 * 2 / sqrt(128) times these, -79 to -996, without a rounding.
KEYS = [3.5, 3.875, 3.96875, 4.25, 4.5, 4.875, 44.0]
# One split (1 and 128 tokens: of a sequence without a group; 300), two and three, six
TOKENS = [1, 128, 300, 700, 1300, 3000]
FORMS = [(4, 2, False), (7, 2, False), (1, 2, False), (4, 4, False), (8, 4, False), (5, 2, True)]  # heads per kv head, bits, sliding


def _decode(n, key, gq, bits, sliding, corr, P0=None):
    """(cache, V, output) of n alike tokens; P0: what P holds instead of its sums, with S = 0."""
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2510_05373_amd as kv
    _, V = tl.gen_kv(88, 1, 1, [n])
    K = np.full((1, 1, n, 128), -key, dtype=np.float16)
    q = np.full((1, gq, 128), 2.0, dtype=np.float16)
    Wq, Wk = (synth.adapters_q(88, gq), synth.adapters_k(88, 1)) if corr else (None, None)
    cache = kv.KVLincCache(1, gq, 1, n + 128, Wq=tl.to_dev(Wq) if corr else None, Wk=tl.to_dev(Wk) if corr else None, bits=bits,
                           flags=kv.KVLINC_FLAG_SLIDING_VALUES if sliding else 0)
    cache.append(tl.to_dev(K), tl.to_dev(V))
    if P0 is not None:
        cache.S16.zero_()
        cache.P.fill_(P0)
    got = cache.decode(tl.to_dev(q)).cpu().numpy()
    assert int(cache.status.item()) == 0 and not cache.split_done.any()
    return K, V, q, Wq, Wk, int(cache.n_quant.item()), got


def _oracle(K, V, q, nq, Wq, Wk, bits, sliding):
    from oracle import attention as o_attn
    from oracle import kvcache as o_cache
    ref = o_cache.build_cache(K[0, 0], V[0, 0], nq, Wk=None if Wk is None else Wk[0], bits=bits)
    return {(0, h): o_attn.decode(q[0, h], ref, None if Wq is None else Wq[h], value_window="sliding" if sliding else "block") for h in range(q.shape[1])}


@pytest.mark.parametrize("corr", [False, True])
@pytest.mark.parametrize("gq,bits,sliding", FORMS)
@pytest.mark.parametrize("n", TOKENS)
def test_logits_far_below_zero(n, gq, bits, sliding, corr):
    for key in KEYS:
        K, V, q, Wq, Wk, nq, got = _decode(n, key, gq, bits, sliding, corr)
        if nq == 0:  # (S = P = 0: nothing is added, and 0 / 0 is what Eq. 5 as written comes to)
            Wq = Wk = None
        tl.check_outputs(got, _oracle(K, V, q, nq, Wq, Wk, bits, sliding))


# P = P0 in every feature: C_d = 2 P0 (each half of phi sums to 1), S = 0: C_n = 0.  The softmax's result is then reduced to the part
# den / (den + 2 P0 2^-M) of it, den = the number of tokens.
@pytest.mark.parametrize("gq,bits", [(4, 2), (7, 2), (1, 4)])
@pytest.mark.parametrize("n", [300, 700, 3000])
@pytest.mark.parametrize("P0", [2.0 ** -20, 2.0 ** -100, 2.0 ** -130])
def test_a_correction_as_small_as_the_sum(n, gq, bits, P0):
    for key in KEYS[:-1]:
        K, V, q, _, _, nq, got = _decode(n, key, gq, bits, False, True, P0=P0)
        part = 1.0 / (1.0 + 2.0 * P0 * np.exp(256.0 * key / np.sqrt(128.0)) / n)
        want = {k: part * y for k, y in _oracle(K, V, q, nq, None, None, bits, False).items()}
        if part > 1e-2:  # (below, the fp16 output has too few digits for a relative comparison)
            tl.check_outputs(got, want)
        else:
            assert np.isfinite(got.astype(np.float32)).all()
            assert max(np.abs(got[0, h].astype(np.float64) - want[0, h]).max() for h in range(gq)) <= 1e-3 * max(1e-2, part)
