"""GPU parity where logits are so large (1e6 to 1e13) that one unit in their last place is more than a softmax can tell apart:
any finite keys and queries have to give finite outputs, and where the answer does not hang on such a unit -- all tokens alike,
or one far ahead -- the right ones; likewise for the feature maps under large adapters."""
import numpy as np
import pytest

import kvlinc_synth as synth
from tests import kvlinc_testlib as tl

pytestmark = pytest.mark.gpu

# query heads per kv head, code width, sliding value window
FORMS = [(4, 2, False), (7, 2, False), (4, 4, False), (8, 4, False), (4, 2, True), (7, 4, True), (1, 2, False)]


@pytest.fixture(scope="module")
def kv():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2510_05373_amd as kvmod
    return kvmod


def _decode_and_check(kv, K, V, q, bits, sliding, keep=0):
    import torch
    n, H_q = K.shape[2], q.shape[1]
    Wq, Wk = synth.adapters_q(81, H_q), (synth.adapters_k(81, 1).astype(np.float32) * 2.0 ** -10).astype(np.float16)
    R = 32 if keep else 128
    cache = kv.KVLincCache(1, H_q, 1, n + 128, R=R, Wq=tl.to_dev(Wq), Wk=tl.to_dev(Wk), bits=bits,
                           flags=kv.KVLINC_FLAG_SLIDING_VALUES if sliding else 0)
    cache.append(tl.to_dev(K), tl.to_dev(V), keep_residual=keep)
    got = cache.decode(tl.to_dev(q)).cpu().numpy()
    assert int(cache.status.item()) == 0 and np.isfinite(got.astype(np.float32)).all()
    from oracle import attention as o_attn
    from oracle import kvcache as o_cache
    ref = o_cache.build_cache(K[0, 0], V[0, 0], int(cache.n_quant.item()), Wk=Wk[0], bits=bits)
    want = {(0, h): o_attn.decode(q[0, h], ref, Wq[h], value_window="sliding" if sliding else "block") for h in range(H_q)}
    tl.check_outputs(got, want)


# (Keys and queries of at most 8 significant bits: the products and all their partial sums are exact in binary32, so the
# window's logits and the quantized tokens' are the same number.)
@pytest.mark.parametrize("gq,bits,sliding", FORMS)
@pytest.mark.parametrize("k,q", [(128.0, 96.0), (1024.0, 8192.0), (20480.0, 20480.0), (-24576.0, 24576.0), (61440.0, 61440.0), (-65280.0, 65280.0)])
def test_all_tokens_alike(kv, gq, bits, sliding, k, q):
    n = 700
    _, V = tl.gen_kv(82, 1, 1, [n])
    _decode_and_check(kv, np.full((1, 1, n, 128), k, dtype=np.float16), V, np.full((1, gq, 128), q, dtype=np.float16), bits, sliding)


# The winner is ahead by a tenth of a logit of up to 4.5e10, which is 400 times what binary16 mid-points and operands of three
# terms leave (2^-12 of it); where: in a group that is walked early, in the newest one, in the window.
@pytest.mark.parametrize("gq,bits,sliding", FORMS)
@pytest.mark.parametrize("gain", [300.0, 4000.0, 20000.0, 55000.0])
@pytest.mark.parametrize("where", [3, 130, 639, 700])
def test_one_token_far_ahead(kv, gq, bits, sliding, gain, where):
    n = 720
    r = np.random.default_rng(83)
    _, V = tl.gen_kv(83, 1, 1, [n])
    K = gain * (1.0 + 0.003 * r.standard_normal((1, 1, n, 128)))
    K[0, 0, where] *= 1.1
    q = gain * (1.0 + 0.003 * r.standard_normal((1, gq, 128)))
    _decode_and_check(kv, K.astype(np.float16), V, q.astype(np.float16), bits, sliding)


def test_one_token_far_ahead_of_a_partial_group(kv):
    r = np.random.default_rng(84)
    n = 450
    _, V = tl.gen_kv(84, 1, 1, [n])
    K = 30000.0 * (1.0 + 0.003 * r.standard_normal((1, 1, n, 128)))
    K[0, 0, 400] *= 1.1
    q = 30000.0 * (1.0 + 0.003 * r.standard_normal((1, 4, 128)))
    _decode_and_check(kv, K.astype(np.float16), V, q.astype(np.float16), 2, False, keep=20)


# Every logit that counts is 0, the sum of a huge centre (zero-points and mid-points of 64 channels) and codes that cancel it;
# a few tokens with one large key each lie far below.  Steps and mid-points are exact in binary16.
@pytest.mark.parametrize("gq,bits,sliding", FORMS)
@pytest.mark.parametrize("step", [2.0 ** 4, 2.0 ** 8, 2.0 ** 11])
def test_large_centres_that_cancel(kv, gq, bits, sliding, step):
    n, levels = 500, 2 ** bits - 1
    _, V = tl.gen_kv(85, 1, 1, [n])
    K = np.zeros((1, 1, n, 128), dtype=np.float16)
    for group in range(3):
        for c in range(64):
            K[0, 0, 128 * group + c, c] = levels * step
    _decode_and_check(kv, K, V, np.full((1, gq, 128), -32768.0, dtype=np.float16), bits, sliding)


# Key errors of up to half a step (1e4) times adapters of up to 6e4: logits of 1e9 to 1e10, of which the largest is ahead of the
# next by far more than one unit in its last place (256 to 1024), so that phi is 1 for one feature of each half.
@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("one_by_one", [False, True])
def test_feature_maps_under_large_adapters(kv, bits, one_by_one):
    n = 300
    r = np.random.default_rng(86)
    K = r.uniform(-60000.0, 60000.0, (1, 1, n, 128)).astype(np.float16)
    _, V = tl.gen_kv(86, 1, 1, [n])
    Wk = r.uniform(-60000.0, 60000.0, (1, 2, 128, 128)).astype(np.float16)
    cache = kv.KVLincCache(1, 4, 1, 512, Wq=tl.to_dev(synth.adapters_q(86, 4)), Wk=tl.to_dev(Wk), bits=bits)
    for t in range(n) if one_by_one else (slice(0, n),):
        rows = slice(t, t + 1) if one_by_one else t
        cache.append(tl.to_dev(K[:, :, rows]), tl.to_dev(V[:, :, rows]))
    assert int(cache.status.item()) == 0
    tl.check_cache_against_oracle(cache, K, V, [n], [(0, 0)], Wk=Wk)
