"""GPU parity of the several-row append at its edges: Eq. 1 where the binary32 decision is delicate, and the window's rows
at every way they can lie in the passes of 16 rows and the blocks of 4 slots."""
import numpy as np
import pytest

import kvlinc_synth as synth
from tests import kvlinc_testlib as tl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kv():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2510_05373_amd as kvmod
    return kvmod


def _delicate_columns(n, seed):
    """[n, 128] fp16 keys, every channel another kind of trouble for fl32(x - z) against (k + 0.5) s."""
    r = np.random.default_rng(seed)
    out = np.zeros((n, 128), dtype=np.float64)
    for c in range(128):
        kind = c % 8
        scale = 2.0 ** r.integers(-6, 10)
        if kind == 0:      # multiples of half a step: every value on a threshold or a level
            x = r.integers(0, 31, n) * 0.5 * scale
        elif kind == 1:    # symmetric range, tiny values in the middle: the subtraction of z rounds
            x = np.where(r.random(n) < 0.9, r.integers(-40, 41, n) * 2.0 ** -24, 0.0)
            x[r.integers(0, n, 4)] = 1.5 * scale
            x[r.integers(0, n, 4)] = -1.5 * scale
        elif kind == 2:    # far from zero: neighbouring binary16 numbers only
            x = 1024.0 + r.integers(0, 7, n)
        elif kind == 3:    # subnormals
            x = r.integers(-9, 10, n) * 2.0 ** -24
        elif kind == 4:    # constant, and zeros of both signs
            x = np.where(r.random(n) < 0.5, 0.0, -0.0) if c % 16 < 8 else np.full(n, -3.25)
        elif kind == 5:    # the whole binary16 range
            x = r.choice([-65504.0, 65504.0, 0.0, 1.0, -1.0, 21840.0, -21824.0], n)
        elif kind == 6:    # a minimum that is huge against the rest
            x = r.standard_normal(n) * 2.0 ** -9
            x[r.integers(0, n)] = -30000.0
        else:
            x = r.standard_normal(n) * scale
        out[:, c] = x
    return out.astype(np.float16)


@pytest.mark.parametrize("bits", [2, 4])
def test_codes_where_the_decision_is_delicate(kv, bits):
    import torch
    n = 3 * 128 + 7
    K = _delicate_columns(n, 1)[None, None]
    r = np.random.default_rng(2)
    V = np.zeros((1, 1, n, 128), dtype=np.float16)
    for t in range(n):  # rotated: constants, two and three levels, sums of a few signs, ordinary rows of any scale
        kind, a = t % 5, np.float16(2.0 ** r.integers(-12, 9))
        if kind < 4:
            V[0, 0, t, r.choice(128, size=(1, 2, 3, 8)[kind], replace=False)] = a
        else:
            V[0, 0, t] = (r.standard_normal(128) * float(a)).astype(np.float16)
    cache = kv.KVLincCache(1, 1, 1, 1024, bits=bits)
    cache.append(tl.to_dev(K), tl.to_dev(V))
    torch.cuda.synchronize()
    assert int(cache.status.item()) == 0
    tl.check_pair_against_oracle(cache, 0, 0, K[0, 0], V[0, 0], 384, 7)


@pytest.mark.parametrize("sliding", [False, True])
@pytest.mark.parametrize("parts", [(1, 2), (5, 11), (3, 60, 1), (127, 2), (128, 128), (100, 157), (16, 112, 129), (130, 3, 250)])
def test_rows_that_stay_in_the_window(kv, parts, sliding):
    """Prompts in pieces: the new rows behind old ones, over a flush, from an odd slot on, a full window, a single row."""
    import torch
    B, H_q, H_kv, n = 2, 2, 2, sum(parts)
    K, V = tl.gen_kv(61, B, H_kv, [n, n])
    Wq, Wk = synth.adapters_q(61, H_q), synth.adapters_k(61, H_kv)
    cache = kv.KVLincCache(B, H_q, H_kv, 1024, Wq=tl.to_dev(Wq), Wk=tl.to_dev(Wk),
                           flags=kv.KVLINC_FLAG_SLIDING_VALUES if sliding else 0)
    done = 0
    for i, m in enumerate(parts):
        cache.append(tl.to_dev(K[:, :, done:done + m]), tl.to_dev(V[:, :, done:done + m]))
        done += m
        pairs = [(b, g) for b in range(B) for g in range(H_kv)]
        tl.check_cache_against_oracle(cache, K[:, :, :done], V[:, :, :done], [done, done], pairs, Wk=Wk)
    assert int(cache.status.item()) == 0 and not cache.split_done.any()


@pytest.mark.parametrize("R,keep", [(4, 4), (20, 3), (32, 32), (64, 61), (128, 17)])
@pytest.mark.parametrize("n", [19, 128 + 5, 300])
def test_static_window_sizes(kv, R, keep, n):
    import torch
    K, V = tl.gen_kv(62, 1, 1, [n])
    Wk = synth.adapters_k(62, 1)
    cache = kv.KVLincCache(1, 1, 1, 512, R=R, Wq=tl.to_dev(synth.adapters_q(62, 1)), Wk=tl.to_dev(Wk))
    cache.append(tl.to_dev(K), tl.to_dev(V), keep_residual=keep)
    torch.cuda.synchronize()
    tl.check_cache_against_oracle(cache, K, V, [n], [(0, 0)], Wk=Wk, keep=keep)
    assert int(cache.status.item()) == 0 and not cache.split_done.any()


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("n_flush", [2, 37, 128 + 100, 256 + 127])
def test_padding_tokens_leave_the_states_alone_whatever_the_keys_span(kv, n_flush, bits):
    """A partial last group with channels that span more than binary16's largest number, their maximum in the last token that
    is quantized: the distance of its key from the padding's code 0 overflows, and nothing of that may reach S, P.  (The
    adapters of these channels are small, so that the errors of the real tokens, half a step at most, leave ordinary logits.)"""
    import torch
    n, R, wide = n_flush + 32, 32, {5: (-40000.0, 30000.0), 77: (-65504.0, 65504.0)}
    K, V = tl.gen_kv(64, 2, 2, [n, n])
    Wk = synth.adapters_k(64, 2).copy()
    for c, (low, high) in wide.items():
        K[:, :, (n_flush - 1) // 128 * 128, c] = low
        K[:, :, n_flush - 1, c] = high
        Wk[:, :, c] = (Wk[:, :, c].astype(np.float32) * 2.0 ** -10).astype(np.float16)
    cache = kv.KVLincCache(2, 2, 2, 512, R=R, Wq=tl.to_dev(synth.adapters_q(64, 2)), Wk=tl.to_dev(Wk), bits=bits)
    cache.append(tl.to_dev(K), tl.to_dev(V), keep_residual=32)
    torch.cuda.synchronize()
    assert int(cache.status.item()) == 0
    tl.check_cache_against_oracle(cache, K, V, [n, n], [(b, g) for b in range(2) for g in range(2)], Wk=Wk, keep=32)


@pytest.mark.parametrize("sliding", [False, True])
def test_no_row_of_a_refused_append_reaches_the_window(kv, sliding):
    """A fault in the last row of one head: nothing live changes, and no non-finite value is stored anywhere."""
    import torch
    B, H = 1, 2
    K, V = tl.gen_kv(63, B, H, [400])
    cache = kv.KVLincCache(B, H, H, 1024, flags=kv.KVLINC_FLAG_SLIDING_VALUES if sliding else 0)
    cache.append(tl.to_dev(K[:, :, :180]), tl.to_dev(V[:, :, :180]))
    before = [t.clone() for t in (cache.groups[:, :, :1], cache.k_res[:, :, :52], cache.v_res if sliding else cache.v_res[:, :, :13], cache.n_quant, cache.n_res)]
    for first, last in ((180, 200), (180, 400)):
        for which in (K, V):
            k, v = K[:, :, first:last].copy(), V[:, :, first:last].copy()
            (k if which is K else v)[0, 1, -1, 77] = np.inf
            cache.append(tl.to_dev(k), tl.to_dev(v))
            torch.cuda.synchronize()
            assert int(cache.status.item()) & kv.KVLINC_ST_NONFINITE
            cache.status.zero_()
            after = (cache.groups[:, :, :1], cache.k_res[:, :, :52], cache.v_res if sliding else cache.v_res[:, :, :13], cache.n_quant, cache.n_res)
            assert all(torch.equal(a, b) for a, b in zip(after, before))
            assert torch.isfinite(cache.k_res.float()).all() and torch.isfinite(cache.v_res.float()).all()
            assert not cache.split_done.any()


def test_more_pairs_than_one_launch_holds(kv):
    """2^23 + 5 (sequence, kv head) pairs: an append of several rows, or one that keeps a residual, takes two workgroups of 256
    threads for each, and a launch holds fewer than 2^32 threads.  (100 GB of cache.)"""
    import torch
    B = 2 ** 23 + 5
    if torch.cuda.mem_get_info()[0] < 130e9:
        pytest.skip("needs 130 GB of free device memory")
    cache = kv.KVLincCache(B, 1, 1, 128, R=4)
    k = torch.randn(B, 1, 1, 128, device="cuda", dtype=torch.float16)
    v = torch.randn(B, 1, 1, 128, device="cuda", dtype=torch.float16)
    k[-2, 0, 0, 9] = float("inf")
    cache.append(k, v, keep_residual=4)
    assert int(cache.status.item()) == kv.KVLINC_ST_NONFINITE and not cache.split_done.any()
    want = torch.ones(B, dtype=torch.int32, device="cuda")
    want[-2] = 0
    assert torch.equal(cache.n_res, want) and not cache.n_quant.any()
    k[-2] = 0
    assert torch.equal(cache.k_res[:, 0, 0], k[:, 0, 0])
    for b in (0, 2 ** 22, 2 ** 23 - 1, 2 ** 23, B - 1):
        tl.check_pair_against_oracle(cache, b, 0, k[b, 0].cpu().numpy(), v[b, 0].cpu().numpy(), 0, 1)
    del cache, k, v
    torch.cuda.empty_cache()
