"""GPU parity where the merge of the splits, the shares of a ragged batch and the one-token window flush change their way:
every size class of the merge, batches beyond one wave of counters, more kv heads than a flush has waves, each way the
states are kept, and the growth of the workspace."""
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


# One sequence and one kv head take ceil(groups / 4) splits, 32 at most: the merge loads 2, 6 or 16 pairs of partial rows, an
# odd number of splits leaves half of a load unused.
@pytest.mark.parametrize("splits", [1, 2, 3, 4, 5, 11, 12, 13, 31, 32])
@pytest.mark.parametrize("H_q,corr", [(4, True), (7, False), (2, True)])
def test_every_size_class_of_the_merge(kv, splits, H_q, corr):
    n = 512 * (splits - 1) + 129 + 37  # (splits - 1) * 4 + 1 full groups and a window
    K, V = tl.gen_kv(71, 1, 1, [n])
    q = tl.gen_q(71, 1, H_q)
    Wq, Wk = (synth.adapters_q(71, H_q), synth.adapters_k(71, 1)) if corr else (None, None)
    cache = kv.KVLincCache(1, H_q, 1, n, Wq=None if Wq is None else tl.to_dev(Wq), Wk=None if Wk is None else tl.to_dev(Wk))
    cache.append(tl.to_dev(K), tl.to_dev(V))
    got = cache.decode(tl.to_dev(q), max_context=n).cpu().numpy()
    want = tl.oracle_decode(K, V, q, [n], cache.n_quant.cpu().numpy(), [(0, 0)], H_q, 1, Wq, Wk)
    tl.check_outputs(got, want)
    assert not cache.split_done.any()


@pytest.mark.parametrize("B", [63, 64, 65, 130])
def test_ragged_batches_around_one_wave_of_counters(kv, B):
    r = np.random.default_rng(B)
    lengths = r.integers(1, 400, B)
    lengths[[0, B // 2, B - 1]] = [2900, 700, 1500]
    pairs = [(0, 0), (1, 1), (B // 2, 1), (B - 2, 0), (B - 1, 1)]
    K, V = tl.gen_kv(72, B, 2, lengths)
    q = tl.gen_q(72, B, 8)
    Wq, Wk = synth.adapters_q(72, 8), synth.adapters_k(72, 2)
    cache = kv.KVLincCache(B, 8, 2, int(lengths.max()), Wq=tl.to_dev(Wq), Wk=tl.to_dev(Wk))
    cache.append(tl.to_dev(K), tl.to_dev(V), n_new=tl.to_dev(lengths.astype(np.int32)))
    got = cache.decode(tl.to_dev(q)).cpu().numpy()
    tl.check_outputs(got, tl.oracle_decode(K, V, q, lengths, cache.n_quant.cpu().numpy(), pairs, 8, 2, Wq, Wk))
    assert not cache.split_done.any()


@pytest.mark.parametrize("H_kv", [1, 8, 9, 17])
@pytest.mark.parametrize("bits,state", [(2, "fp32"), (4, "fp32"), (2, "none")])
def test_flush_of_one_token(kv, H_kv, bits, state):
    """Two windows flushed token by token (the second one into states that are not zero), beside a sequence that flushes at
    another time; then a flush refused for a fault in the last head."""
    import torch
    lengths = [128 + 130, 90 + 130]
    K, V = tl.gen_kv(73, 2, H_kv, lengths)
    Wk = synth.adapters_k(73, H_kv) if state != "none" else None
    Wq = synth.adapters_q(73, H_kv) if state != "none" else None
    cache = kv.KVLincCache(2, H_kv, H_kv, 640, Wq=None if Wq is None else tl.to_dev(Wq), Wk=None if Wk is None else tl.to_dev(Wk), bits=bits)
    kd, vd = tl.to_dev(K), tl.to_dev(V)
    first = np.array([128, 90], dtype=np.int32)
    cache.append(kd[:, :, :128].contiguous(), vd[:, :, :128].contiguous(), n_new=tl.to_dev(first))
    for i in range(130):
        k1 = torch.stack([kd[b, :, first[b] + i] for b in range(2)])[:, :, None].contiguous()
        v1 = torch.stack([vd[b, :, first[b] + i] for b in range(2)])[:, :, None].contiguous()
        cache.append(k1, v1)
    pairs = [(b, g) for b in range(2) for g in sorted({0, H_kv // 2, H_kv - 1})]
    tl.check_cache_against_oracle(cache, K, V, lengths, pairs, Wk=Wk)
    assert int(cache.status.item()) == 0 and not cache.split_done.any()
    # fill both windows, then refuse the flush
    n_res = cache.n_res.cpu().numpy()
    fill = (128 - n_res).astype(np.int32)
    more = torch.randn(2, H_kv, int(fill.max()), 128, device="cuda").half()
    cache.append(more, more, n_new=tl.to_dev(fill))
    live = [t for t in (cache.k_res, cache.v_res, cache.n_quant, cache.n_res, cache.S, cache.S16, cache.P) if t is not None]
    before = [t.clone() for t in live]
    bad = torch.randn(2, H_kv, 1, 128, device="cuda").half()
    bad[:, H_kv - 1, 0, 5] = float("inf")
    for k1, v1 in ((bad, bad.nan_to_num(1.0, 1.0, 1.0)), (bad.nan_to_num(1.0, 1.0, 1.0), bad)):
        cache.append(k1, v1)
        torch.cuda.synchronize()
        assert int(cache.status.item()) == kv.KVLINC_ST_NONFINITE
        cache.status.zero_()
        assert all(torch.equal(a, b) for a, b in zip(live, before)) and not cache.split_done.any()


def test_flush_with_the_state_in_binary16_only(kv):
    """Against the same tokens with the binary32 master copy: one rounding per flush apart."""
    import torch
    K, V = tl.gen_kv(74, 1, 2, [300])
    Wq, Wk = synth.adapters_q(74, 2), synth.adapters_k(74, 2)
    kd, vd = tl.to_dev(K), tl.to_dev(V)
    out = []
    for storage in ("fp32", "fp16"):
        cache = kv.KVLincCache(1, 2, 2, 512, Wq=tl.to_dev(Wq), Wk=tl.to_dev(Wk), state_storage=storage)
        for t in range(300):
            cache.append(kd[:, :, t:t + 1].contiguous(), vd[:, :, t:t + 1].contiguous())
        assert (int(cache.n_quant.item()), int(cache.n_res.item())) == (256, 44)
        out.append((cache.S16.float(), cache.P.clone(), cache.groups.clone()))
    (a, pa, ga), (b, pb, gb) = out
    assert torch.equal(ga, gb) and torch.equal(pa, pb)
    # two roundings to binary16 (2^-11 each) against one, of entries that may have cancelled between the flushes
    assert (a - b).abs().max().item() <= 3 * 2.0 ** -11 * a.abs().max().item()


def test_workspace_grows_with_the_context(kv):
    import torch
    K, V = tl.gen_kv(75, 1, 1, [4000])
    q = tl.gen_q(75, 1, 4)
    qd, kd, vd = tl.to_dev(q), tl.to_dev(K), tl.to_dev(V)
    cache = kv.KVLincCache(1, 4, 1, 4000)
    done, sizes = 0, []
    for n in (300, 1500, 4000):
        cache.append(kd[:, :, done:n].contiguous(), vd[:, :, done:n].contiguous())
        done = n
        got = cache.decode(qd, max_context=n).cpu().numpy()
        sizes.append(cache._ws.numel())
        tl.check_outputs(got, tl.oracle_decode(K, V, q, [n], cache.n_quant.cpu().numpy(), [(0, 0)], 4, 1))
    assert sizes[0] < sizes[1] < sizes[2]
    fresh = torch.empty_like(qd)
    cache.decode(qd, out=fresh, max_context=300 + 3700)
    assert torch.equal(fresh, tl.to_dev(got))
