"""GPU parity of appends of a few rows (one launch up to 8 rows and 192 over the kv heads of a sequence, two beyond): rows that
stay in the window, rows that complete a group, both at once, unequal numbers of rows in one call, and refusals, which leave
everything live as it was."""
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


def _cache(kv, B, H_kv, bits, sliding, corr, seed, capacity=640):
    Wq, Wk = (synth.adapters_q(seed, H_kv), synth.adapters_k(seed, H_kv)) if corr else (None, None)
    cache = kv.KVLincCache(B, H_kv, H_kv, capacity, Wq=tl.to_dev(Wq) if corr else None, Wk=tl.to_dev(Wk) if corr else None, bits=bits,
                           flags=kv.KVLINC_FLAG_SLIDING_VALUES if sliding else 0)
    return cache, Wq, Wk


def _live(cache, sliding):
    """Copies of what a refused append has to leave alone (all sequences alike)."""
    nq, nr = int(cache.n_quant[0]), int(cache.n_res[0])
    assert (cache.n_quant == nq).all() and (cache.n_res == nr).all()
    live = [cache.groups[:, :, :nq // 128], cache.k_res[:, :, :nr], cache.n_quant, cache.n_res, cache.split_done]
    if sliding:
        live.append(cache.v_res)
    else:  # 4 slots per channel
        live += [cache.v_res[:, :, :nr // 4], cache.v_res[:, :, nr // 4:nr // 4 + 1, :, :nr % 4]]
    return [t.clone() for t in live + [t for t in (cache.S, cache.S16, cache.P) if t is not None]]


@pytest.mark.parametrize("bits,sliding,corr", [(2, False, True), (4, True, True), (2, True, False), (4, False, True)])
@pytest.mark.parametrize("T,H_kv", [(2, 1), (3, 1), (8, 1), (9, 1), (2, 3), (8, 3), (3, 9), (8, 9), (2, 17), (8, 24), (8, 25)])
def test_rows_over_two_flushes(kv, T, H_kv, bits, sliding, corr):
    """From a prompt that leaves the window almost full, T rows a call until a second group has gone: every way in which T
    rows can lie across a flush occurs for one of the starts."""
    B, calls = 5, -(-134 // T)
    starts = np.array([121, 123, 125, 126, 128], dtype=np.int32)
    lengths = starts + T * calls
    K, V = tl.gen_kv(91, B, H_kv, lengths)
    cache, Wq, Wk = _cache(kv, B, H_kv, bits, sliding, corr, 91)
    kd, vd = tl.to_dev(K), tl.to_dev(V)
    cache.append(kd[:, :, :128].contiguous(), vd[:, :, :128].contiguous(), n_new=tl.to_dev(starts))
    pairs = [(b, g) for b in range(B) for g in sorted({0, H_kv // 2, H_kv - 1})]
    import torch
    for i in range(calls):
        pick = lambda x: torch.stack([x[b, :, starts[b] + T * i:starts[b] + T * (i + 1)] for b in range(B)]).contiguous()
        cache.append(pick(kd), pick(vd))
        if i in (0, 1, 2, 3):
            done = starts + T * (i + 1)
            tl.check_cache_against_oracle(cache, K, V, done, pairs, Wk=Wk)
    tl.check_cache_against_oracle(cache, K, V, lengths, pairs, Wk=Wk)
    assert int(cache.status.item()) == 0 and not cache.split_done.any()
    q = tl.gen_q(91, B, H_kv)
    got = cache.decode(tl.to_dev(q)).cpu().numpy()
    if not sliding:
        tl.check_outputs(got, tl.oracle_decode(K, V, q, lengths, cache.n_quant.cpu().numpy(), pairs, H_kv, H_kv, Wq, Wk, bits=bits))
    else:  # the value window holds the newest 128 values, token t in slot t % 128
        from oracle import hadamard, layout
        for b, g in pairs:
            n = int(lengths[b])
            want = hadamard.fwht_spec32(V[b, g, n - 128:n])
            win = layout.unpack_value_window(cache.v_res[b, g].cpu().numpy(), 128)
            assert np.array_equal(tl.u16(win[np.arange(n - 128, n) % 128]), tl.u16(want)), (b, g)


@pytest.mark.parametrize("sliding", [False, True])
@pytest.mark.parametrize("H_kv", [1, 5])
def test_unequal_numbers_of_rows_in_a_call(kv, H_kv, sliding):
    """n_new from below 0 to above T, the rows beyond it NaN; more sequences than a launch has waves in its first round."""
    import torch
    B, T = 700, 6
    r = np.random.default_rng(92)
    starts = r.integers(118, 129, B).astype(np.int32)
    kd = torch.randn(B, H_kv, 180, 128, device="cuda").half()
    vd = torch.randn(B, H_kv, 180, 128, device="cuda").half()
    cache, _, _ = _cache(kv, B, H_kv, 2, sliding, False, 92, capacity=256)
    cache.append(kd, vd, n_new=tl.to_dev(starts))
    done = starts.copy()
    ar = torch.arange(T, device="cuda")
    for _ in range(4):
        n_new = r.integers(-1, T + 2, B).astype(np.int32)
        at = (tl.to_dev(done.astype(np.int64))[:, None] + ar).view(B, 1, T, 1).expand(B, H_kv, T, 128)
        beyond = (ar >= tl.to_dev(n_new)[:, None]).view(B, 1, T, 1)
        k, v = (x.gather(2, at).masked_fill(beyond, float("nan")) for x in (kd, vd))
        cache.append(k, v, n_new=tl.to_dev(n_new))
        done += np.clip(n_new, 0, T)
    assert int(cache.status.item()) == 0 and not cache.split_done.any()
    tl.check_counters(cache, done)
    K, V = kd.cpu().numpy(), vd.cpu().numpy()
    for b in list(range(0, B, 37)) + [B - 1]:
        for g in range(H_kv):
            tl.check_pair_against_oracle(cache, b, g, K[b, g, :done[b]], V[b, g, :done[b]], int(cache.n_quant[b]), int(cache.n_res[b]))


@pytest.mark.parametrize("bits,sliding", [(2, False), (2, True), (4, False)])
@pytest.mark.parametrize("H_kv", [1, 9])
@pytest.mark.parametrize("held", [128 + 60, 128 + 122, 256])
@pytest.mark.parametrize("T", [2, 8])
def test_refused_as_a_whole(kv, T, held, H_kv, bits, sliding):
    """A fault in any row of the first or last head: a key, a value, a value that only leaves binary16 when it is rotated."""
    import torch
    B = 2
    kd, vd = (torch.randn(B, H_kv, held, 128, device="cuda").half() for _ in range(2))
    cache, _, _ = _cache(kv, B, H_kv, bits, sliding, True, 93)
    cache.append(kd, vd)
    before = _live(cache, sliding)
    for row in (0, T - 1):
        for head in {0, H_kv - 1}:
            for kind in range(3):
                k, v = (torch.randn(B, H_kv, T, 128, device="cuda").half() for _ in range(2))
                for b in range(B):
                    if kind == 0: k[b, head, row, 7] = float("nan")
                    if kind == 1: v[b, head, row, 127] = -float("inf")
                    if kind == 2: v[b, head, row] = 60000.0
                cache.append(k, v)
                assert int(cache.status.item()) == kv.KVLINC_ST_NONFINITE
                cache.status.zero_()
                assert all(torch.equal(a, b) for a, b in zip(_live(cache, sliding), before)), (row, head, kind)
                assert torch.isfinite(cache.k_res.float()).all() and torch.isfinite(cache.v_res.float()).all()


def test_no_room_for_the_group(kv):
    import torch
    cache, _, _ = _cache(kv, 1, 2, 2, False, True, 94, capacity=128)
    x = torch.randn(1, 2, 256, 128, device="cuda").half()
    cache.append(x, x)
    before = _live(cache, False)
    cache.append(x[:, :, :3].contiguous(), x[:, :, :3].contiguous())
    assert int(cache.status.item()) == kv.KVLINC_ST_CAPACITY
    assert all(torch.equal(a, b) for a, b in zip(_live(cache, False), before))


@pytest.mark.parametrize("sliding", [False, True])
@pytest.mark.parametrize("T", [3, 150])
def test_appends_of_several_rows_replayed_from_a_graph(kv, T, sliding):
    """One launch (3 rows) and two (150 rows), through the current stream; every replay against an eager twin, a refused call
    among them."""
    import torch
    B, H_kv, replays = 3, 2, 50 if T == 3 else 8
    pair = [_cache(kv, B, H_kv, 2, sliding, True, 95, capacity=1536)[0] for _ in range(2)]
    first = torch.randn(B, H_kv, 120, 128, device="cuda").half()
    for c in pair:
        c.append(first, first, n_new=tl.to_dev(np.array([120, 60, 1], dtype=np.int32)))
    graphed, eager = pair
    k_in, v_in = (torch.zeros(B, H_kv, T, 128, dtype=torch.float16, device="cuda") for _ in range(2))
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        graphed.append(k_in, v_in)
    for i in range(replays):
        k, v = (torch.randn(B, H_kv, T, 128, device="cuda").half() for _ in range(2))
        if i == replays // 2:
            k[1, 1, T - 1, 5] = float("inf")
        k_in.copy_(k)
        v_in.copy_(v)
        torch.cuda.synchronize()
        g.replay()
        eager.append(k, v)
        torch.cuda.synchronize()
        names = ["n_quant", "n_res", "S", "P", "S16", "status", "split_done"]
        assert all(torch.equal(getattr(graphed, n), getattr(eager, n)) for n in names), i
        for b in range(B):
            nq, nr = int(eager.n_quant[b]), int(eager.n_res[b])
            assert torch.equal(graphed.groups[b, :, :nq // 128], eager.groups[b, :, :nq // 128])
            assert torch.equal(graphed.k_res[b, :, :nr], eager.k_res[b, :, :nr])
    assert int(graphed.status.item()) == kv.KVLINC_ST_NONFINITE and int(graphed.n_quant.max().item()) > 0
