"""GPU parity of decodes over batches of many sequences of unequal lengths: every workgroup sums the groups of the whole batch from
its counters, 64 at a time and the first 256 at once, and the splits of every sequence hang on that sum."""
import numpy as np
import pytest

import kvlinc_synth as synth
from tests import kvlinc_testlib as tl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("corr", [True, False])
@pytest.mark.parametrize("B", [2, 64, 65, 192, 255, 256, 257, 320, 321])
def test_many_sequences(B, corr):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2510_05373_amd as kv
    from oracle import attention as o_attn
    from oracle import kvcache as o_cache
    r = np.random.default_rng([96, B])
    lengths = r.integers(1, 700, size=B)
    lengths[r.integers(0, B, size=max(1, B // 40))] = 3000  # a few long ones, which take several splits
    lengths[-1] = 2900
    # 7 histories, dealt to the sequences in turn
    n_max = int(lengths.max())
    Kb, Vb = tl.gen_kv(96, 7, 1, [n_max] * 7)
    of = np.arange(B) % 7
    K, V = tl.to_dev(Kb)[torch.from_numpy(of).cuda()], tl.to_dev(Vb)[torch.from_numpy(of).cuda()]
    Wq, Wk = (synth.adapters_q(96, 2), synth.adapters_k(96, 1)) if corr else (None, None)
    cache = kv.KVLincCache(B, 2, 1, n_max + 128, Wq=tl.to_dev(Wq) if corr else None, Wk=tl.to_dev(Wk) if corr else None)
    cache.append(K, V, n_new=tl.to_dev(lengths.astype(np.int32)))
    q = r.standard_normal((B, 2, 128)).astype(np.float16)
    got = [cache.decode(tl.to_dev(q), max_context=n_max).cpu().numpy() for _ in range(2)]
    assert np.isfinite(got[0].astype(np.float32)).all() and np.array_equal(tl.u16(got[0]), tl.u16(got[1]))
    assert int(cache.split_done.abs().sum().item()) == 0  # every count was completed
    n_quant = cache.n_quant.cpu().numpy()
    want = {}
    for b in sorted({0, B // 2, min(63, B - 1), min(64, B - 1), min(255, B - 1), B - 1, int(np.argmax(lengths))}):
        ref = o_cache.build_cache(Kb[of[b], 0, :lengths[b]], Vb[of[b], 0, :lengths[b]], int(n_quant[b]), Wk=Wk[0] if corr else None)
        for h in range(2):
            want[b, h] = o_attn.decode(q[b, h], ref, Wq[h] if corr else None)
    tl.check_outputs(got[0], want)
