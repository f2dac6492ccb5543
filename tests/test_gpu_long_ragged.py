"""GPU parity of decodes over a few long sequences of unequal lengths: one of them takes as many splits as the merge holds."""
import numpy as np
import pytest

import kvlinc_synth as synth
from tests import kvlinc_testlib as tl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("B,H_q,H_kv", [(2, 28, 4), (4, 12, 2), (8, 8, 1)])
def test_a_long_sequence_among_shorter_ones(B, H_q, H_kv, bits):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2510_05373_amd as kv
    from oracle import attention as o_attn
    from oracle import kvcache as o_cache
    gq = H_q // H_kv
    lengths = [32768] + [16384 if B == 2 else 5000] * (B - 1)
    pairs = [(0, H_kv - 1), (1, 0)]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(97)
    K = torch.randn(B, H_kv, max(lengths), 128, device="cuda", dtype=torch.float16, generator=gen)
    V = torch.randn(B, H_kv, max(lengths), 128, device="cuda", dtype=torch.float16, generator=gen)
    Wq, Wk = synth.adapters_q(97, H_q), synth.adapters_k(97, H_kv)
    cache = kv.KVLincCache(B, H_q, H_kv, max(lengths) + 128, Wq=tl.to_dev(Wq), Wk=tl.to_dev(Wk), bits=bits)
    cache.append(K, V, n_new=tl.to_dev(np.asarray(lengths, dtype=np.int32)))
    q = tl.gen_q(97, B, H_q)
    got = cache.decode(tl.to_dev(q), max_context=max(lengths)).cpu().numpy()
    want = {}
    for b, g in pairs:
        n = lengths[b]
        ref = o_cache.build_cache(K[b, g, :n].cpu().numpy(), V[b, g, :n].cpu().numpy(), int(cache.n_quant[b].item()), Wk=Wk[g], bits=bits)
        for h in range(g * gq, (g + 1) * gq):
            want[b, h] = o_attn.decode(q[b, h], ref, Wq[h])
    tl.check_outputs(got, want)
    assert int(cache.split_done.abs().sum().item()) == 0
