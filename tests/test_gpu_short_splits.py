"""GPU parity of decodes over many short sequences of unequal lengths: around the number of groups from which on one is cut in two where a
sequence has one split on average (more than 24), and, with 24 at most, without any second split in the launch."""
import numpy as np
import pytest

import kvlinc_synth as synth
from tests import kvlinc_testlib as tl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("top", [24, 25, 26])
def test_splits_of_short_sequences(top, bits):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2510_05373_amd as kv
    from oracle import attention as o_attn
    from oracle import kvcache as o_cache
    B, H = 8, 32
    lengths = [128 * top, 128 * 24 - 1, 128 * (top - 1), 128 * 12 + 1, 130, 300, 1, 128]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(96)
    K = torch.randn(B, H, max(lengths), 128, device="cuda", dtype=torch.float16, generator=gen)
    V = torch.randn(B, H, max(lengths), 128, device="cuda", dtype=torch.float16, generator=gen)
    Wq, Wk = synth.adapters_q(96, H), synth.adapters_k(96, H)
    cache = kv.KVLincCache(B, H, H, max(lengths) + 128, Wq=tl.to_dev(Wq), Wk=tl.to_dev(Wk), bits=bits)
    cache.append(K, V, n_new=tl.to_dev(np.asarray(lengths, dtype=np.int32)))
    q = tl.gen_q(96, B, H)
    got = cache.decode(tl.to_dev(q), max_context=max(lengths)).cpu().numpy()
    want = {}
    for b in range(B):
        h, n = (5 * b) % H, lengths[b]
        ref = o_cache.build_cache(K[b, h, :n].cpu().numpy(), V[b, h, :n].cpu().numpy(), int(cache.n_quant[b].item()), Wk=Wk[h], bits=bits)
        want[b, h] = o_attn.decode(q[b, h], ref, Wq[h])
    tl.check_outputs(got, want)
    assert int(cache.split_done.abs().sum().item()) == 0
