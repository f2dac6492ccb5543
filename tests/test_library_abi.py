"""The C-ABI library loads without a GPU, exports every function include/kvlinc.h declares, and its host-side checks
reject bad descriptors before any launch (no compute call is made here: every rejected call returns before a launch,
and the accepted ones only compute sizes)."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "kvlinc.h")

# An unbuilt library is built here (hipcc cross-compiles without a GPU); a library that cannot be built or loaded is a
# failure of these tests, never a skip.
if not os.path.exists(os.path.join(ROOT, "paper_2510_05373_amd", "libkvlinc.so")):
    import importlib.util
    _spec = importlib.util.spec_from_file_location("_kvlinc_build", os.path.join(ROOT, "paper_2510_05373_amd", "build.py"))
    _build = importlib.util.module_from_spec(_spec)  # by path: importing the package itself needs the library
    _spec.loader.exec_module(_build)
    _build.build()
from paper_2510_05373_amd import binding as kb  # noqa: E402


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(kvlinc_[a-z_]+)\s*\(", text)))


def fake_struct(**over):
    """A descriptor whose pointers are aligned non-NULL integers; never dereferenced by the host checks."""
    base = 0x10000
    f = dict(B=2, H_q=8, H_kv=2, d=128, G=128, R=128, D=256, bits=2, max_groups=8, groups=base, k_res=base,
             v_res=base, n_quant=base, n_res=base, S=base, S16=base, P=base, Wq=base, Wk=base, status=base,
             split_done=base, flags=0)
    f.update(over)
    return kb.CacheStruct(**f)


def test_header_functions_are_exported():
    names = declared_functions()
    assert names == ["kvlinc_append_quantize", "kvlinc_cache_validate", "kvlinc_decode_attention",
                     "kvlinc_decode_attention_noalloc", "kvlinc_decode_attention_timed", "kvlinc_decode_workspace_bytes",
                     "kvlinc_strerror", "kvlinc_version"]
    lib = ctypes.CDLL(kb.lib_path)
    for n in names:
        assert hasattr(lib, n), n
        assert callable(getattr(kb, n)), "binding lacks " + n


def test_struct_mirror_matches_header_order():
    text = open(HEADER).read()
    body = text[text.index("typedef struct kvlinc_cache {"):text.index("} kvlinc_cache;")]
    body = re.sub(r"/\*.*?\*/", "", body, flags=re.S)
    fields = []
    for decl in body.split("{", 1)[1].split(";"):
        decl = decl.strip()
        if not decl:
            continue
        first, *rest = decl.split(",")
        fields.append(re.findall(r"\**\s*(\w+)$", first.strip())[0])
        fields += [re.sub(r"[\s\*]", "", r) for r in rest]
    assert fields == [n for n, _ in kb.CacheStruct._fields_]


def test_version_and_messages():
    assert kb.kvlinc_version() >= 100
    for code in (0, -1, -2, -3, -4):
        assert "unknown" not in kb.kvlinc_strerror(code)
    assert "unknown" in kb.kvlinc_strerror(-99)


def test_validate_accepts_and_rejects():
    ok = fake_struct()
    assert kb.kvlinc_cache_validate(ok) == kb.KVLINC_OK
    bad = [dict(d=64), dict(G=64), dict(D=128), dict(bits=3), dict(bits=8), dict(R=0), dict(R=130), dict(R=30), dict(H_q=9),
           dict(H_q=32, H_kv=2), dict(B=0), dict(max_groups=0), dict(groups=0), dict(groups=0x10004), dict(k_res=0),
           dict(v_res=8), dict(n_quant=0), dict(n_res=2), dict(status=0), dict(split_done=0), dict(S16=0),
           dict(S16=0x10008), dict(Wk=0), dict(P=0x10002), dict(S=0x10004), dict(flags=4), dict(flags=-1), dict(flags=kb.KVLINC_FLAG_SLIDING_VALUES, R=64),
           dict(S16=0, P=0, Wq=0, Wk=0)]  # (the last: an fp32 master copy without the rest of the correction)
    for over in bad:
        assert kb.kvlinc_cache_validate(fake_struct(**over)) == kb.KVLINC_EINVAL, over
    # correction off = all of S, S16, P, Wq, Wk NULL; S alone NULL = the state is stored in 16 bits only
    assert kb.kvlinc_cache_validate(fake_struct(S=0, S16=0, P=0, Wq=0, Wk=0)) == kb.KVLINC_OK
    assert kb.kvlinc_cache_validate(fake_struct(S=0)) == kb.KVLINC_OK
    assert kb.kvlinc_cache_validate(fake_struct(flags=kb.KVLINC_FLAG_ALG1_LITERAL)) == kb.KVLINC_OK
    assert kb.kvlinc_cache_validate(fake_struct(flags=kb.KVLINC_FLAG_SLIDING_VALUES | kb.KVLINC_FLAG_ALG1_LITERAL)) == kb.KVLINC_OK
    assert kb.lib.kvlinc_cache_validate(None) == kb.KVLINC_EINVAL


def test_rejections_happen_before_any_launch():
    ok = fake_struct()
    p = ctypes.c_void_p(0x20000)
    ap = kb.lib.kvlinc_append_quantize
    assert ap(ctypes.byref(fake_struct(d=64)), p, p, None, 1, 0, None) == kb.KVLINC_EINVAL
    assert ap(ctypes.byref(ok), None, p, None, 1, 0, None) == kb.KVLINC_EINVAL
    assert ap(ctypes.byref(ok), p, ctypes.c_void_p(0x20002), None, 1, 0, None) == kb.KVLINC_EINVAL
    assert ap(ctypes.byref(ok), p, p, None, 0, 0, None) == kb.KVLINC_EINVAL
    assert ap(ctypes.byref(ok), p, p, None, 1, 129, None) == kb.KVLINC_EINVAL
    assert ap(ctypes.byref(ok), p, p, None, 1, -1, None) == kb.KVLINC_EINVAL
    assert ap(ctypes.byref(fake_struct(R=32)), p, p, None, 1, 0, None) == kb.KVLINC_EINVAL  # lazy flush needs R == G
    # the sliding value window maps token t to slot t % 128: no static cache with kept tokens
    assert ap(ctypes.byref(fake_struct(flags=kb.KVLINC_FLAG_SLIDING_VALUES)), p, p, None, 64, 32, None) == kb.KVLINC_EINVAL
    de = kb.lib.kvlinc_decode_attention
    need = kb.kvlinc_decode_workspace_bytes(ok, 0)
    assert need > 0
    assert de(ctypes.byref(ok), None, p, p, need, 0, None) == kb.KVLINC_EINVAL
    assert de(ctypes.byref(ok), p, p, None, need, 0, None) == kb.KVLINC_EWORKSPACE
    assert de(ctypes.byref(ok), p, p, p, need - 1, 0, None) == kb.KVLINC_EWORKSPACE
    assert de(ctypes.byref(ok), p, p, ctypes.c_void_p(0x20004), need, 0, None) == kb.KVLINC_EWORKSPACE
    assert kb.kvlinc_decode_workspace_bytes(fake_struct(bits=3), 0) == 0
    dt = kb.lib.kvlinc_decode_attention_timed
    ev = ctypes.c_void_p(0x30000)
    assert dt(ctypes.byref(ok), p, p, p, need, 0, None, None, ev) == kb.KVLINC_EINVAL
    assert dt(ctypes.byref(ok), p, p, p, need, 0, None, ev, None) == kb.KVLINC_EINVAL
    assert dt(ctypes.byref(ok), p, p, p, need - 1, 0, None, ev, ev) == kb.KVLINC_EWORKSPACE


def test_cache_bytes_reproduce_the_average_bit_figures():
    """Table 1, column "KV Cache": the buffers of a cache holding 8192 tokens per (sequence, KV head) -- 63 group
    records, the 128-token fp16 window, and with the correction the state stored in 16 bits (S == NULL) plus P --
    average to the printed 2.46 / 2.71 bits per cached element; P is kept in fp32 here, 16 bits more per entry than the
    paper counts (0.002 bits).  Host tensors: nothing is launched."""
    import torch
    from oracle import accounting
    B, H_q, H_kv, n = 2, 8, 2, 8192
    elements = 2 * B * H_kv * n * 128
    plain = kb.KVLincCache(B, H_q, H_kv, n - 128, device="cpu")
    assert plain.max_groups == 63
    bits_plain = plain.bytes() * 8 / elements
    assert abs(bits_plain - accounting.average_bits(n)) < 1e-12 and abs(bits_plain - 2.46) < 0.01
    W = torch.zeros(H_q, 2, 128, 128, dtype=torch.float16)
    c16 = kb.KVLincCache(B, H_q, H_kv, n - 128, Wq=W, Wk=W[:H_kv], device="cpu", state_storage="fp16")
    assert c16.S is None and c16.struct.S is None and c16.struct.S16 is not None
    bits16 = c16.bytes() * 8 / elements
    assert abs(bits16 - (accounting.average_bits(n, D=256) + 256 * 16 / (2 * n * 128))) < 1e-12
    assert abs(bits16 - 2.71) < 0.01
    c32 = kb.KVLincCache(B, H_q, H_kv, n - 128, Wq=W, Wk=W[:H_kv], device="cpu")  # with the fp32 master copy of S
    assert abs(c32.bytes() * 8 / elements - (bits16 + 256 * 128 * 32 / (2 * n * 128))) < 1e-12
    # 4-bit codes: 4 + 32 / 128 bits per quantized element (Sec. 2: a scale and a zero-point of 16 bits per group of 128)
    four = kb.KVLincCache(B, H_q, H_kv, n - 128, device="cpu", bits=4)
    assert four.struct.bits == 4 and four.groups.shape[-1] == 4352
    assert kb.kvlinc_cache_validate(four) == kb.KVLINC_OK
    assert abs(four.bytes() * 8 / elements - accounting.average_bits(n, bits=4)) < 1e-12


def test_noalloc_entry_rejects_on_the_host():
    """kvlinc_decode_attention_noalloc: bad descriptors and pointers, and launches that need more scratch than the
    static buffer, are refused before any HIP call (the pointers here are fakes)."""
    p = ctypes.c_void_p(0x20000)
    na = kb.lib.kvlinc_decode_attention_noalloc
    ok = fake_struct()
    assert na(ctypes.byref(fake_struct(d=64)), p, p, 0, None) == kb.KVLINC_EINVAL
    assert na(ctypes.byref(ok), None, p, 0, None) == kb.KVLINC_EINVAL
    assert na(ctypes.byref(ok), p, ctypes.c_void_p(0x20008), 0, None) == kb.KVLINC_EINVAL
    wide = fake_struct(B=256, H_q=32, H_kv=8, max_groups=32)
    assert kb.kvlinc_decode_workspace_bytes(wide, 4096) > kb.KVLINC_STATIC_SCRATCH_BYTES
    assert na(ctypes.byref(wide), p, p, 4096, None) == kb.KVLINC_ESCRATCH
    text = open(HEADER).read()
    assert "#define KVLINC_STATIC_SCRATCH_BYTES (16u << 20)" in text and kb.KVLINC_STATIC_SCRATCH_BYTES == 16 << 20


def test_workspace_size_is_monotone_and_bounded():
    c = fake_struct(B=16, H_q=32, H_kv=8, max_groups=80)
    sizes = [kb.kvlinc_decode_workspace_bytes(c, n) for n in (1, 128, 129, 1024, 8192, 10240, 0)]
    assert all(s > 0 and s % 16 == 0 for s in sizes)
    assert sizes == sorted(sizes)
    assert sizes[-1] == kb.kvlinc_decode_workspace_bytes(c, 80 * 128 + 128)
    # per (sequence, query head): at most 1024 splits + 4 correction parts of 132 floats
    assert sizes[-1] <= 16 * 32 * (1024 + 4) * 132 * 4


def test_split_policy_of_the_workloads():
    """The most splits a sequence may take, read off the workspace size (B * H_q * (splits + 4 correction parts) * 132
    floats): twice the batch's average of 3 / 4 / 1 / 1 / 1 splits for workloads 2, 4, 5, 6, 7 (head room for
    unequal lengths), 30 for the single long sequence of workload 3, one group per wave (2 splits) for the 1k context
    of workload 1.  A change of the launch policy has to show up here."""
    import kvlinc_synth as synth
    want = {1: 2, 2: 6, 3: 30, 4: 8, 5: 2, 6: 2, 7: 2}
    for cfg_id, cfg in synth.CONFIGS.items():
        n = cfg.get("n") or cfg["n_max"]
        c = fake_struct(B=cfg["B"], H_q=cfg["H_q"], H_kv=cfg["H_kv"], max_groups=(n + 512) // 128)
        per_row = kb.kvlinc_decode_workspace_bytes(c, n) // (cfg["B"] * cfg["H_q"] * 132 * 4)
        assert per_row - 4 == want[cfg_id], (cfg_id, per_row)
        # without the correction there are no correction parts
        c0 = fake_struct(B=cfg["B"], H_q=cfg["H_q"], H_kv=cfg["H_kv"], max_groups=(n + 512) // 128, S=0, S16=0, P=0,
                         Wq=0, Wk=0)
        assert kb.kvlinc_decode_workspace_bytes(c0, n) % (cfg["B"] * cfg["H_q"] * 132 * 4) == 0


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_current_stream_without_the_private_shortcut(monkeypatch, missing):
    import types

    import torch
    monkeypatch.delattr(torch._C, missing, raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=0x1230))
    assert kb._stream(None) == 0x1230
    assert kb._stream(types.SimpleNamespace(cuda_stream=0x4560)) == 0x4560 and kb._stream(0x7890) == 0x7890
