"""Performance cases of the KVLinC cache path: what a serving program has it do, through KVLincCache.append / decode.

Two kinds of pass:

  "step"     STEPS generated tokens, one window length: per token and layer cache one append of the new row of every
             sequence and one decode of its queries.  Every sequence therefore flushes its window exactly once per
             pass.  A pass first puts the caches back to the end of the prompt (another sample of the same prompt).
  "prefill"  the prompt of every sequence appended to an emptied cache, in `chunks` calls.

Fields of a case:
  B, Hq, Hkv     sequences, query heads, KV heads
  n              longest prompt of the batch in tokens
  spread         the other prompts are uniform in [n (1 - spread), n]; 0: all alike
  bits           width of the codes
  state          "fp32": fp32 master copy of S kept; "fp16": S in binary16 only; "none": correction off
  sliding        values leave the fp16 window one token at a time
  layers         layer caches a pass goes through in turn (step): a model's layers, so that a cache is not in the
                 on-chip caches from the token before
  chunks         calls a prompt arrives in (prefill)
"""
import math

import numpy as np
import torch

import paper_2510_05373_amd as kv

STEPS = 128


def _case(name, kind, B, Hq, Hkv, n, spread=0.0, bits=2, state="fp32", sliding=False, layers=1, chunks=1):
    return {"name": name, "kind": kind, "B": B, "Hq": Hq, "Hkv": Hkv, "n": n, "spread": spread, "bits": bits, "state": state,
            "sliding": sliding, "layers": layers, "chunks": chunks}


def listed():
    return [
        # first tokens of one user's chat: the smallest calls, launch and latency bound
        _case("step_b1_ctx300", "step", 1, 32, 8, 300),
        # grouped-query model, medium batch, 8k context: the workload the benchmark quotes
        _case("step_b16_ctx8k", "step", 16, 32, 8, 8192, layers=3),
        # the same with 4-bit codes and prompts of unequal length
        _case("step_b16_ctx8k_4bit", "step", 16, 32, 8, 8192, spread=0.25, bits=4, layers=2),
        # one very long document
        _case("step_b1_ctx128k", "step", 1, 32, 8, 131072, layers=4),
        # seven query heads per KV head, long contexts: the largest call
        _case("step_b32_ctx32k_gq7", "step", 32, 28, 4, 32768),
        # continuous batching: 64 users anywhere between 1k and 16k tokens
        _case("step_b64_ragged_16k", "step", 64, 32, 8, 16384, spread=0.9375),
        # throughput serving of short contexts: a multi-head model, and a grouped-query model at a large batch
        _case("step_b32_mha_ctx1280", "step", 32, 32, 32, 1280, layers=2),
        _case("step_b144_ctx1280", "step", 144, 32, 8, 1280, spread=0.5, layers=2),
        # one chat prompt
        _case("prefill_b1_700", "prefill", 1, 32, 8, 700),
        # a batch of 8k prompts in one call
        _case("prefill_b16_8k", "prefill", 16, 32, 8, 8192),
        # one very long document in one call
        _case("prefill_b1_128k", "prefill", 1, 32, 8, 131072),
        # prompts of unequal length arriving in chunks, 4-bit codes
        _case("prefill_b32_ragged_4bit", "prefill", 32, 28, 4, 4100, spread=0.9, bits=4, chunks=3),
    ]


def draw(rng):
    """Another case of the same ranges: sizes log-uniform and odd, at most the work of the largest listed case."""
    kind = "step" if rng.random() < 0.6 else "prefill"
    Hq, Hkv = rng.choice([(32, 8), (32, 8), (28, 4), (32, 32), (64, 8), (16, 8), (12, 2)])
    bits = 4 if rng.random() < 0.25 else 2
    rows = (2_000_000 if kind == "step" else 1_000_000) // (2 if bits == 4 else 1)  # (sequence, KV head, token) rows
    B = max(1, int(round(math.exp(rng.uniform(0.0, math.log(144.5))))))
    most = min(131072, rows // (B * Hkv))
    n = int(math.exp(rng.uniform(math.log(160), math.log(max(most, 161)))))
    spread = rng.choice([0.0, 0.0, round(rng.uniform(0.05, 0.9), 2)]) if B > 1 else 0.0
    state = rng.choice(["fp32", "fp32", "fp32", "fp16", "none"])
    sliding = rng.random() < 0.15
    per_layer = B * Hkv * (n * 36 * bits + 200_000)
    layers = max(1, min(4, round(300e6 / per_layer))) if kind == "step" else 1
    chunks = rng.choice([1, 1, 2, 4]) if kind == "prefill" and n >= 1024 else 1
    c = _case("", kind, B, Hq, Hkv, n, spread, bits, state, sliding, layers, chunks)
    del c["name"]
    return c


def _lengths(case):
    """Prompt lengths, a function of the case alone (the work of a pass does not depend on the seed)."""
    n, B = case["n"], case["B"]
    lo = max(1, int(n * (1.0 - case["spread"])))
    r = np.random.default_rng([B, n, 7])
    out = r.integers(lo, n + 1, size=B)
    out[0] = n
    return out.astype(np.int64)


def _prompt(B, Hkv, n, gen):
    """Keys and values N(0, 1) in fp16, the keys of 4 channels per KV head 8 times as large."""
    dev = gen.device
    k = torch.randn(B, Hkv, n, 128, dtype=torch.float16, device=dev, generator=gen)
    v = torch.randn(B, Hkv, n, 128, dtype=torch.float16, device=dev, generator=gen)
    gain = torch.ones(Hkv, 128, dtype=torch.float16, device=dev)
    gain.scatter_(1, torch.rand(Hkv, 128, device=dev, generator=gen).argsort(1)[:, :4], 8.0)
    return k.mul_(gain[None, :, None, :]), v, gain


def prepare(case, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    B, Hq, Hkv, n = case["B"], case["Hq"], case["Hkv"], case["n"]
    step = case["kind"] == "step"
    lengths = _lengths(case)
    room = n + (STEPS if step else 0) + 128
    layers = []
    for _ in range(case["layers"]):
        Wq = Wk = None
        if case["state"] != "none":
            Wq = torch.randn(Hq, 2, 128, 128, device=dev, generator=gen).mul_(128 ** -0.5).half()
            Wk = torch.randn(Hkv, 2, 128, 128, device=dev, generator=gen).mul_(128 ** -0.5).half()
        cache = kv.KVLincCache(B, Hq, Hkv, room, Wq=Wq, Wk=Wk, bits=case["bits"],
                               state_storage="fp16" if case["state"] == "fp16" else "fp32",
                               flags=kv.KVLINC_FLAG_SLIDING_VALUES if case["sliding"] else 0)
        k, v, gain = _prompt(B, Hkv, n, gen)
        layer = {"cache": cache}
        if step:
            cache.append(k, v, n_new=torch.from_numpy(lengths.astype(np.int32)).to(dev))
            live = [t for t in (cache.n_quant, cache.n_res, cache.k_res, cache.v_res, cache.S, cache.S16, cache.P) if t is not None]
            layer["at_prompt"] = [(t, t.clone()) for t in live]
            kn = torch.randn(STEPS, B, Hkv, 1, 128, dtype=torch.float16, device=dev, generator=gen).mul_(gain[None, None, :, None, :])
            vn = torch.randn(STEPS, B, Hkv, 1, 128, dtype=torch.float16, device=dev, generator=gen)
            q = torch.randn(STEPS, B, Hq, 128, dtype=torch.float16, device=dev, generator=gen)
            out = torch.empty(STEPS, B, Hq, 128, dtype=torch.float16, device=dev)
            layer["out"] = out
            layer["tokens"] = [(kn[t], vn[t], q[t], out[t]) for t in range(STEPS)]
            cache.workspace(n + STEPS)
        else:
            # the chunks of a prompt that is shorter than the longest one run out earlier
            cut = [n * i // case["chunks"] for i in range(case["chunks"] + 1)]
            layer["calls"] = [(k[:, :, a:b].contiguous(), v[:, :, a:b].contiguous(),
                               torch.from_numpy(np.clip(lengths - a, 0, b - a).astype(np.int32)).to(dev))
                              for a, b in zip(cut[:-1], cut[1:])]
            layer["empty"] = [t for t in (cache.n_quant, cache.n_res, cache.S, cache.S16, cache.P) if t is not None]
        layers.append(layer)
    return {"step": step, "bound": n + STEPS, "layers": layers}


def run(state):
    layers = state["layers"]
    if state["step"]:
        bound = state["bound"]
        for layer in layers:
            for t, at_prompt in layer["at_prompt"]:
                t.copy_(at_prompt)
        for i in range(STEPS):
            for layer in layers:
                k, v, q, out = layer["tokens"][i]
                layer["cache"].append(k, v)
                layer["cache"].decode(q, out=out, max_context=bound)
    else:
        for layer in layers:
            for t in layer["empty"]:
                t.zero_()
            for k, v, n_new in layer["calls"]:
                layer["cache"].append(k, v, n_new=n_new)
    result = []
    for layer in layers:
        c = layer["cache"]
        result.append({"out": layer.get("out"), "groups": c.groups, "k_res": c.k_res, "v_res": c.v_res, "n_quant": c.n_quant,
                       "n_res": c.n_res, "S": c.S, "S16": c.S16, "P": c.P, "status": c.status})
    return result


def work(case):
    B, Hq, Hkv, bits = case["B"], case["Hq"], case["Hkv"], case["bits"]
    lengths = _lengths(case)
    corr = case["state"] != "none"
    record = 2 * 2048 * bits + 1024           # bytes of a group of 128 tokens of one KV head
    state16, master = 256 * 128 * 2 + 256 * 4, 256 * 128 * 4 if case["state"] == "fp32" else 0
    flush_flops = 128 * (4 * 256 * 128) if corr else 0   # one group: logits of phi_k, and S
    groups = (lengths - 1) // 128             # groups a prompt leaves behind
    if case["kind"] == "prefill":
        pairs = B * Hkv
        byts = float(lengths.sum()) * Hkv * 512 + float(groups.sum()) * Hkv * record + float((lengths - 128 * groups).sum()) * Hkv * 512
        flops = float(groups.sum()) * Hkv * flush_flops + float(lengths.sum()) * Hkv * 7 * 128
        if corr:
            byts += pairs * (state16 + master) + Hkv * 65536
        return {"bytes": byts, "flops": flops}
    byts = flops = 0.0
    for t in range(1, STEPS + 1):
        n = lengths + t
        nq = (n - 1) // 128
        nr = n - 128 * nq
        byts += float(nq.sum()) * Hkv * record + float(nr.sum()) * Hkv * 512 + B * Hq * 512 + B * Hkv * 1024
        flops += 4.0 * 128 * float(n.sum()) * Hq
        if corr:
            byts += B * Hkv * state16 + Hq * 65536
            flops += 4.0 * 128 * 256 * B * Hq
    # each sequence's one flush: its window in, a record out, the states in and out
    byts += B * Hkv * (65536 + record + ((2 * master + 2 * state16) if corr else 0))
    flops += B * Hkv * flush_flops
    return {"bytes": byts * case["layers"], "flops": flops * case["layers"]}


def tolerance(case):
    """Records, counters and window rows are the same bits (rel 0).  Outputs: fp16 results of a softmax whose operands carry
    2^-12; against the same in 64 bits they are off by 2.6e-4 (256 tokens) to 9e-4.  States: binary32 sums, 2.5e-7 from
    64-bit ones and 3e-6 of the root mean square at most; their binary16 copy then rounds a few entries the other way,
    1.2e-5 of the whole and one unit in the last place (1e-3) of such an entry, once per chunk where only that copy is kept."""
    return {"rel": 2e-3} if case["kind"] == "step" else {"rel": 6e-5, "max": 4e-3}
