"""The layer's work as users give it, for timing: whole calls of MoEExpertLayer.forward on seeded synthetic
inputs, from one decoder token to the largest batch, and the quantisation of a layer's expert weights.

The sizes are the ones this repository's configurations, tests and benchmark use (workloads.py: the paper's
model with d_model 1024, d_ff 4096 and 32 experts, and the workloads built on it) and generic ones beside them."""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2211_10017_amd import MoEExpertLayer, binding

_ACT = {"f16": torch.float16, "bf16": torch.bfloat16}


def _layer(name=None, **kw):
    case = dict(op="layer", T=64, d=1024, F=4096, E=32, k=2, bits=4, group=0, act="f16", activation="relu", bias=False,
                load="even", finished=0.0)
    case.update(kw)
    return dict(name=name, **case) if name else case


def _quantize(name=None, **kw):
    case = dict(op="quantize", E=32, K=1024, N=4096, bits=4, group=0, canon=False)
    case.update(kw)
    return dict(name=name, **case) if name else case


def listed():
    return [
        # one sentence, beam 1, one decoder step: the smallest call, launches and latency
        _layer("decode_1_int4", T=1),
        # the paper's Table 1: about 40 decoder tokens, 8-bit experts, one expert per token
        _layer("decode_40_int8", T=40, k=1, bits=8),
        # the benchmark's headline: a beam batch of 64 tokens, 4-bit experts
        _layer("decode_64_int4", T=64),
        # the largest decoder batch of the paper's tables (96 sentences, beam 2), a third of the rows already ended
        _layer("decode_192_int4_pruned", T=192, finished=0.33),
        # decoding with the large group-quantised layer
        _layer("decode_64_group", T=64, d=4096, F=16384, E=64, group=128),
        # a small 8-bit layer with one expert per token (workload c1)
        _layer("small_256_int8", T=256, d=512, F=2048, E=8, k=1, bits=8),
        # a ragged batch of sentences through a bf16 encoder layer with biases and GELU
        _layer("ragged_997_bf16", T=997, d=768, F=3072, E=16, bits=8, act="bf16", activation="gelu", bias=True),
        # an encoder batch, unevenly loaded experts (workload c3)
        _layer("encoder_16384_int4", T=16384, E=64, k=1, load="uneven"),
        # skewed routing over many 8-bit experts, a few of them without rows (workload c4)
        _layer("skewed_4096_int8", T=4096, d=2048, F=8192, E=128, bits=8, load="skewed"),
        # the largest layer, group-wise scales, in both activation types (workload c5)
        _layer("large_8192_f16", T=8192, d=4096, F=16384, E=64, group=128),
        _layer("large_8192_bf16", T=8192, d=4096, F=16384, E=64, group=128, act="bf16"),
        # loading a model: one weight tensor of the paper's layer from its fp32 masters
        _quantize("quantize_int4"),
    ]


_SHAPES = [(512, 2048), (768, 3072), (1024, 4096), (2048, 8192), (4096, 16384)]
_MAX_FLOPS = 4.3e12          # the largest listed case
_MAX_WEIGHT_BYTES = 4.3e9


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode"] * 3 + ["prefill"] * 3 + ["quantize"])
    if kind == "quantize":
        d, F = rng.choice(_SHAPES[:4])
        K, N = rng.choice([(d, F), (F, d)])
        bits = rng.choice([4, 8])
        E = _log_int(rng, 1, max(1, min(64, (1 << 28) // (K * N))))
        return _quantize(E=E, K=K, N=N, bits=bits, group=rng.choice([0, 0, 128]), canon=rng.random() < 0.25)
    while True:
        d, F = rng.choice(_SHAPES)
        E = rng.choice([8, 16, 32, 64, 128])
        k = rng.choice([1, 2])
        bits = rng.choice([4, 4, 8])
        T = _log_int(rng, 1, 256) if kind == "decode" else _log_int(rng, 257, 16384)
        group = 128 if bits == 4 and rng.random() < 0.3 else 0
        act = "bf16" if rng.random() < 0.25 else "f16"
        if 4.0 * T * k * d * F <= _MAX_FLOPS and E * 2 * d * F * bits / 8 <= _MAX_WEIGHT_BYTES:
            break
    return _layer(T=T, d=d, F=F, E=E, k=k, bits=bits, group=group, act=act,
                  activation=rng.choice(["relu", "relu", "gelu"]), bias=rng.random() < 0.3,
                  load="even" if kind == "decode" else rng.choice(["even", "uneven", "skewed"]),
                  finished=rng.choice([0.0, 0.0, rng.uniform(0.1, 0.6)]) if kind == "decode" and T > 8 else 0.0)


def _gate_bias(case, seed):
    """The router bias of workloads.py: none, uniform (loads within about 2x of the mean) or Zipf popularity with one expert in
    twenty switched off (a few experts take much of the load, some take none)."""
    rng = np.random.Generator(np.random.Philox(key=[seed, 2]))
    E = case["E"]
    if case["load"] == "even":
        return None
    if case["load"] == "uneven":
        return torch.from_numpy(rng.uniform(-0.18, 0.18, E).astype(np.float32)).cuda()
    z = rng.zipf(1.2, E).astype(np.float64)
    b = (0.09 * np.log(z)).astype(np.float32)
    b[np.lexsort((np.arange(E), z))[:E // 20]] = -30.0
    return torch.from_numpy(b).cuda()


def _expert_masters(gen, K, N):
    return torch.randn((K, N), generator=gen, device="cuda", dtype=torch.float32).mul_(0.02)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if case["op"] == "quantize":
        w = torch.randn((case["E"], case["K"], case["N"]), generator=gen, device="cuda", dtype=torch.float32).mul_(0.02)
        return {"case": case, "w": w}
    T, d, F, E, act = case["T"], case["d"], case["F"], case["E"], _ACT[case["act"]]
    layer = MoEExpertLayer(T, d, F, E, case["k"], case["bits"], case["group"], act_dtype=act, activation=case["activation"])
    layer.wg.copy_(torch.randn((d, E), generator=gen, device="cuda").mul_(0.02))
    layer.gate_bias = _gate_bias(case, seed)
    if case["bias"]:
        layer.b1 = torch.randn((E, F), generator=gen, device="cuda").mul_(0.02).half()
        layer.b2 = torch.randn((E, d), generator=gen, device="cuda").mul_(0.02).half()
    for e in range(E):
        layer.load_expert(1, e, _expert_masters(gen, d, F))
        layer.load_expert(2, e, _expert_masters(gen, F, d))
    x = torch.randn((T, d), generator=gen, device="cuda").to(act)
    finished = None
    if case["finished"]:
        finished = torch.zeros(T, dtype=torch.uint8, device="cuda")
        finished[torch.randperm(T, generator=gen, device="cuda")[:max(1, round(case["finished"] * T))]] = 1
    return {"case": case, "layer": layer, "x": x, "finished": finished}


def run(state):
    case = state["case"]
    if case["op"] == "quantize":
        canon, scales, packed = binding.moe_quantize_experts(state["w"], case["bits"], case["group"], want_canon=case["canon"])
        return {"canon": canon, "scales": scales, "packed": packed}
    layer = state["layer"]
    out = layer.forward(state["x"], state["finished"])
    return {"out": out, "expert_idx": layer.expert_idx, "expert_scale": layer.expert_scale}


def _active(case):
    """Experts that rows reach: all that a draw of T * k assignments over the experts in use is expected to touch."""
    E = case["E"] - (case["E"] // 20 if case["load"] == "skewed" else 0)
    R = (case["T"] - round(case["finished"] * case["T"])) * case["k"]
    return E * (1.0 - (1.0 - 1.0 / E) ** R) if E > 1 else 1.0


def work(case):
    if case["op"] == "quantize":
        n = case["E"] * case["K"] * case["N"]
        groups = case["K"] // (case["group"] or case["K"])
        return {"bytes": n * 4 + n * case["bits"] / 8 * (2 if case["canon"] else 1) + 2 * case["E"] * groups * case["N"], "flops": 0}
    T, d, F, E, k = case["T"], case["d"], case["F"], case["E"], case["k"]
    live = T - round(case["finished"] * T)
    g1, g2 = (case["group"] or d), (case["group"] or F)
    expert = 2 * d * F * case["bits"] / 8 + 2 * (d // g1 * F + F // g2 * d) + (2 * (d + F) if case["bias"] else 0)
    return {"bytes": _active(case) * expert + 2 * d * E + 2 * T * d + 4 * T * d + 8 * T * k,
            "flops": 4.0 * live * k * d * F + 2.0 * T * d * E}


def tolerance(case):
    """Four times what the layer's output was measured to be away from the same layer in 64 bits, with h rounded to the
    activation type in both. FP16: y is rounded to FP16 (2.1e-4, largest difference 1.8e-3); group scales: the weights are as
    well (3.9e-4, 2.0e-3); bf16: y stays in 32 bits (2.5e-5, 1.6e-3; with group scales 1.7e-4, 1.1e-3). The routing is exact."""
    if case["op"] == "quantize":
        return "exact"
    if case["act"] == "bf16":
        return {"rel": 7e-4, "max": 6e-3} if case["group"] else {"rel": 1e-4, "max": 6e-3}
    return {"rel": 1.6e-3, "max": 8e-3} if case["group"] else {"rel": 8e-4, "max": 8e-3}
