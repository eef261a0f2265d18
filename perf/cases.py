"""Timed cases of the MoE-offloading decode and prefill paths.

Each case is one call sequence a user of `offload.OffloadedMoE` makes: decoding
a few tokens through a stack (`decode`), or taking a batch of tokens through it
(`prefill`, which is also batched decode).  The sizes are those of the
package's own configurations (`workload.CONFIGS`): the tiny fp32 stack, the
Mixtral-shaped layer (8 experts, top-2, d 4096, d_ff 14336) and the 64-expert
layer (top-8, d 2048, d_ff 1408); `draw` spreads over what lies between and
around them.

Weights are N(0, 0.02^2), drawn on the GPU from the seed one expert at a time,
so that `exact` can draw the same ones again; hidden states come from
`workload.hidden_states` (Zipf-distributed concepts with Markov persistence).
"""
from __future__ import annotations

import math
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import torch

from paper_2511_05814_amd import binding, entropy, offload, workload as wl

TINY = dict(dtype="f32", layers=2, experts=8, top_k=2, d_model=256, d_ff=512)
FINE = dict(dtype="bf16", layers=1, experts=64, top_k=8, d_model=2048, d_ff=1408)
MIXTRAL = dict(dtype="bf16", layers=1, experts=8, top_k=2, d_model=4096, d_ff=14336)


def _case(name, model, mode, slots, tokens, **options):
    return {"name": name, "mode": mode, "slots": slots, "tokens": tokens, "policy": "lfu", "prefetch": 0,
            "store": "plain", **model, **options}


def listed():
    return [
        # the smallest stack: fp32 experts of 1.5 MB, half of them resident, so
        # launches and small copies are what a token costs
        _case("decode-tiny-f32", TINY, "decode", slots=4, tokens=8),
        # one token through two 64-expert layers held whole in HBM: the latency of a single decode step
        _case("decode-fine-one", FINE, "decode", slots=64, tokens=1, layers=2),
        # Mixtral-shaped decode with every expert resident (the whole model fits one card's HBM)
        _case("decode-mixtral", MIXTRAL, "decode", slots=8, tokens=4),
        # the same with the paper's 2-bit group-quantised experts
        _case("decode-mixtral-q2", MIXTRAL, "decode", slots=8, tokens=4, dtype="q2g16"),
        # the paper's setting: half of the experts resident, misses over the host link
        _case("decode-mixtral-offload", MIXTRAL, "decode", slots=4, tokens=4),
        # 64-expert decode with next-layer speculation from an entropy-coded host store
        _case("decode-fine-offload", FINE, "decode", slots=16, tokens=4, layers=2, prefetch=2, store="entropy"),
        # batched decode of 8 sequences, every expert resident
        _case("batch8-mixtral", MIXTRAL, "batch", slots=8, tokens=8),
        # batched decode of 32 sequences over 64 experts
        _case("batch32-fine", FINE, "batch", slots=64, tokens=32),
        # a short prompt of ragged length
        _case("prefill509-fine", FINE, "batch", slots=64, tokens=509),
        # the 64-expert workload's own prompt length
        _case("prefill4096-fine", FINE, "batch", slots=64, tokens=4096),
        # a long prompt through the Mixtral-shaped layer
        _case("prefill2048-mixtral", MIXTRAL, "batch", slots=8, tokens=2048),
        # a prompt while a quarter of the experts are resident: the others stream in over the host link
        _case("prefill1024-fine-offload", FINE, "batch", slots=16, tokens=1024),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """A case between and around the listed ones: odd multiples of 8 among the
    sizes (of 64 for 2-bit experts), odd expert and token counts."""
    mode = rng.choice(("decode", "batch"))
    dtype = "bf16" if mode == "batch" else rng.choice(("bf16", "bf16", "q2g16", "f32"))
    odd = rng.random() < 0.5
    unit = 64 if dtype == "q2g16" else (8 if odd else 128)

    def size(lo, hi):
        return max(unit, int(_log(rng, lo, hi)) // unit * unit)

    d, f = size(256, 4096), size(256, 14336)
    experts = rng.randint(4, 64)
    layers = rng.choice((1, 2)) if mode == "decode" else 1
    probe = wl.Config("size", 0, 1, 1, 1, d, f, dtype, 1, (1,), ("lfu",), 1.1, 0.6)
    # the store stays below that of one Mixtral-shaped layer
    experts = max(2, min(experts, (2800 << 20) // (layers * probe.expert_bytes)))
    k = rng.randint(1, min(8, experts))
    if mode == "decode":
        tokens = rng.randint(1, 4)
    else:
        top = min(4096, 1.4e12 / (6.0 * d * f * k))  # no more work than the largest listed case
        tokens = max(1, int(_log(rng, 1, top)))
    slots = experts if rng.random() < 0.7 else rng.randint(k, experts)
    policy = rng.choice(("lfu", "lru", "lfu-aged:32"))
    prefetch = rng.randint(0, min(2, k)) if mode == "decode" and layers > 1 else 0
    coded = dtype == "bf16" and slots < experts and d * f % 512 == 0 and rng.random() < 0.3
    return dict(mode=mode, dtype=dtype, layers=layers, experts=experts, top_k=k, d_model=d, d_ff=f, slots=slots,
                tokens=tokens, policy=policy, prefetch=prefetch, store="entropy" if coded else "plain")


def _config(case, seed):
    return wl.Config("case", seed, case["layers"], case["experts"], case["top_k"], case["d_model"], case["d_ff"],
                     case["dtype"], case["tokens"], (case["slots"],), (case["policy"],), 1.2, 0.6,
                     prefetch_max=case["prefetch"])


def _normal(seed, tag, *shape):
    g = torch.Generator(device="cuda")
    g.manual_seed((seed * 7919 + tag) % (1 << 62))
    return torch.randn(*shape, generator=g, device="cuda") * wl.WEIGHT_STD


def _quantise(w):
    """2-bit codes, fp16 scales and zero codes of groups of 16 columns."""
    rows, cols = w.shape
    g = w.view(rows, cols // 16, 16)
    lo, hi = g.amin(2), g.amax(2)
    s = ((hi - lo) / 3).half()
    z = (-lo / s.float() * wl.Q_ZERO_STEPS).round().clamp(0, 255)
    q = (g / s.float()[..., None] + (z / wl.Q_ZERO_STEPS)[..., None]).round().clamp(0, 3).view(rows, cols)
    return q.to(torch.uint8), s, z.to(torch.uint8)


def _expert(case, seed, layer, expert):
    """The three matrices (W1, W3, W2) of one expert: bytes as stored, and a
    function that widens matrix j to fp64."""
    d, f, dtype = case["d_model"], case["d_ff"], case["dtype"]
    mats = []
    for j, shape in enumerate(((f, d), (f, d), (d, f))):
        w = _normal(seed, 3 * (64 * layer + expert) + j + 1000, *shape)
        mats.append(w if dtype == "f32" else w.bfloat16() if dtype == "bf16" else _quantise(w))
    if dtype != "q2g16":
        return [m.view(torch.uint8).view(-1) for m in mats], lambda j: mats[j].double()

    def stored(q, s, z):
        c = q.view(q.shape[0], -1, 4)
        c = c[..., 0] | (c[..., 1] << 2) | (c[..., 2] << 4) | (c[..., 3] << 6)
        return torch.cat([c.reshape(-1), s.reshape(-1).view(torch.uint8), z.reshape(-1)])

    def wide(j):
        q, s, z = mats[j]
        g = q.double().view(*s.shape, 16) - (z.double() / wl.Q_ZERO_STEPS)[..., None]
        return (g * s.double()[..., None]).view(q.shape)

    return [stored(*m) for m in mats], wide


def _gates(case, seed):
    g = _normal(seed, 1, case["layers"], case["experts"], case["d_model"])
    return g if case["dtype"] == "f32" else g.bfloat16()


def prepare(case, seed):
    cfg = _config(case, seed)
    L, E, n = cfg.layers, cfg.experts, cfg.matrix_elems
    coded = case["store"] == "entropy"
    store = offload.HostStore(cfg, fill=False, fmt=case["store"], cap=entropy.default_cap_words(n) if coded else None)
    jobs = []
    with ThreadPoolExecutor(16) as pool:
        for layer in range(L):
            rows = store.layer_array(layer).reshape(E, -1)
            for e in range(E):
                raw = torch.cat(_expert(case, seed, layer, e)[0])
                if not coded:
                    torch.from_numpy(rows[e]).copy_(raw)
                    continue
                mats = raw.cpu().numpy().view(np.uint16).reshape(3, n)
                jobs += [pool.submit(entropy.pack_matrix, mats[j], store.cap,
                                     rows[e][j * store.matrix_stride:(j + 1) * store.matrix_stride])
                         for j in range(3)]
    for j in jobs:
        j.result()
    g = _gates(case, seed)
    gates = offload.DeviceGates(cfg, g.cpu().numpy() if case["dtype"] == "f32" else
                                g.view(torch.int16).cpu().numpy().view(np.uint16))
    batch = case["mode"] == "batch"
    start = torch.from_numpy(wl.hidden_states(cfg, cfg.tokens)).cuda()
    moe = offload.OffloadedMoE(cfg, store, gates, case["slots"], case["policy"], prefetch_max=cfg.prefetch_max,
                               max_prefill_tokens=cfg.tokens if batch else 0)
    return dict(moe=moe, start=start, h=torch.empty_like(start), batch=batch,
                flags=binding.MOE_PREFETCH_NEXT if cfg.prefetch_max else 0)


def run(state):
    moe, h = state["moe"], state["h"]
    with torch.cuda.stream(moe.compute):  # the program works on the handle's own compute stream
        h.copy_(state["start"])
        if state["batch"]:
            moe.prefill(h)
        else:
            moe.decode(h, flags=state["flags"])
    return h


def work(case):
    cfg = _config(case, 0)
    T, L, E, K, d, f = cfg.tokens, cfg.layers, cfg.experts, cfg.top_k, cfg.d_model, cfg.d_ff
    gate = E * d * (4 if cfg.dtype == "f32" else 2)
    flops = L * T * (2.0 * E * d + 6.0 * K * d * f)
    if case["mode"] == "decode":  # a token's experts are known only when it gets there: read once a token
        return dict(bytes=float(L * T * (gate + K * cfg.expert_bytes + 8 * d)), flops=flops)
    used = E * (1.0 - (1.0 - K / E) ** T)  # experts a batch of evenly routed tokens needs
    return dict(bytes=float(L * (gate + used * cfg.expert_bytes + 8 * T * d)), flops=flops)


def _share(case):
    """About what share of the result's norm the experts' sum has (weights g of
    about 1 / top_k each): the rest is the residual, which both sides carry
    unchanged."""
    s2 = wl.WEIGHT_STD ** 2 * case["d_model"]
    y = wl.WEIGHT_STD * math.sqrt(case["d_ff"] / case["top_k"]) * 0.6 * s2
    return y / math.sqrt(y * y + 2.0)


def tolerance(case):
    # The batch path takes bf16 activations on the matrix cores: 3e-3 of the
    # experts' sum, 2.9e-4 of the result at the 64-expert shape and 2.3e-3 at
    # the Mixtral shape, where the sum dominates.  Decode keeps fp32
    # activations and sums: 4e-8 to 2.6e-7.  Four times that.
    if case["mode"] == "batch":
        return {"rel": 1.2e-2 * _share(case)}
    return {"rel": 1e-6}


def exact(case, seed):
    cfg = _config(case, seed)
    h = torch.from_numpy(wl.hidden_states(cfg, cfg.tokens)).cuda().double()
    gates = _gates(case, seed).double()
    for layer in range(cfg.layers):
        r = (h.square().mean(1, keepdim=True) + 1e-5).sqrt()
        z, ids = (h @ gates[layer].T).sort(dim=1, descending=True, stable=True)
        z, ids = z[:, :cfg.top_k], ids[:, :cfg.top_k]
        g = torch.softmax(z / r, 1)
        x, y = h / r, torch.zeros_like(h)
        for e in range(cfg.experts):
            t, rank = (ids == e).nonzero(as_tuple=True)
            if t.numel() == 0:
                continue
            wide = _expert(case, seed, layer, e)[1]
            a = x[t] @ wide(0).T
            a = a * torch.sigmoid(a) * (x[t] @ wide(1).T)
            y.index_add_(0, t, g[t, rank][:, None] * (a @ wide(2).T))
        h = h + y
    return h
