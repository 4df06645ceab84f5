"""The forwards this library is measured on: sizes, inputs, the call, and what a pass cannot do without.

A case is one MoE layer on one GPU's share of the experts and one call of it:

``hidden, inter, n_experts, n_local, top_k, n_shared, shared_inter``
    the layer (M, H, E, E / eg, k, N_shared); the four layers of this repository's configurations
``tokens``    tokens handed to the call
``zipf``      exponent of a Zipf prior over the experts added to the gate scores (0 = balanced load)
``prepared``  the weights were laid out once with ``MoeEp.prepare_weights`` (a serving process keeps
              its weights); False = the call reads the caller's row-major weights
``pinned``    tokens, gate scores and outputs live in pinned host memory and cross the host link in
              the call (the stand-in for the transfers between attention and expert group)
``noalloc``   ``forward_noalloc``, the entry point of callers that keep no context
``chunks``    r_chunks;   ``interleaved``  order of the shared experts
"""
from __future__ import annotations

import math

import torch

import paper_2512_21487_amd as moe_ep

# DeepSeek-V2-Lite-shaped layer, every expert on this GPU, two shared experts
_LITE = dict(hidden=2048, inter=1408, n_experts=64, n_local=64, top_k=6, n_shared=2, shared_inter=1408)
# Qwen3-30B-A3B-shaped layer, every expert on this GPU, none shared
_QWEN30 = dict(hidden=2048, inter=768, n_experts=128, n_local=128, top_k=8, n_shared=0, shared_inter=0)
# DeepSeek-V2-shaped share: 20 of 160 experts, two shared experts on all tokens
_DSV2 = dict(hidden=5120, inter=1536, n_experts=160, n_local=20, top_k=6, n_shared=2, shared_inter=1536)
# Qwen3-235B-A22B-shaped share: 16 of 128 experts, none shared
_QWEN235 = dict(hidden=4096, inter=1536, n_experts=128, n_local=16, top_k=8, n_shared=0, shared_inter=0)


def _case(layer, tokens, *, zipf=0.0, prepared=True, pinned=False, noalloc=False, chunks=1, interleaved=False):
    return dict(layer, tokens=tokens, zipf=zipf, prepared=prepared and not noalloc, pinned=pinned, noalloc=noalloc,
                chunks=chunks, interleaved=interleaved)


def listed():
    named = {
        # one sequence being decoded: six experts and the shared ones on a single row, all latency
        "lite_decode_1": _case(_LITE, 1),
        # a few sequences decoded together, an odd number of them
        "lite_decode_33": _case(_LITE, 33),
        # a small decode step from a loop that may not allocate: no context, weights as the caller holds them
        "qwen235_noalloc_61": _case(_QWEN235, 61, noalloc=True),
        # the decode micro-batches of an expert-group member, its inputs already on the GPU
        "qwen235_decode_256": _case(_QWEN235, 256),
        "qwen235_decode_1024": _case(_QWEN235, 1024),
        # the same member fed over the host link: one small micro-batch, and a large one cut into two chunks
        # so that transfers and experts overlap
        "qwen235_pinned_256": _case(_QWEN235, 256, pinned=True),
        "qwen235_pinned_4096": _case(_QWEN235, 4096, pinned=True, chunks=2),
        # prefill of one long prompt, or of a batch of short ones, on a layer that fits one GPU
        "lite_prefill_4096": _case(_LITE, 4096),
        # a ragged prefill by a caller that rewrites its weights (fine-tuning) and so keeps no prepared copy
        "lite_ragged_1531": _case(_LITE, 1531, prepared=False),
        # prefill with the skewed expert load real routers show: some experts empty, some with thousands of rows
        "qwen30_skewed_8192": _case(_QWEN30, 8192, zipf=1.1),
        # prefill share of a large model: the benchmark's layer, and a part of it in two interleaved chunks
        "dsv2_share_16384": _case(_DSV2, 16384),
        "dsv2_chunked_5003": _case(_DSV2, 5003, chunks=2, interleaved=True),
    }
    return [dict(case, name=name) for name, case in named.items()]


# layer and the largest token count it is handed
_RANGES = ((_LITE, 4096), (_QWEN30, 8192), (_DSV2, 16384), (_QWEN235, 4096))


def draw(rng):
    """One more forward of the same ranges: any of the layers, from one token to its largest micro-batch."""
    layer, top = rng.choice(_RANGES)
    tokens = max(1, min(top, round(math.exp(rng.uniform(0.0, math.log(top))))))
    pinned = layer is not _DSV2 and rng.random() < 0.25
    # chunks are for calls with something to overlap, and repeat the weight stream: not on the largest ones
    chunks = rng.choice((1, 1, 2, 4)) if 256 <= tokens <= 5120 else 1
    noalloc = layer is _QWEN235 and not pinned and tokens <= 128 and chunks == 1 and rng.random() < 0.5
    return _case(layer, tokens, zipf=1.1 if layer is _QWEN30 and rng.random() < 0.7 else 0.0,
                 prepared=rng.random() < 0.75, pinned=pinned, noalloc=noalloc, chunks=chunks,
                 interleaved=layer["n_shared"] > 0 and rng.random() < 0.5)


def _on_host(x):
    host = torch.empty(x.shape, dtype=x.dtype, pin_memory=True)
    host.copy_(x)
    return host


def _inputs(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    T, M, E = case["tokens"], case["hidden"], case["n_experts"]

    def normal(n, std):
        return torch.empty(n, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=gen)

    # activations behind a normalisation, weights at the usual initialisation scale
    tokens = normal(T * M, 1.0).view(T, M)
    scores = torch.empty((T, E), dtype=torch.float32, device="cuda").normal_(generator=gen)
    if case["zipf"] > 0.0:
        rank = torch.randperm(E, generator=gen, device="cuda").double() + 1.0
        scores += (-case["zipf"] * torch.log(rank)).float()
    routed = normal(case["n_local"] * 3 * case["inter"] * M, 0.02)
    shared = normal(case["n_shared"] * 3 * case["shared_inter"] * M, 0.02) if case["n_shared"] else None
    return tokens, scores, routed, shared


def prepare(case, seed):
    T, M, E = case["tokens"], case["hidden"], case["n_experts"]
    tokens, scores, routed, shared = _inputs(case, seed)
    out = torch.zeros((T, M), dtype=torch.bfloat16, device="cuda")
    io_mode = moe_ep.IO_DEVICE
    if case["pinned"]:
        tokens, scores, out = _on_host(tokens), _on_host(scores), _on_host(out)
        io_mode = moe_ep.IO_PINNED_HOST
    layer = dict(hidden=M, inter=case["inter"], n_experts=E, n_local=case["n_local"], n_shared=case["n_shared"],
                 shared_inter=case["shared_inter"], max_tokens=T, max_top_k=case["top_k"], max_chunks=case["chunks"],
                 io_mode=io_mode, device=0)
    if case["noalloc"]:
        ctx = moe_ep.MoeEpConfig(local_begin=0, **layer)
    else:
        ctx = moe_ep.MoeEp(**layer)
        if case["prepared"]:
            ctx.prepare_weights(routed, shared)
    order = moe_ep.ORDER_INTERLEAVED if case["interleaved"] else moe_ep.ORDER_SHARED_FIRST
    return dict(ctx=ctx, noalloc=case["noalloc"], out=out,
                args=(tokens, scores, routed, shared, case["top_k"], case["chunks"], order))


def run(state):
    if state["noalloc"]:
        moe_ep.forward_noalloc(state["ctx"], *state["args"], out=state["out"])
    else:
        state["ctx"].forward(*state["args"], out=state["out"])
    return state["out"]


def work(case):
    T, M, H, E, El, k = (case[n] for n in ("tokens", "hidden", "inter", "n_experts", "n_local", "top_k"))
    Ns, Hs = case["n_shared"], case["shared_inter"]
    rows = T * k * El / E                                  # assignments expected to stay on this GPU
    experts = El * (1.0 - (1.0 - k / E) ** T)              # local experts expected to receive a row
    nothing_kept = 1.0                                     # share of the tokens no local expert sees
    for i in range(k):
        nothing_kept *= max(0.0, (E - El - i) / (E - i))
    token_rows = T if Ns else T * (1.0 - nothing_kept)
    return {"bytes": 2.0 * M * (token_rows + T) + 4.0 * T * E + 2.0 * 3 * M * (H * experts + Hs * Ns),
            "flops": 6.0 * M * (H * rows + Hs * Ns * T)}


def tolerance(case):
    # bf16 inputs and results, activation and expert outputs rounded to bf16 once each, sums in fp32: against
    # the same layer in fp32 with fp64 sums over the experts, 20 cases showed 2.6e-3 .. 2.9e-3 of the norm and a
    # largest difference of 0.9e-2 .. 2.7e-2 (on the shares, where few experts of a token are here, the rounded
    # activation alone gives 1.5e-2); about four times that.
    return {"rel": 1e-2, "max": 0.1}


def exact(case, seed):
    """The layer in float64: gate over all experts, the local ones' SwiGLU projections, the weighted sum."""
    tokens, scores, routed, shared = _inputs(case, seed)
    T, M, k = case["tokens"], case["hidden"], case["top_k"]
    x = tokens.double()

    def ffn(rows, weights, inter):
        gate, up, down = weights.view(3, -1)
        gate, up, down = gate.view(inter, M).double(), up.view(inter, M).double(), down.view(M, inter).double()
        z = rows @ gate.t()
        return (z * torch.sigmoid(z) * (rows @ up.t())) @ down.t()

    # equal scores go to the lower expert
    top, chosen = torch.sort(scores, dim=1, descending=True, stable=True)
    top, chosen = torch.softmax(top[:, :k].double(), dim=1), chosen[:, :k]
    out = torch.zeros((T, M), dtype=torch.float64, device="cuda")
    for e, weights in enumerate(routed.view(case["n_local"], -1)):
        row, slot = torch.nonzero(chosen == e, as_tuple=True)
        if row.numel():
            out.index_add_(0, row, top[row, slot, None] * ffn(x[row], weights, case["inter"]))
    if case["n_shared"]:
        for weights in shared.view(case["n_shared"], -1):
            out += ffn(x, weights, case["shared_inter"])
    return out.cpu() if case["pinned"] else out
