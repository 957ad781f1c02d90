"""The calls whose speed this repository answers for, as a program that serves or prepares a W4A8KV4 model makes them.

Four kinds of work, all through the public functions of paper_2405_04532_amd.api, called eagerly:

  linear   FP16 activations through one quantized layer: the activation quantizer and the W4A8 GEMM
  decode   one generation step of one decoder layer: the fused producers and the quantizer, the layer's GEMMs, one token
           per sequence appended to the 4-bit KV cache, and attention over the cache
  prefill  the same layer over whole prompts (attention over a prompt is not part of this framework: its result is an
           input here)
  load     one layer's FP16 weights on their way to the packed form: as they are, rotated, or with the input channels
           reordered by the salience that calibration activations give them

Rotary embedding and residual additions are the calling program's own, so queries, keys, values and the residual stream
are inputs.  Weights and activations are synthetic: normal values with 1% of outlier channels, the structure that the
method is built for.  Token counts, widths, batch sizes and contexts are spread over what these models are served with:
1 to 4096 tokens in a call, 1 to 64 sequences, contexts of 64 to 8192 tokens.
"""
import math

import torch

from paper_2405_04532_amd import api
from paper_2405_04532_amd import workloads as wl

D = 128                                     # head dimension of every model here
EPS = 1e-5

FAMILIES = {
    "llama2_7b": dict(layers=wl.LLAMA2_7B, mode=api.QOQ_GROUP128, **wl.KV4_DECODE["llama2_7b"]),
    "llama3_70b": dict(layers=wl.LLAMA3_70B, mode=api.QOQ_GROUP128, **wl.KV4_DECODE["llama3_70b"]),
    "llama3_8b": dict(layers=dict(wl.LLAMA3_8B, o=(4096, 4096)), mode=api.QOQ_PER_CHANNEL, **wl.KV4_DECODE["llama3_8b"]),
}


# ------------------------------------------------------------------------------------------------------------------
# The cases
# ------------------------------------------------------------------------------------------------------------------
def listed():
    return [
        # the smallest layer of the test configurations: launches and host work only
        dict(name="linear-16x256x256", kind="linear", M=16, K=256, N=256, mode=0, form="linear"),
        # a single token through one projection, per-channel weights: interactive use, one request in flight
        dict(name="linear-1x4096x6144-pc", kind="linear", M=1, K=4096, N=6144, mode=1, form="linear"),
        # a ragged chunk of prompt tokens through a long-K layer whose input channels were reordered offline
        dict(name="linear-389x11008x4096-reordered", kind="linear", M=389, K=11008, N=4096, mode=0, form="reordered"),
        # a ragged chunk through a wide per-channel layer, zero points folded through the token sums
        dict(name="linear-130x4096x28672-tokensum", kind="linear", M=130, K=4096, N=28672, mode=1, form="token_sum"),
        # generation for one user: every call is latency
        dict(name="decode-7b-1x1023", kind="decode", family="llama2_7b", batch=1, context=1023),
        # generation for a full batch at the context the attention benchmark uses
        dict(name="decode-7b-64x1024", kind="decode", family="llama2_7b", batch=64, context=1024),
        # few sequences with long contexts, grouped-query heads: the cut-up attention
        dict(name="decode-8b-4x8192", kind="decode", family="llama3_8b", batch=4, context=8192),
        # a batch of ordinary requests on the largest model
        dict(name="decode-70b-37x700", kind="decode", family="llama3_70b", batch=37, context=700),
        # one ordinary prompt
        dict(name="prefill-7b-1x1024", kind="prefill", family="llama2_7b", batch=1, tokens=1024),
        # two prompts batched together on the largest model: the most work in one pass
        dict(name="prefill-70b-2x1024", kind="prefill", family="llama3_70b", batch=2, tokens=1024),
        # preparing a model: a block input module's weights, rotated and packed in groups of 128
        dict(name="load-22016x4096-rotated", kind="load", N=22016, K=4096, mode=0, step="rotate"),
        # preparing a model: calibration, channel reordering and packing of a long-K layer, per channel
        dict(name="load-4096x14336-reordered-pc", kind="load", N=4096, K=14336, mode=1, step="reorder"),
    ]


def _log_int(rng, lo, hi, step=1):
    """An integer from lo to hi, uniform in its logarithm, rounded down to a multiple of `step`."""
    v = int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))
    return max(lo, min(hi, v) // step * step)


def draw(rng):
    kind = rng.choice(("linear", "linear", "decode", "decode", "prefill", "load"))
    if kind == "linear":
        mode = rng.randint(0, 1)
        K, N = _log_int(rng, 256, 14336, 128), _log_int(rng, 256, 28672, 64)
        form = rng.choice(("linear", "linear", "reordered") if mode == 0 else ("linear", "linear", "token_sum"))
        return dict(kind=kind, M=_log_int(rng, 1, 2048), K=K, N=N, mode=mode, form=form)
    if kind == "decode":
        family = rng.choice(sorted(FAMILIES))
        batch = _log_int(rng, 1, 64)
        most = min(8192, 64 * 1024 * 32 // (batch * FAMILIES[family]["Hkv"]))
        return dict(kind=kind, family=family, batch=batch, context=_log_int(rng, 64, most))
    if kind == "prefill":
        family = rng.choice(sorted(FAMILIES))
        total = _log_int(rng, 128, 1024 if family == "llama3_70b" else 4096)
        batch = _log_int(rng, 1, 8)
        return dict(kind=kind, family=family, batch=batch, tokens=max(16, total // batch))
    mode = rng.randint(0, 1)
    return dict(kind=kind, N=_log_int(rng, 1024, 28672, 64), K=_log_int(rng, 1024, 14336, 128), mode=mode,
                step=rng.choice(("plain", "rotate", "reorder")))


# ------------------------------------------------------------------------------------------------------------------
# Inputs
# ------------------------------------------------------------------------------------------------------------------
def _normal(g, *shape):
    return torch.randn(shape, generator=g, device=g.device, dtype=torch.float16)


def _weights(g, N, K):
    w = _normal(g, N, K) * 0.02
    w[torch.randperm(N, generator=g, device=g.device)[: max(1, N // 100)]] *= 10.0
    return w


def _activations(g, M, K):
    x = _normal(g, M, K)
    cols = torch.randperm(K, generator=g, device=g.device)[: max(1, K // 100)]
    x[:, cols] *= 20.0
    return x


def _keys(g, *shape):
    k = _normal(g, *shape)                  # [..., Hkv, D]: two large channels in every KV head
    for h in range(shape[-2]):
        cols = torch.randperm(D, generator=g, device=g.device)[:2]
        k[..., h, cols] *= 8.0
    return k


class _Layer:
    """Packed weights of one linear layer with the output and the workspace that a serving program keeps beside them."""

    def __init__(self, g, M, K, N, mode):
        self.N, self.mode = N, mode
        self.packed = api.pack_weights(_weights(g, N, K), mode)
        self.out = torch.empty((M, N), dtype=torch.float16, device=g.device)
        self.workspace = api.new_workspace(api.gemm_workspace_bytes(M, N, K, mode), g.device)

    def gemm(self, qx, sx, rowsum):
        return api.w4a8_gemm(qx, sx, self.packed, self.N, self.mode, rowsum=rowsum, out=self.out, workspace=self.workspace)


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    kind = case["kind"]
    s = dict(case)
    if kind == "linear":
        M, K, N = case["M"], case["K"], case["N"]
        s["layer"] = _Layer(g, M, K, N, case["mode"])
        s["x"] = _activations(g, M, K)
        s["qx"] = torch.empty((M, K), dtype=torch.int8, device="cuda")
        s["sx"] = torch.empty(M, dtype=torch.float16, device="cuda")
        s["rowsum"] = torch.empty(M, dtype=torch.int32, device="cuda")
        s["perm"] = torch.randperm(K, generator=g, device="cuda").to(torch.int32)
        return s
    if kind == "load":
        s["w"] = _weights(g, case["N"], case["K"])
        s["calibration"] = _activations(g, 1024, case["K"]) if case["step"] == "reorder" else None
        return s
    f = FAMILIES[case["family"]]
    B, H, Hkv, mode = case["batch"], f["H"], f["Hkv"], f["mode"]
    T = 1 if kind == "decode" else case["tokens"]
    M = B * T
    for name, (K, N) in f["layers"].items():
        s[name] = _Layer(g, M, K, N, mode)
    hidden = f["layers"]["qkv"][0]
    s["x1"], s["x2"] = _activations(g, M, hidden), _activations(g, M, hidden)
    s["gamma1"] = 1.0 + 0.1 * _normal(g, hidden)
    s["gamma2"] = 1.0 + 0.1 * _normal(g, hidden)
    s["k"], s["v"] = _keys(g, B, T, Hkv, D), _normal(g, B, T, Hkv, D)
    if kind == "prefill":
        s["S_max"] = T + 64                 # room for the answer
        s["cache"] = api.kv4_new_cache(B, Hkv, s["S_max"], "cuda")
        s["positions"] = torch.zeros(B, dtype=torch.int32, device="cuda")
        s["attention"] = _normal(g, M, H * D)
        return s
    S = s["S_max"] = case["context"]
    s["cache"] = api.kv4_new_cache(B, Hkv, S, "cuda")
    api.kv4_append(s["cache"], _keys(g, B, S, Hkv, D), _normal(g, B, S, Hkv, D),
                   torch.zeros(B, dtype=torch.int32, device="cuda"), S)
    lens = torch.randint(S // 2, S + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    lens[0] = S
    s["seq_lens"], s["positions"] = lens, lens - 1
    s["q"] = _normal(g, B, H, D)
    s["attention"] = torch.empty((B, H, D), dtype=torch.float16, device="cuda")
    need = api.kv4_attention_workspace_bytes(B, H, Hkv, S)
    s["attention_workspace"] = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None
    return s


# ------------------------------------------------------------------------------------------------------------------
# One pass
# ------------------------------------------------------------------------------------------------------------------
def _run_linear(s):
    layer = s["layer"]
    if s["form"] == "linear":
        out, qx, sx, rowsum = api.w4a8_linear(s["x"], layer.packed, layer.N, layer.mode, out=layer.out, qx=s["qx"], sx=s["sx"],
                                              rowsum=s["rowsum"], workspace=layer.workspace)
        return out, qx, sx, rowsum
    if s["form"] == "reordered":
        qx, sx, _, _ = api.quant_act_per_token_reordered(s["x"], s["perm"], want_rowsum=False)
        return layer.gemm(qx, sx, None), qx, sx
    qx, sx, _, tx = api.quant_act_per_token(s["x"], want_rowsum=False, want_tx=True)
    out = api.w4a8_gemm_token_sum(qx, sx, tx, layer.packed, layer.N, out=layer.out, workspace=layer.workspace)
    return out, qx, sx, tx


def _run_load(s):
    w, order = s["w"], None
    if s["step"] == "rotate":
        w = api.hadamard_rotate(w)
    elif s["step"] == "reorder":
        order = api.channel_order(api.channel_absmax(s["calibration"]))
        w = api.gather_channels(w, order)
    return (api.pack_weights(w, s["mode"]),) if order is None else (api.pack_weights(w, s["mode"]), order)


def _run_decoder_layer(s):
    f = FAMILIES[s["family"]]
    rows = f["mode"] == api.QOQ_PER_CHANNEL                    # the per-channel GEMM folds zero points through row sums
    _, qx, sx, rowsum, _ = api.rmsnorm_quant(s["x1"], s["gamma1"], EPS, want_y=False, want_rowsum=rows)
    qkv = s["qkv"].gemm(qx, sx, rowsum)
    api.kv4_append(s["cache"], s["k"], s["v"], s["positions"], s["S_max"])
    attention = s["attention"]
    if s["kind"] == "decode":
        api.kv4_attention_decode(s["q"], s["cache"], s["seq_lens"], f["Hkv"], s["S_max"], out=attention,
                                 workspace=s["attention_workspace"])
    qx, sx, rowsum, _ = api.quant_act_per_token(attention.view(attention.shape[0], -1), want_rowsum=rows)
    o = s["o"].gemm(qx, sx, rowsum)
    _, qx, sx, rowsum, _ = api.rmsnorm_quant(s["x2"], s["gamma2"], EPS, want_y=False, want_rowsum=rows)
    gate_up = s["gate_up"].gemm(qx, sx, rowsum)
    _, qx, sx, rowsum, _ = api.silu_mul_quant(gate_up, want_y=False, want_rowsum=rows)
    down = s["down"].gemm(qx, sx, rowsum)
    out = dict(qkv=qkv, cache=s["cache"], o=o, gate_up=gate_up, down=down)
    if s["kind"] == "decode":
        out["attention"] = attention
    return out


def run(state):
    return {"linear": _run_linear, "load": _run_load}.get(state["kind"], _run_decoder_layer)(state)


# ------------------------------------------------------------------------------------------------------------------
# What a pass cannot do without, and how far another correct implementation may be
# ------------------------------------------------------------------------------------------------------------------
def _packed(N, K, mode):
    """Codes, the two levels' parameters as the method defines them (1.5 bytes a group), channel scales."""
    return N * K / 2 + (1.5 * N * (K // 128) if mode == 0 else N) + 2 * N


def _gemm(M, N, K, mode):
    """Weights and INT8 activations read, FP16 output written."""
    return _packed(N, K, mode) + M * K + 2 * M + 2 * M * N, 2.0 * M * N * K


def work(case):
    kind = case["kind"]
    if kind == "linear":
        M, K, N = case["M"], case["K"], case["N"]
        b, ops = _gemm(M, N, K, case["mode"])
        return dict(bytes=b + 3 * M * K + 2 * M + (4 * K if case["form"] == "reordered" else 0), flops=ops)
    if kind == "load":
        N, K = case["N"], case["K"]
        b, ops = 2 * N * K + _packed(N, K, case["mode"]), 0.0
        if case["step"] == "rotate":
            b, ops = b + 4 * N * K, N * K * math.log2(min(K & -K, 8192))
        elif case["step"] == "reorder":
            b += 4 * N * K + 2 * 1024 * K + 12 * K
        return dict(bytes=b, flops=ops)
    f = FAMILIES[case["family"]]
    B, H, Hkv = case["batch"], f["H"], f["Hkv"]
    M = B if kind == "decode" else B * case["tokens"]
    b = ops = 0.0
    for K, N in f["layers"].values():
        bb, oo = _gemm(M, N, K, f["mode"])
        b, ops = b + bb, ops + oo
    hidden, inner = f["layers"]["qkv"][0], f["layers"]["down"][0]
    b += M * (3 * 3 * hidden + 5 * inner)                      # producers and quantizer: FP16 in, INT8 out
    b += M * Hkv * 2 * (2 * D + D / 2 + 4)                     # keys and values in, their codes and parameters out
    if kind == "decode":
        tokens = 0.75 * B * case["context"]                    # lengths are between half the context and all of it
        b += tokens * Hkv * 2 * (D / 2 + 4) + 4 * B * H * D
        ops += 4.0 * tokens * H * D
    return dict(bytes=b, flops=ops)


def tolerance(case):
    kind = case["kind"]
    if kind == "load":
        return "exact"                                         # integer codes, scales that are one rounding of one quotient
    if kind == "linear":
        # the FP32 epilogue against the same accumulators scaled in FP64: up to 8.5e-6, and one FP16 step where they differ
        return {"rel": 4e-5, "max": 4e-3, "differ": 0.0}
    if kind == "prefill":
        # the same, and an FP16 step in front of a quantizer may move a code of the next layer's input by one
        return {"rel": 5e-4, "max": 1e-2, "differ": 0.0}
    # attention against FP64 on the same cache: 2.0e-4 to 2.5e-4; through the INT8 quantizer, where up to 0.8% of the codes
    # then move by one, the output projection differs by 1.9e-3 to 5.4e-3 (largest single difference 0.08)
    return {"rel": 2e-2, "max": 0.3, "differ": 0.0}
