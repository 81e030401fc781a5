"""The calls whose time counts: what an RL step built on this library has it do, through its public entry points.

A rollout engine runs quantized MoE layers at decode sizes (one to a few hundred tokens); the learner runs the same
layers at prefill / training-forward sizes, their straight-through backward, the LM head's per-token log-probs, and the
re-quantization of the masters after an update.  The layer shape is the one the library is written around (128 experts,
hidden 2048, intermediate 768, top-8); drawn cases also take smaller layers, other batch sizes, formats and routers.

listed() names the cases, draw() gives more of the same ranges, prepare() makes what a program holds before the call,
run() is one pass, work() the bytes and operations a pass cannot do without, tolerance() how far two correct
implementations of the same precision may differ.
"""
import math

import torch

from paper_2604_07853_amd import binding as q
from paper_2604_07853_amd import synth

FORMATS = {"w4a16": q.QARL_W4A16_G128, "fp8": q.QARL_FP8_E4M3_CH, "fp4": q.QARL_FP4_E2M1_CH, "w4a8": q.QARL_W4A8_G128}
LAYER = dict(experts=synth.E, hidden=synth.H, inter=synth.I, topk=synth.TOPK)
DECODE_LAYERS = 4      # layers of one decode pass: their weights (1.2 GB in int4) do not stay in the last-level cache
DECODE_MAX_TOKENS = 512
VOCAB = synth.V


def listed():
    return [
        # one sequence being generated: eight experts per layer, latency and launches
        dict(LAYER, name="decode_w4a16_1tok", kind="decode", fmt="w4a16", tokens=1, zipf=0.0, layers=DECODE_LAYERS),
        # a rollout batch of ordinary size: all experts active, the weight stream
        dict(LAYER, name="decode_w4a16_256tok", kind="decode", fmt="w4a16", tokens=256, zipf=0.0, layers=DECODE_LAYERS),
        # the largest rollout batch: about 32 rows per expert
        dict(LAYER, name="decode_w4a16_512tok", kind="decode", fmt="w4a16", tokens=512, zipf=0.0, layers=DECODE_LAYERS),
        # the W8A8 rollout scheme at the ordinary batch
        dict(LAYER, name="decode_fp8_256tok", kind="decode", fmt="fp8", tokens=256, zipf=0.0, layers=DECODE_LAYERS),
        # a rollout batch that has drained to an odd few tens of sequences, FP4 weights
        dict(LAYER, name="decode_fp4_37tok", kind="decode", fmt="fp4", tokens=37, zipf=0.0, layers=DECODE_LAYERS),
        # the learner's low-bit forward of one layer over 8 sequences x 2048 tokens, popular experts
        dict(LAYER, name="prefill_w4a16_16384tok_zipf", kind="prefill", fmt="w4a16", tokens=16384, zipf=1.1),
        # the same at W8A8
        dict(LAYER, name="prefill_fp8_8192tok", kind="prefill", fmt="fp8", tokens=8192, zipf=0.0),
        # prefill of a ragged batch of prompts under the W4A8 scheme
        dict(LAYER, name="prefill_w4a8_3001tok", kind="prefill", fmt="w4a8", tokens=3001, zipf=0.0),
        # the learner's backward of the gate_up projection: both gradients
        dict(LAYER, name="backward_gate_up_16384tok_zipf", kind="backward", proj="gate_up", tokens=16384, zipf=1.1),
        # after an optimizer step: one layer's masters to int4
        dict(experts=synth.E, hidden=synth.H, inter=synth.I, name="requantize_w4a16_layer", kind="requantize", fmt="w4a16"),
        # log-probs of 8 sampled sequences under the learner, compared with the sampler's
        dict(name="logprob_16384tok", kind="logprob", tokens=16384, seqs=8, hidden=synth.H, vocab=VOCAB),
        # log-probs of the tokens of one decode step
        dict(name="logprob_61tok", kind="logprob", tokens=61, seqs=0, hidden=synth.H, vocab=VOCAB),
    ]


def _log_uniform(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_layer(rng):
    if rng.random() < 0.6:
        return dict(LAYER)
    return dict(experts=rng.choice((64, 128)), hidden=rng.choice((1024, 2048)), inter=rng.choice((512, 768)),
                topk=rng.choice((4, 8)))


def draw(rng):
    kind = rng.choice(("decode", "decode", "decode", "prefill", "prefill", "backward", "requantize", "logprob"))
    zipf = rng.choice((0.0, 1.1))
    if kind == "decode":
        return dict(_draw_layer(rng), kind=kind, fmt=rng.choice(sorted(FORMATS)),
                    tokens=_log_uniform(rng, 1, DECODE_MAX_TOKENS), zipf=zipf, layers=DECODE_LAYERS)
    if kind == "prefill":   # from the first batch the decode entry does not take
        return dict(_draw_layer(rng), kind=kind, fmt=rng.choice(sorted(FORMATS)),
                    tokens=_log_uniform(rng, DECODE_MAX_TOKENS + 1, 16384), zipf=zipf)
    if kind == "backward":
        return dict(_draw_layer(rng), kind=kind, proj=rng.choice(("gate_up", "down")),
                    tokens=_log_uniform(rng, 512, 16384), zipf=zipf)
    if kind == "requantize":
        return dict(experts=_log_uniform(rng, 8, 128), hidden=rng.choice((1024, 2048, 4096)),
                    inter=128 * rng.randint(2, 8), kind=kind, fmt=rng.choice(("fp4", "fp8", "w4a16")))
    tokens = _log_uniform(rng, 1, 16384)
    return dict(kind=kind, tokens=tokens, seqs=rng.choice((0, 1, 8)) if tokens >= 64 else 0,
                hidden=rng.choice((1024, 2048)), vocab=rng.choice((32003, 65536, VOCAB)))


def _experts(case, layer_seed, fmt):
    gu, dn = synth.expert_weights(case["experts"], case["hidden"], case["inter"], layer_seed, device="cuda")
    return q.qarl_quantize_weights(gu, fmt), q.qarl_quantize_weights(dn, fmt)


def prepare(case, seed):
    kind = case["kind"]
    s = seed * 1000
    if kind == "decode":
        # a stack of layers, each with its own weights, token rows and router logits
        layers = []
        for l in range(case["layers"]):
            gu, dn = _experts(case, s + 10 * l, FORMATS[case["fmt"]])
            layer = q.MoELayer(gu, dn, case["tokens"], case["topk"], q.QARL_PATH_DECODE)
            x = synth.normal_bf16((case["tokens"], case["hidden"]), 1.0, s + 10 * l + 2, device="cuda")
            lg = synth.router_logits(case["tokens"], case["experts"], s + 10 * l + 3, device="cuda", zipf_s=case["zipf"])
            layers.append((layer, x, lg))
        return dict(kind=kind, layers=layers)
    if kind == "prefill":
        gu, dn = _experts(case, s, FORMATS[case["fmt"]])
        layer = q.MoELayer(gu, dn, case["tokens"], case["topk"])
        x = synth.normal_bf16((case["tokens"], case["hidden"]), 1.0, s + 2, device="cuda")
        lg = synth.router_logits(case["tokens"], case["experts"], s + 3, device="cuda", zipf_s=case["zipf"])
        return dict(kind=kind, layer=layer, x=x, logits=lg)
    if kind == "backward":
        # after the forward: routing, weights, the projection's input rows and the gradient of its output rows
        E, M = case["experts"], case["tokens"] * case["topk"]
        gate_up = case["proj"] == "gate_up"
        N, K = (2 * case["inter"], case["hidden"]) if gate_up else (case["hidden"], case["inter"])
        W = q.qarl_quantize_weights(synth.normal_bf16((E, N, K), 0.02, s, device="cuda"))
        lg = synth.router_logits(case["tokens"], E, s + 1, device="cuda", zipf_s=case["zipf"])
        r = q.qarl_moe_route(lg, case["topk"])
        x = synth.normal_bf16((case["tokens"] if gate_up else M, K), 1.0, s + 2, device="cuda")
        dy = synth.normal_bf16((M, N), 0.01, s + 3, device="cuda")
        return dict(kind=kind, W=W, x=x, dy=dy, M=M, offsets=r.offsets, row_map=r.tokens if gate_up else None,
                    dx=torch.empty((M, K), dtype=torch.bfloat16, device="cuda"),
                    dw=torch.empty((E, N, K), dtype=torch.bfloat16, device="cuda"))
    if kind == "requantize":
        masters = synth.expert_weights(case["experts"], case["hidden"], case["inter"], s, device="cuda")
        fmt = FORMATS[case["fmt"]]
        return dict(kind=kind, fmt=fmt, masters=masters,
                    out=[q.QWeight.empty(fmt, w.shape[0], w.shape[1], w.shape[2]) for w in masters])
    if kind == "logprob":
        T, H, V = case["tokens"], case["hidden"], case["vocab"]
        h = synth.normal_bf16((T, H), 1.0, s, device="cuda")
        w_lm = synth.normal_bf16((V, H), 0.02, s + 1, device="cuda")
        target = synth.targets(T, V, s + 2, device="cuda")
        st = dict(kind=kind, h=h, w_lm=w_lm, target=target, ref=None, seq_offsets=None,
                  ws=torch.empty((max(q.qarl_logprob_workspace_bytes(T, H, V), 16),), dtype=torch.uint8, device="cuda"))
        if case["seqs"]:   # the sampler's log-probs of the same tokens: logits of spread 1 around a mean of -ln V
            g = torch.Generator(device="cuda")
            g.manual_seed(s + 3)
            st["ref"] = torch.randn((T,), generator=g, device="cuda") - (math.log(V) + 0.5)
            n = case["seqs"]
            st["seq_offsets"] = torch.tensor([T * i // n for i in range(n + 1)], dtype=torch.int32, device="cuda")
        return st
    raise ValueError(kind)


def run(state):
    kind = state["kind"]
    if kind == "decode":
        return [layer.forward(x, lg) for layer, x, lg in state["layers"]]
    if kind == "prefill":
        return state["layer"].forward(state["x"], state["logits"])
    if kind == "backward":
        dx = q.qarl_qgemm_grouped_dx(state["W"], state["dy"], state["offsets"], state["M"], out=state["dx"])
        dw = q.qarl_grouped_dw(state["dy"], state["x"], state["offsets"], state["W"].E, row_map=state["row_map"],
                               out=state["dw"])
        return dict(dx=dx, dw=dw)
    if kind == "requantize":
        outs = [q.qarl_quantize_weights(w, state["fmt"], out=o) for w, o in zip(state["masters"], state["out"])]
        return [t for o in outs for t in (o.codes, o.scales)]
    r = q.qarl_token_logprob(state["h"], state["w_lm"], state["target"], ref_logprob=state["ref"],
                             seq_offsets=state["seq_offsets"], ws=state["ws"], want_delta=state["ref"] is not None)
    return {k: v for k, v in r.items() if v is not None}


def _weight_bytes(fmt, E, N, K):
    return q.lib().qarl_codes_bytes(FORMATS[fmt], E, N, K) + q.lib().qarl_scales_bytes(FORMATS[fmt], E, N, K)


def _active_experts(case):
    """Experts that at least one of the tokens picks, on average (each token picks topk of them; uniform router)."""
    E = case["experts"]
    return E * (1.0 - (1.0 - case["topk"] / E) ** case["tokens"])


def work(case):
    kind = case["kind"]
    if kind in ("decode", "prefill"):
        E, H, I, T, n = case["experts"], case["hidden"], case["inter"], case["tokens"], case.get("layers", 1)
        w = (_weight_bytes(case["fmt"], E, 2 * I, H) + _weight_bytes(case["fmt"], E, H, I)) * _active_experts(case) / E
        return dict(bytes=n * (w + T * E * 2 + 2 * T * H * 2), flops=n * synth.flops_moe(T, H, I, case["topk"]))
    if kind == "backward":
        E, M = case["experts"], case["tokens"] * case["topk"]
        gate_up = case["proj"] == "gate_up"
        N, K = (2 * case["inter"], case["hidden"]) if gate_up else (case["hidden"], case["inter"])
        rows = case["tokens"] if gate_up else M
        return dict(bytes=_weight_bytes("w4a16", E, N, K) + 2 * (M * N + rows * K + M * K + E * N * K),
                    flops=2 * 2 * M * N * K)
    if kind == "requantize":
        E, H, I = case["experts"], case["hidden"], case["inter"]
        n = 3 * E * H * I
        return dict(bytes=2 * n + _weight_bytes(case["fmt"], E, 2 * I, H) + _weight_bytes(case["fmt"], E, H, I),
                    flops=2 * n)
    T, H, V = case["tokens"], case["hidden"], case["vocab"]
    return dict(bytes=2 * (T * H + V * H) + T * 8 + (T * 8 if case["seqs"] else 0), flops=2 * T * H * V)


# Relative error (2-norm) of one layer's bf16 output against the same layer with every sum in 64 bits and the same
# roundings in between (bf16 intermediate, e4m3 rows where the format has them), measured at 512 tokens: w4a16 1.8e-4,
# w4a8 3.8e-4, fp4 1.05e-3, fp8 1.95e-3 (a sum that lands on the other side of a rounding moves an e4m3 code, and a row's
# largest value moves its scale).  Four times that is stated.
LAYER_REL = {"w4a16": 7e-4, "w4a8": 1.5e-3, "fp4": 4e-3, "fp8": 8e-3}


def tolerance(case):
    kind = case["kind"]
    if kind == "requantize":
        return "exact"
    if kind == "backward":   # against 64-bit sums: dx 2.3e-3 (the scaled gradient is rounded to bf16, so is dx), dw 1.7e-3
        return dict(rel=9e-3)
    if kind == "logprob":    # against 64-bit sums: 6e-8 of values near -13, that is 8e-7; differences to the sampler are of size 1
        return dict(rel=3e-6)
    return dict(rel=LAYER_REL[case["fmt"]])
