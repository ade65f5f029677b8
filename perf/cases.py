"""Workloads of the dynamically gated MoE layer over the range a user of this library meets.

Shapes come from the repository's own workloads (``paper_2303_06182_amd/workloads.py``: an LM layer of
1024 -> 4096, an MT layer of 2048 -> 8192, top-2, load skewed but dense for prefill and mostly idle
experts in a decoder step), from the 512 experts its LM layers have at full size, and from generic
ragged sizes.  ``listed()`` gives the fixed ones, ``draw(rng)`` more of the same ranges.

A case is one MoE layer and one batch of tokens:

    T, D, F, E, k       tokens, model dimension, expert hidden dimension, experts, experts per token
    weights             storage of the expert weights: "bf16", "f32", "e4m3" or "mxfp4" (activations are
                        f32 for "f32" and bf16 otherwise)
    bias                with the experts' b1 / b2
    renorm              gate weights renormalised over the selected experts
    zipf                exponent of the experts' popularity (0 = none), at the workloads' scale ``zipf_c``
    gate_scale          factor on the gate's weights (1: nearly equal gate weights, 50: a decided gate)
    steps               False: the fused layer call.  True: the five steps called one by one, as a program does
                        that exchanges the dispatched rows with other devices between them

Not listed: the static-capacity form of the layer, which exists to be compared with, and expert buffering,
whose time is the host link's.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2303_06182_amd import binding, workloads


def _case(name, T, D, F, E, k=2, weights="bf16", bias=False, renorm=True, zipf=0.0, zipf_c=0.0, gate_scale=1.0, steps=False):
    return dict(name=name, T=T, D=D, F=F, E=E, k=k, weights=weights, bias=bias, renorm=renorm, zipf=zipf, zipf_c=zipf_c,
                gate_scale=gate_scale, steps=steps)


def listed():
    return [
        # one sequence being decoded: two experts' weights and nothing else; launches and latency
        _case("decode_1", 1, 2048, 8192, 128),
        # a decoder step of a served batch (the workload mt_decoder), with each storage of the weights
        _case("decode_64", 64, 2048, 8192, 128),
        _case("decode_64_e4m3", 64, 2048, 8192, 128, weights="e4m3"),
        # ... and of a smaller batch, where a fifth of the experts are active
        _case("decode_16_mxfp4", 16, 2048, 8192, 128, weights="mxfp4"),
        # the fp32 accuracy configuration (tiny_f32)
        _case("tiny_f32", 512, 512, 2048, 8, weights="f32"),
        # prefill of an LM layer (lm): weights and arithmetic weigh about the same
        _case("lm", 8192, 1024, 4096, 64, zipf=0.8, zipf_c=0.25),
        # a full-size LM layer: 512 experts, an odd batch, biases, gate weights over all experts
        _case("lm_512", 4099, 1024, 4096, 512, bias=True, renorm=False, zipf=0.8, zipf_c=0.25, gate_scale=50.0),
        # prefill over 4-bit weights
        _case("lm_mxfp4", 8192, 1024, 4096, 64, weights="mxfp4", zipf=0.8, zipf_c=0.25),
        # one device's share of an MT encoder batch (mt_encoder): bound by the matrix cores
        _case("mt_encoder", 16384, 2048, 8192, 16),
        # the step-by-step entry points on a batch between decoding and a full prefill
        _case("mt_steps", 9001, 2048, 8192, 128, zipf=0.8, zipf_c=0.25, gate_scale=50.0, steps=True),
        # the largest batch, with hot experts (skewed_large)
        _case("skewed_large", 65536, 2048, 8192, 128, zipf=1.2, zipf_c=0.5),
        # dimensions that are no multiples of any tile, top-1, biases
        _case("odd_dims", 3001, 1000, 4000, 24, k=1, bias=True, gate_scale=50.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# (D, F, expert counts) of the layers the cases are about
_LAYERS = [(1024, 4096, (16, 64, 128, 512)), (2048, 8192, (8, 16, 64, 128)), (512, 2048, (8, 32, 64))]


def draw(rng: random.Random):
    """One more case (without a name)."""
    kind = rng.choice(["decode"] * 4 + ["prefill"] * 4 + ["steps", "f32", "odd"])
    D, F, experts = rng.choice(_LAYERS)
    E = rng.choice(experts)
    weights = "bf16"
    if kind == "decode":
        T = _log_int(rng, 1, 256)
        weights = rng.choice(["bf16", "bf16", "e4m3", "mxfp4"])
    elif kind == "prefill":
        weights = rng.choice(["bf16", "bf16", "bf16", "e4m3", "mxfp4"])
        T = _log_int(rng, 257, 65536 if weights == "bf16" else 16384)
    elif kind == "steps":
        T = _log_int(rng, 65, 16384)
    elif kind == "f32":
        D, F, E = rng.choice([(512, 2048, 8), (256, 1024, 32), (1024, 4096, 8), (520, 1560, 5)])
        weights, T = "f32", _log_int(rng, 1, 4096)
    else:
        D = 8 * rng.randint(33, 255)
        F = 8 * rng.randint(65, 1023)
        E, T = rng.randint(2, 60), _log_int(rng, 1, 8192)
    c = _case("", T, D, F, E, min(E, rng.choice([1, 2, 2, 2, 4] if T < 16384 else [1, 2, 2])), weights, bias=rng.random() < 0.3,
              renorm=rng.random() < 0.7, gate_scale=rng.choice([1.0, 50.0]), steps=kind == "steps")
    if rng.random() < 0.5:
        c["zipf"], c["zipf_c"] = rng.choice([(0.8, 0.25), (1.2, 0.5)])
    del c["name"]
    return c


def _normal(shape, std, dtype, gen):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=gen)


def prepare(case, seed):
    """The layer's handle, its weights in their storage format and one batch of tokens."""
    T, D, F, E, k = (case[n] for n in ("T", "D", "F", "E", "k"))
    wfmt = case["weights"]
    dt = torch.float32 if wfmt == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    s = {"case": case, "layer": binding.MoeLayer(T, D, F, E, k, "f32" if wfmt == "f32" else "bf16", case["renorm"])}
    s["x"] = _normal((T, D), 0.02, dt, gen)
    s["wg"] = _normal((E, D), case["gate_scale"] / math.sqrt(D), dt, gen)
    w = workloads.Workload("case", "f32" if wfmt == "f32" else "bf16", T=T, D=D, F=F, E=E, k=k, zipf_s=case["zipf"],
                           zipf_c=case["zipf_c"] * case["gate_scale"], seed=seed)
    gb = workloads.zipf_bias(w)
    s["gate_bias"] = None if gb is None else gb.cuda()
    w1 = _normal((E, F, D), 0.02, dt, gen)
    w2 = _normal((E, D, F), 0.02, dt, gen)
    s["b1"] = _normal((E, F), 0.02, dt, gen) if case["bias"] else None
    s["b2"] = _normal((E, D), 0.02, dt, gen) if case["bias"] else None
    if wfmt in ("e4m3", "mxfp4"):
        quantise = s["layer"].moe_quantize_e4m3 if wfmt == "e4m3" else s["layer"].moe_quantize_mxfp4
        s["w1"], s["s1"] = quantise(w1)
        s["w2"], s["s2"] = quantise(w2)
    else:
        s["w1"], s["w2"] = w1, w2
    return s


def run(s):
    """One pass of the layer over the batch."""
    m, c = s["layer"], s["case"]
    if c["weights"] == "e4m3":
        return m.moe_layer_forward_w8(s["x"], s["wg"], s["w1"], s["w2"], s["s1"], s["s2"], s["gate_bias"], s["b1"], s["b2"])
    if c["weights"] == "mxfp4":
        return m.moe_layer_forward_w4(s["x"], s["wg"], s["w1"], s["w2"], s["s1"], s["s2"], s["gate_bias"], s["b1"], s["b2"])
    if not c["steps"]:
        return m.moe_layer_forward(s["x"], s["wg"], s["w1"], s["w2"], s["gate_bias"], s["b1"], s["b2"])
    logits, idx, gw = m.moe_gate_topk(s["x"], s["wg"], s["gate_bias"])
    counts, offsets, dst_row, src_tok = m.moe_route_counts(idx)
    xp = m.moe_dispatch(s["x"], dst_row)
    yp = m.moe_expert_ffn(xp, offsets, s["w1"], s["w2"], s["b1"], s["b2"])
    y = m.moe_combine(yp, dst_row, gw)
    return {"y": y, "logits": logits, "topk_idx": idx, "topk_w": gw, "counts": counts, "offsets": offsets, "dst_row": dst_row,
            "src_tok": src_tok}


def work(case):
    """Bytes: tokens in and out, the gate, and the weights of the experts that an even gate makes active; the steps also
    write the dispatched rows and the expert outputs and read them again.  Flops: the gate and k experts per token."""
    T, D, F, E, k = (case[n] for n in ("T", "D", "F", "E", "k"))
    es = 4 if case["weights"] == "f32" else 2
    per_weight = {"bf16": 2.0, "f32": 4.0, "e4m3": 1.0, "mxfp4": 0.5 + 1.0 / 32.0}[case["weights"]]
    active = E * (1.0 - (1.0 - k / E) ** T)
    b = 2.0 * T * D * es + float(E) * D * es + active * 2.0 * D * F * per_weight
    if case["steps"]:
        b += 4.0 * T * k * D * es + 4.0 * T * E
    return {"bytes": b, "flops": 4.0 * T * k * D * F + 2.0 * T * D * E}


def tolerance(case):
    """About four times the largest of two comparisons measured on these cases: with the layer in fp64 (bf16: the hidden
    rows, the expert outputs and y are each rounded once, 2.9e-3 in norm and 1.6e-2 at most; f32: 7e-7 and 5e-6), and
    with the layer's inner dimensions permuted, i.e. its sums in another order (3.5e-4 and 1.5e-2; 9e-7 and 6e-6)."""
    if case["weights"] == "f32":
        return {"rel": 4e-6, "max": 2.4e-5}
    return {"rel": 1e-2, "max": 6e-2}
