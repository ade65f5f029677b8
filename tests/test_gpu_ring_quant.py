"""Tiles cut to an expert's rows over e4m3 and mxfp4 weights (gemm_ring.hip): row counts around the 32-row units and the 256-row
tile, K of five to seventeen K tiles (mxfp4's block scales come in groups of eight K tiles, whole or cut short), column tiles that
end inside the matrix, idle experts, few active ones.  Every case asks the library whether this is its choice."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import moe_oracle as orc
from oracle import quant_e4m3, quant_mxfp4
from paper_2303_06182_amd import binding
from helpers import TOL, norm_max_err, to_np, worst_row_rms_rel_err

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 31, 32, 33, 0, 64, 97, 255, 256, 257, 288, 289, 513, 16, 17]
CUT = {8: 28, 4: 49}


def choice(wbits, n_rows, E, F, D):
    lib = binding.load_library()
    if wbits == 8:
        rule, args = lib["_ZN6moe35520gemm_bf16_variant_w8Eliii"], (n_rows, E, F, D)
    else:
        rule, args = lib["_ZN6moe35520gemm_bf16_variant_w4Eliiii"], (n_rows, E, F, D, 256)
    rule.argtypes, rule.restype = [ctypes.c_int64] + [ctypes.c_int] * (len(args) - 1), ctypes.c_int
    return rule(*args)


def dequantised(wbits, q, s, rows, cols):
    if wbits == 8:
        d = quant_e4m3.dequantize(quant_e4m3.unblocked(to_np(q), rows, cols), to_np(s))
    else:
        d = quant_mxfp4.dequantize(quant_mxfp4.unblocked_data(to_np(q), rows, cols), quant_mxfp4.unblocked_scales(to_np(s), rows, cols))
    return torch.from_numpy(d.astype(np.float32)).to(torch.bfloat16)


def setup(wbits, E, D, F, N, k=1):
    g = torch.Generator(device="cuda").manual_seed(11)
    t = lambda s, std: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g)
    m = binding.MoeLayer(N, D, F, E, k, "bf16")
    w1, w2 = t((E, F, D), D ** -0.5), t((E, D, F), F ** -0.5)
    w1[1] *= 37.0   # experts with different scales
    quantise = m.moe_quantize_e4m3 if wbits == 8 else m.moe_quantize_mxfp4
    (q1, s1), (q2, s2) = quantise(w1), quantise(w2)
    return t, m, (q1, q2, s1, s2)


@pytest.mark.parametrize("wbits", [8, 4])
@pytest.mark.parametrize("kind,E,D,F,bias", [
    ("even", 140, 320, 1088, True),     # 5 and 17 K tiles: a group of scales of one K tile, column tiles of 64
    ("even", 100, 576, 1024, False),    # 9 and 16 K tiles
    ("even", 100, 1024, 512, False),     # 16 and 8: whole groups
    ("hot", 60, 832, 1088, True),       # one expert over several XCDs
    ("few", 16, 1088, 1600, False),     # 17 and 25 K tiles; the XCDs share the list
    ("even", 240, 256, 1152, False)])   # 4 and 18: the shortest K
def test_expert_ffn(wbits, kind, E, D, F, bias):
    print("ring, quantised", wbits, kind, E, D, F, flush=True)
    rng = np.random.default_rng(6)
    if kind == "even":
        counts = EDGES + [int(v) for v in rng.integers(230, 480, E - len(EDGES))]
    elif kind == "hot":
        counts = EDGES + [int(v) for v in rng.integers(60, 130, E - len(EDGES))]
        counts[len(EDGES)] = 14000
    else:
        counts = [0] * E
        counts[3], counts[4], counts[11] = 7000, 33, 2600
    N = sum(counts)
    assert choice(wbits, N, E, F, D) == choice(wbits, N, E, D, F) == CUT[wbits]
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    t, m, (q1, q2, s1, s2) = setup(wbits, E, D, F, N)
    for e, c in enumerate(counts):
        if c == 0:       # the weights of an idle expert must not reach a result: NaN codes, the largest scales
            q1[e], q2[e] = (0x7F, 0x7F) if wbits == 8 else (0x77, 0x77)
            if wbits == 4:
                s1[e], s2[e] = 254, 254
    xp = t((N, D), 1.0)
    b1, b2 = (t((E, F), 0.5), t((E, D), 0.5)) if bias else (None, None)
    ffn = m.moe_expert_ffn_w8 if wbits == 8 else m.moe_expert_ffn_w4
    yp = ffn(xp, torch.from_numpy(offsets).cuda(), q1, q2, s1, s2, b1, b2)
    assert bool(torch.isfinite(yp).all())
    # against the fp64 oracle on dequantised weights (exact in bf16): the first experts' first and last rows, and some in between
    n = min(E, 18)
    rows = [np.unique(np.concatenate([np.arange(min(c, 300)), np.arange(max(0, c - 40), c), np.arange(0, c, 97)])) for c in counts[:n]]
    live = [e for e in range(n) if counts[e]]
    d1, d2 = torch.zeros((n, F, D), dtype=torch.bfloat16), torch.zeros((n, D, F), dtype=torch.bfloat16)
    d1[live], d2[live] = dequantised(wbits, q1[live], s1[live], F, D), dequantised(wbits, q2[live], s2[live], D, F)
    sel = torch.from_numpy(np.concatenate([o + r for o, r in zip(offsets, rows)])).cuda().long()
    ref = orc.expert_ffn(xp[sel].cpu(), np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32), d1, d2,
                         None if b1 is None else b1[:n].cpu(), None if b2 is None else b2[:n].cpu())
    got = to_np(yp[sel])
    assert norm_max_err(got, ref) <= TOL["bf16"]   # h and y are each rounded to bf16 once, as in the bf16 tiles' tests
    for e in live:                                 # expert 1's scale is 37 times the others'
        part = slice(sum(len(r) for r in rows[:e]), sum(len(r) for r in rows[:e + 1]))
        assert worst_row_rms_rel_err(got[part], ref[part]) <= 2.0 ** -7


@pytest.mark.parametrize("wbits", [8, 4])
def test_layer_equals_its_steps(wbits):
    """The first GEMM gathers its rows from the tokens and the ranking kernel writes the schedule: the same bits as the steps'."""
    T, D, F, E, k = 10000, 768, 1088, 70, 2
    assert choice(wbits, T * k, E, F, D) == CUT[wbits]
    t, m, (q1, q2, s1, s2) = setup(wbits, E, D, F, T, k)
    x, wg = t((T, D), 1.0), t((E, D), 10 * D ** -0.5)
    bias = torch.zeros(E, device="cuda")
    bias[5] = 25.0
    layer, ffn = (m.moe_layer_forward_w8, m.moe_expert_ffn_w8) if wbits == 8 else (m.moe_layer_forward_w4, m.moe_expert_ffn_w4)
    r = m.empty_routing(T)
    y = layer(x, wg, q1, q2, s1, s2, bias, routing_out=r)
    yp = ffn(m.moe_dispatch(x, r["dst_row"]), r["offsets"], q1, q2, s1, s2)
    assert int(r["counts"].max()) > 1000
    assert torch.equal(y, m.moe_combine(yp, r["dst_row"], r["topk_w"]))
