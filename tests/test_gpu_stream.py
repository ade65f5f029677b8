"""The weight-streaming expert GEMM (a few rows per expert) against the fp64 oracle: row counts at the edges of its 16-
and 32-row tiles, idle experts, the cuts of K it is instantiated for, and every storage of the weights."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as orc
from oracle import quant_e4m3 as o8
from oracle import quant_mxfp4 as o4
from paper_2303_06182_amd import binding, workloads as wl
from helpers import TOL, norm_max_err, to_np, worst_row_rms_rel_err

pytestmark = pytest.mark.gpu

EDGES = [1, 15, 0, 16, 17, 31, 0, 32, 33, 48]
SPARSE = [1, 0, 3, 17, 0, 2, 16, 1] * 4 + [33, 0, 1, 1]
CASES = [
    # counts, D, F, bias
    (EDGES, 512, 1024, True),       # few tiles: eight and four waves share K
    ([1], 2048, 1024, False),       # the smallest call
    ([2, 0, 1], 1024, 4096, True),
    (EDGES, 256, 192, False),       # K the kernel does not serve (some formats): the tiled one takes over
    (SPARSE, 512, 2048, True),      # mxfp4: one wave with 64 columns, four with 32
    (SPARSE, 1024, 512, False),     # ... four waves, one
    ([2] * 64, 2048, 512, True),    # more tiles than resident blocks
    ([0, 1, 31, 32, 33, 64, 65, 200] + [3, 0, 1, 5] * 30, 256, 512, True),   # tiled: weights' cache policy by the expert's rows
]

# bf16 with K that ends inside a K tile, for every tile height; the neighbouring rows hold NaN (idle experts)
RAGGED = [
    ([1, 0, 17, 33], 8, 72, True),                  # K below one step
    ([3, 0, 20] * 100, 72, 1032, False),            # 32-row tiles, more of them than the streaming form takes
    ([64, 0, 130, 50], 200, 328, True),             # 128-row tiles, few rows per expert
    ([100, 257, 0, 60, 128], 1000, 136, False),     # 128-row tiles
    ([300, 0, 513, 1], 264, 456, True),             # 128-row tiles, too few for tiles cut to the rows
    ([1, 0, 17, 33], 264, 328, True),               # streaming form, eight waves: fewer steps of K than waves
    ([1, 0, 17, 33, 8, 0, 2, 31] * 2, 264, 1032, True),     # ... four waves and 32 columns in the first GEMM
]


@pytest.mark.parametrize("case", range(len(RAGGED)))
def test_expert_ffn_ragged_k(case):
    run_ffn("bf16", *RAGGED[case])


@pytest.mark.parametrize("weights", ["bf16", "e4m3", "mxfp4"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_expert_ffn_stream(case, weights):
    run_ffn(weights, *CASES[case])


# mxfp4 with 64 columns: four, two and one waves (K a multiple of 2048, 1024, 512), tiles below and above 16 rows
@pytest.mark.parametrize("D", [2048, 1024, 512])
def test_expert_ffn_stream_mxfp4_wide(D):
    run_ffn("mxfp4", [17, 0, 31, 1, 16, 32, 0, 5], D, 4096, True)


@pytest.mark.parametrize("T,k,E", [(512, 2, 7), (1025, 1, 7), (513, 2, 300)])   # around one round of the single-block routing kernel
def test_route_small_limit(T, k, E):
    g = torch.Generator().manual_seed(T)
    idx = torch.stack([torch.randperm(E, generator=g)[:k] for _ in range(T)]).to(torch.int32)
    out = binding.MoeLayer(T, 64, 64, E, k, "bf16").moe_route_counts(idx.cuda())
    for got, ref in zip(out, orc.route(idx.numpy(), E)):
        assert np.array_equal(to_np(got), ref)


def run_ffn(weights, counts, D, F, bias):
    print("stream ffn", weights, counts, D, F, bias, flush=True)
    E, N = len(counts), int(sum(counts))
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    bf = torch.bfloat16
    xp = wl.normal(61, 0, (N, D), 1.0, bf)
    w1 = wl.normal(61, 1, (E, F, D), 1.0 / np.sqrt(D), bf)
    w2 = wl.normal(61, 2, (E, D, F), 1.0 / np.sqrt(F), bf)
    b1 = wl.normal(61, 3, (E, F), 0.5, bf) if bias else None
    b2 = wl.normal(61, 4, (E, D), 0.5, bf) if bias else None
    m = binding.MoeLayer(N, D, F, E, 1, "bf16")
    xg, og = xp.cuda(), torch.from_numpy(offsets).cuda()
    bg1, bg2 = (None if b is None else b.cuda() for b in (b1, b2))
    idle = [e for e, c in enumerate(counts) if c == 0]
    if weights == "bf16":
        g1, g2 = w1.cuda(), w2.cuda()
        g1[idle], g2[idle] = float("nan"), float("nan")
        yp = m.moe_expert_ffn(xg, og, g1, g2, bg1, bg2)
    else:
        quantise = m.moe_quantize_e4m3 if weights == "e4m3" else m.moe_quantize_mxfp4
        (q1, s1), (q2, s2) = quantise(w1.cuda()), quantise(w2.cuda())
        q1[idle], q2[idle] = 0x77, 0x77
        ffn = m.moe_expert_ffn_w8 if weights == "e4m3" else m.moe_expert_ffn_w4
        yp = ffn(xg, og, q1, q2, s1, s2, bg1, bg2)
        oq = o8 if weights == "e4m3" else o4
        w1, w2 = (torch.from_numpy(oq.dequantize(*oq.quantize(w.float().numpy().astype(np.float64))).astype(np.float32)).to(bf)
                  for w in (w1, w2))
    torch.cuda.synchronize()
    ref = orc.expert_ffn(xp, offsets, w1, w2, b1, b2)
    got = to_np(yp)
    assert np.all(np.isfinite(got))
    # the bf16 bar of the tiled kernels; in norm, H and Yp are each rounded once (2^-9 relative at most, 2^-9.8 on average)
    assert norm_max_err(got, ref) <= TOL["bf16"]
    assert worst_row_rms_rel_err(got, ref) <= 2.0 ** -7


F32_CASES = [
    # counts, D, F, bias: the fp32 kernels' tiles (32 rows, K cut between waves; 64 rows) and K that ends inside a step
    ([1], 8, 16, True),
    ([31, 0, 33, 1, 64, 65], 40, 72, True),
    ([31, 0, 33, 1, 64, 65], 520, 1560, False),
    ([130, 5, 0, 97], 256, 1024, True),
    ([1500, 0, 1, 1700], 64, 2048, True),   # 64-row tiles in the first GEMM, 32-row ones in the second
]


@pytest.mark.parametrize("case", range(len(F32_CASES)))
def test_expert_ffn_f32(case):
    counts, D, F, bias = F32_CASES[case]
    print("f32 ffn", counts, D, F, bias, flush=True)
    E, N = len(counts), int(sum(counts))
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    f32 = torch.float32
    xp = wl.normal(62, 0, (N, D), 1.0, f32)
    w1 = wl.normal(62, 1, (E, F, D), 1.0 / np.sqrt(D), f32)
    w2 = wl.normal(62, 2, (E, D, F), 1.0 / np.sqrt(F), f32)
    b1 = wl.normal(62, 3, (E, F), 0.5, f32) if bias else None
    b2 = wl.normal(62, 4, (E, D), 0.5, f32) if bias else None
    g1, g2 = w1.cuda(), w2.cuda()
    idle = [e for e, c in enumerate(counts) if c == 0]
    g1[idle], g2[idle] = float("nan"), float("nan")
    m = binding.MoeLayer(N, D, F, E, 1, "f32")
    yp = m.moe_expert_ffn(xp.cuda(), torch.from_numpy(offsets).cuda(), g1, g2, *(None if b is None else b.cuda() for b in (b1, b2)))
    torch.cuda.synchronize()
    ref = orc.expert_ffn(xp, offsets, w1, w2, b1, b2)
    got = to_np(yp)
    assert np.all(np.isfinite(got))
    assert norm_max_err(got, ref) <= TOL["f32"]


@pytest.mark.parametrize("T", [1, 16, 64, 65])
@pytest.mark.parametrize("E,k,dtype", [(8, 2, "bf16"), (12, 3, "f32"), (64, 8, "bf16"), (130, 1, "bf16"), (512, 2, "f32"), (1024, 4, "bf16")])
def test_decoder_step_topk_and_routing_in_one_launch(T, E, k, dtype):
    w = wl.Workload("route", dtype, T=T, D=64, F=64, E=E, k=k, seed=5)
    m = binding.MoeLayer(T, 64, 64, E, k, dtype)
    inp = {n: (None if v is None else v.cuda()) for n, v in wl.make_inputs(w).items()}
    r = m.empty_routing(T)
    m.moe_layer_forward(inp["x"], inp["wg"], inp["w1"], inp["w2"], inp["gate_bias"], routing_out=r)
    torch.cuda.synchronize()
    idx, gw = orc.topk(to_np(r["logits"]), k)
    assert np.array_equal(to_np(r["topk_idx"]), idx)
    assert np.abs(to_np(r["topk_w"]) - gw).max() <= 2e-6
    for got, ref in zip((r["counts"], r["offsets"], r["dst_row"], r["src_tok"]), orc.route(idx, E)):
        assert np.array_equal(to_np(got), ref)
