"""Expert GEMMs with a tile or two per CU (few_tiles, gemm_bf16.hip): narrower tiles and more LDS stages.  Row counts around the tiles'
edges, K of one K tile and of fewer than the stages, K loops that go round K, idle experts, biases; and the choice around its lines.
Every case asks the library which kernels its two GEMMs run on."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as orc
from paper_2303_06182_amd import binding
from helpers import TOL, expert_kernels, expert_tile_shape, norm_max_err, to_np, worst_row_rms_rel_err
from test_gpu_ring_quant import dequantised, setup
from test_gpu_tile_shapes import ragged, run

EDGES = [0, 1, 31, 32, 33, 63, 64, 65]
MORE = [0, 1, 31, 200, 33, 129, 64, 127]


@pytest.mark.gpu
@pytest.mark.parametrize("shape,E,D,F,edges,lo,hi,kernels", [
    ("64x128", 16, 1024, 1088, EDGES, 10, 60, "64x128x3 64x64x4"), ("64x128", 16, 576, 1088, EDGES, 10, 60, "64x128x3 64x64x4"),
    ("64x128", 8, 2048, 2112, EDGES, 0, 0, "64x128x3 64x64x4"), ("64x128", 8, 2048, 2112, [0, 1, 5, 33, 20, 4, 2, 63], 0, 0, "64x64x4 64x64x4"),
    ("64x128", 16, 64, 256, EDGES + [127, 128, 129, 200], 90, 140, "64x64x4 64x64x4"),
    ("64x128", 16, 256, 64, EDGES + [127, 128, 129, 200], 90, 140, "64x64x4 64x64x4"),
    ("64x128", 4, 192, 128, [65, 129, 0, 127], 0, 0, "64x64x4 64x64x4"),
    ("128x128", 8, 1024, 1024, [0, 1, 127, 128, 129, 257, 255, 256], 0, 0, "128x64x4 128x64x4"),
    ("128x128", 8, 1024, 576, [600, 127, 128, 129, 257, 255, 0, 700], 0, 0, "128x128 128x128"),
    ("128x128", 12, 64, 384, EDGES + [600, 900, 700, 1000], 0, 0, "128x128 128x64x4"),
    ("32x128", 16, 2048, 2112, EDGES[:6], 16, 32, "32x128x4 32x128x4"),
    # K of fewer K tiles than stages
    ("32x128", 40, 192, 768, EDGES[:6], 6, 14, "32x128x2 stream32"),
    # K that ends inside a K tile
    ("64x128", 16, 1000, 1096, EDGES, 10, 60, "64x128x3 64x64x4"), ("64x128", 8, 72, 264, MORE, 0, 0, "64x64x4 64x64x4"),
    ("64x128", 8, 200, 1992, MORE, 0, 0, "64x128x3 64x64x4"), ("64x128", 24, 1000, 4000, EDGES, 40, 50, "64x128x2 64x128x3"),
    ("128x128", 8, 1000, 1000, [0, 1, 127, 128, 129, 257, 255, 256], 0, 0, "128x64x4 128x64x4"),
    ("128x128", 40, 1000, 1096, EDGES, 40, 50, "128x128 128x128"), ("32x128", 24, 1000, 1992, EDGES, 6, 20, "32x128x4 32x128x4")])
def test_ffn(shape, E, D, F, edges, lo, hi, kernels):
    counts = ragged(E, edges, lo, hi, 5) if hi else edges
    assert " ".join(expert_kernels(16, sum(counts), E, F, D)) == kernels
    run(shape, counts, D, F)


@pytest.mark.gpu
def test_nothing_past_k_is_multiplied():
    """Every other row of an expert's batch is infinite: what its row's neighbour has behind the end of K."""
    E, D, F, n = 8, 200, 328, 48
    g = torch.Generator(device="cuda").manual_seed(9)
    t = lambda s, std: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g)
    xp, w1, w2 = t((E * n, D), 1.0), t((E, F, D), D ** -0.5), t((E, D, F), F ** -0.5)
    assert expert_tile_shape(E * n, E, F, D) in ("64x128", "32x128")
    m = binding.MoeLayer(E * n, D, F, E, 1, "bf16")
    offsets = torch.arange(0, E * n + 1, n, dtype=torch.int32, device="cuda")
    want = m.moe_expert_ffn(xp, offsets, w1, w2)
    xp[1::2] = float("inf")
    assert torch.equal(m.moe_expert_ffn(xp, offsets, w1, w2)[::2], want[::2])


@pytest.mark.parametrize("E,D,F,rows,shape", [
    # 33 to 64 weight panels, 17 to 32, 16 and fewer
    (8, 2048, 8192, 7, "32x128"), (8, 2048, 8192, 8, "64x128"), (8, 2048, 8192, 95, "64x128"), (8, 2048, 8192, 96, "128x128"),
    (32, 512, 2048, 20, "64x128"), (8, 1024, 4096, 32, "32x128"), (8, 1024, 4096, 33, "64x128"), (8, 1024, 4096, 128, "64x128"),
    (8, 1024, 4096, 129, "128x128"), (8, 512, 2048, 64, "32x128"), (8, 512, 2048, 65, "64x128"), (8, 512, 2048, 191, "64x128"),
    (8, 512, 2048, 192, "128x128"),
    # K that ends inside a K tile
    (8, 1000, 4000, 32, "32x128"), (8, 1000, 4000, 33, "64x128"), (8, 1000, 4000, 119, "64x128"), (8, 1000, 4000, 120, "128x128"),
    (24, 1000, 4000, 29, "32x128"), (24, 1000, 4000, 30, "64x128"), (24, 1000, 4000, 49, "64x128"), (24, 1000, 4000, 50, "128x128"),
    (17, 680, 5896, 59, "64x128"), (17, 680, 5896, 60, "128x128"), (32, 496, 4984, 95, "64x128"), (47, 1496, 4504, 29, "32x128"),
    (47, 1496, 4504, 30, "128x128"), (130, 200, 600, 49, "64x128"),
    # few weights, a dimension of 64
    (100, 128, 512, 16, "32x128"), (100, 128, 512, 17, "64x128"), (250, 64, 512, 47, "32x128"), (250, 64, 512, 48, "64x128")])
def test_choice(E, D, F, rows, shape):
    assert expert_tile_shape(E * rows, E, F, D) == shape


@pytest.mark.gpu
@pytest.mark.parametrize("counts,D,F,kernel", [
    ([0, 1, 31, 32, 33, 63, 64, 65] * 2, 2048, 1984, "32x128x4"),   # K of 32 and 31 K tiles
    # K of 16 and 17 K tiles, 3 and 5
    ([0, 1, 127, 128, 129, 257, 63, 300], 1024, 1088, "64x128x4"), ([64, 0, 150, 129, 190], 192, 320, "64x128x4")])
def test_mxfp4(counts, D, F, kernel):
    print("mxfp4", counts, D, F, flush=True)
    E, N = len(counts), sum(counts)
    assert expert_kernels(4, N, E, F, D) == (kernel, kernel)
    t, m, (q1, q2, s1, s2) = setup(4, E, D, F, N)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    for e in (e for e, c in enumerate(counts) if c == 0):   # NaN's place in this format: the largest scale
        q1[e], q2[e], s1[e], s2[e] = 0x77, 0x77, 254, 254
    xp, b1, b2 = t((N, D), 1.0), t((E, F), 0.5), t((E, D), 0.5)
    got = to_np(m.moe_expert_ffn_w4(xp, torch.from_numpy(offsets).cuda(), q1, q2, s1, s2, b1, b2))
    live = [e for e, c in enumerate(counts) if c]
    d1, d2 = torch.zeros((E, F, D), dtype=torch.bfloat16), torch.zeros((E, D, F), dtype=torch.bfloat16)
    d1[live], d2[live] = dequantised(4, q1[live], s1[live], F, D), dequantised(4, q2[live], s2[live], D, F)
    ref = orc.expert_ffn(xp.cpu(), offsets, d1, d2, b1.cpu(), b2.cpu())
    assert norm_max_err(got, ref) <= TOL["bf16"]   # h and y are each rounded to bf16 once
    for e in live:
        part = slice(int(offsets[e]), int(offsets[e + 1]))
        assert worst_row_rms_rel_err(got[part], ref[part]) <= 2.0 ** -7
