"""Expert GEMMs whose K loop goes round K from a place of the tile's own (turned_k: weight rows of a multiple of 4 KB), in every
tile shape that does so, at row counts around the tiles' edges and with columns that end inside a tile; with biases and idle
experts."""
import numpy as np
import pytest
import torch

from helpers import TOL, expert_kernels, norm_max_err, to_np, worst_row_rms_rel_err
from oracle import moe_oracle as orc
from oracle import quant_e4m3
from paper_2303_06182_amd import binding
from test_gpu_tile_shapes import ragged, run

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 31, 32, 33, 0, 63, 64, 65, 127, 128, 129]


@pytest.mark.parametrize("shape,E,D,F,lo,hi", [
    ("cut to rows", 40, 2048, 1096, 120, 260),    # the first GEMM turns: 32 K tiles
    ("cut to rows", 40, 1096, 4096, 120, 260),    # the second one: 64
    ("128x128", 14, 2048, 776, 350, 360), ("128x128", 14, 776, 2048, 350, 360),   # 96 rows in the mean: fewer are 64x128's
    ("64x128", 14, 2048, 776, 60, 70),
    ("64x128", 80, 2048, 320, 25, 50), ("64x128", 80, 320, 4096, 25, 50),
    ("32x128", 120, 2048, 320, 5, 15), ("32x128", 120, 320, 2048, 5, 15)])
def test_tiles(shape, E, D, F, lo, hi):
    run(shape, ragged(E, EDGES, lo, hi, 4), D, F)


@pytest.mark.parametrize("D,F", [(4096, 544), (544, 8192)])   # the streaming kernel: 4096 and 8192 in parts of a wave each
def test_streams(D, F):
    counts = [0, 1, 3, 0, 16, 17, 2, 33]
    assert "stream16" in expert_kernels(16, sum(counts), len(counts), F, D)
    run("32x128", counts, D, F)


@pytest.mark.parametrize("counts,D,F,kernel", [
    ([0, 1, 31, 33, 64, 0, 17, 40], 1024, 2112, "32x128x3"),                     # the first GEMM turns: 16 K tiles
    ([20, 0, 33, 1, 32, 15, 40, 31, 30, 29] * 3, 2048, 1024, "32x128x3"),        # the second one: N = 2048 and K = 1024
    ([0, 1, 0, 3, 16, 2], 2048, 2112, "stream32"), ([1, 0, 17, 2], 4096, 576, "stream16")])
def test_e4m3(counts, D, F, kernel):
    print("e4m3", len(counts), D, F, flush=True)
    E, N = len(counts), sum(counts)
    assert kernel in expert_kernels(8, N, E, F, D)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    g = torch.Generator(device="cuda").manual_seed(8)
    t = lambda s, std: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g)
    m = binding.MoeLayer(N, D, F, E, 1, "bf16")
    xp = t((N, D), 1.0)
    (q1, s1), (q2, s2) = m.moe_quantize_e4m3(t((E, F, D), D ** -0.5)), m.moe_quantize_e4m3(t((E, D, F), F ** -0.5))
    yp = to_np(m.moe_expert_ffn_w8(xp, torch.from_numpy(offsets).cuda(), q1, q2, s1, s2))
    deq = lambda q, s, r, c: torch.from_numpy(quant_e4m3.dequantize(quant_e4m3.unblocked(to_np(q), r, c), to_np(s)).astype(np.float32)).to(torch.bfloat16)
    ref = orc.expert_ffn(xp.cpu(), offsets, deq(q1, s1, F, D), deq(q2, s2, D, F))
    assert norm_max_err(yp, ref) <= TOL["bf16"]
    assert worst_row_rms_rel_err(yp, ref) <= 2.0 ** -7
