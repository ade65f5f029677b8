"""The expert GEMM whose tiles are cut to an expert's rows (gemm_ring.hip) and its schedule: row counts around the 32-row
units and the 256-row tile, one expert spread over several XCDs, so few rows that the XCDs share them, idle experts, K that
ends inside a K tile, column tiles that end inside the matrix."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as orc
from paper_2303_06182_amd import binding
from helpers import TOL, expert_tile_shape, norm_max_err, to_np, worst_row_rms_rel_err

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 31, 32, 33, 0, 64, 97, 255, 256, 257, 288, 289, 513, 16, 17]


def counts_of(kind, E):
    rng = np.random.default_rng(5)
    if kind == "even":
        c = EDGES + [int(v) for v in rng.integers(170, 350, E - len(EDGES))]
    elif kind == "hot":        # one expert holds most of the rows, its neighbours a handful
        c = EDGES + [int(v) for v in rng.integers(0, 40, E - len(EDGES))]
        c[len(EDGES)] = 200 * E
    elif kind == "level":      # parts of whole row tiles have a tile more than blocks: the XCDs share the tiles
        c = [372 + e % 3 for e in range(E)]
    elif kind.startswith("few"):   # so many active experts, one to eight row tiles each
        c = [0] * E
        for i in range(int(kind[3:])):
            c[(5 * i + 2) % E] = 124 * E // int(kind[3:]) + 37 * i
    else:                      # few active experts, far apart
        c = [0] * E
        c[3], c[4], c[E - 1] = 90 * E, 33, 110 * E
    return c


@pytest.mark.parametrize("kind,E,D,F,bias", [
    ("even", 150, 128, 1024, False), ("even", 80, 264, 1032, True), ("hot", 100, 520, 1032, True), ("hot", 80, 1024, 264, False),
    ("sparse", 76, 328, 1344, True), ("even", 150, 72, 1032, True),
    ("few1", 8, 3080, 3144, True), ("few2", 8, 3080, 3144, False), ("few7", 8, 3072, 3080, False), ("few6", 16, 1544, 1608, True),
    ("level", 42, 520, 1288, True)])
def test_rows_of_every_height(kind, E, D, F, bias):
    print("ring", kind, E, D, F, flush=True)
    counts = counts_of(kind, E)
    N = sum(counts)
    assert expert_tile_shape(N, E, F, D) == "cut to rows"
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    g = torch.Generator(device="cuda").manual_seed(7)
    t = lambda s, std: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g)
    xp, w1, w2 = t((N, D), 1.0), t((E, F, D), D ** -0.5), t((E, D, F), F ** -0.5)
    b1, b2 = (t((E, F), 0.5), t((E, D), 0.5)) if bias else (None, None)
    idle = [e for e, c in enumerate(counts) if c == 0]
    w1[idle], w2[idle] = float("nan"), float("nan")
    layer = binding.MoeLayer(N, D, F, E, 1, "bf16")
    yp = to_np(layer.moe_expert_ffn(xp, torch.from_numpy(offsets).cuda(), w1, w2, b1, b2))
    ref = orc.expert_ffn(xp.cpu(), offsets, w1.nan_to_num().cpu(), w2.nan_to_num().cpu(), None if b1 is None else b1.cpu(),
                         None if b2 is None else b2.cpu())
    assert np.all(np.isfinite(yp))
    assert norm_max_err(yp, ref) <= TOL["bf16"]          # h and y are each rounded to bf16 once, as in the other shapes' tests
    assert worst_row_rms_rel_err(yp, ref) <= 2.0 ** -7
