"""The expert GEMM's tile shapes that only some sizes reach, against the fp64 oracle.  Each case names the shape it is
for and asks the library whether that is its choice, so that it cannot drift to another one."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as orc
from paper_2303_06182_amd import binding, workloads as wl
from helpers import TOL, expert_tile_shape, norm_max_err, to_np, worst_row_rms_rel_err

pytestmark = pytest.mark.gpu


def ragged(E, edges, lo, hi, seed):
    """Rows per expert: the edges first, the rest spread over lo ... hi."""
    rng = np.random.default_rng(seed)
    return list(edges) + [int(c) for c in rng.integers(lo, hi + 1, E - len(edges))]


def run(shape, counts, D, F):
    """One FFN call with biases; idle experts' weights are NaN.  The reference covers the first experts (the edges)."""
    print("tile shape", shape, len(counts), D, F, sum(counts), flush=True)
    E, N = len(counts), int(sum(counts))
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert expert_tile_shape(N, E, F, D, cus) == shape
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    g = torch.Generator(device="cuda").manual_seed(7)
    t = lambda s, std: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g)
    xp, w1, w2, b1, b2 = t((N, D), 1.0), t((E, F, D), D ** -0.5), t((E, D, F), F ** -0.5), t((E, F), 0.5), t((E, D), 0.5)
    idle = [e for e, c in enumerate(counts) if c == 0]
    w1[idle], w2[idle] = float("nan"), float("nan")
    yp = to_np(binding.MoeLayer(N, D, F, E, 1, "bf16").moe_expert_ffn(xp, torch.from_numpy(offsets).cuda(), w1, w2, b1, b2))
    assert np.all(np.isfinite(yp))
    n = min(E, 12)
    rows = int(offsets[n])
    w1, w2 = (w[:n].nan_to_num().cpu() for w in (w1, w2))
    ref = orc.expert_ffn(xp[:rows].cpu(), offsets[:n + 1], w1, w2, b1[:n].cpu(), b2[:n].cpu())
    assert norm_max_err(yp[:rows], ref) <= TOL["bf16"]
    assert worst_row_rms_rel_err(yp[:rows], ref) <= 2.0 ** -7


def test_64x128():
    run("64x128", ragged(80, [0, 1, 63, 64, 65, 33, 0, 127, 128, 129], 20, 60, 1), 256, 320)


EDGES = [0, 1, 127, 128, 129, 257, 33, 0, 64, 65, 16, 17]   # around half a tile and a tile and a bit


def test_cut_tiles_with_few_rows():
    run("cut to rows", ragged(512, EDGES, 5, 40, 2), 1088, 1088)   # 17 K tiles, a last column tile of 64


def test_cut_tiles_of_about_half_the_height():
    run("cut to rows", ragged(512, EDGES, 120, 150, 3), 1088, 1088)


def test_128x128_with_many_rows():
    run("128x128", [1100, 0, 900, 257, 1500, 640, 3, 700], 264, 3328)   # too few tiles to cut, K that ends inside a K tile


def test_layer_on_cut_tiles():
    """Rows gathered from the token array by the first GEMM; the tokens of the fullest expert (several tiles) and a sample of
    the others against the oracle."""
    T, D, F, E, k = 6000, 1024, 1088, 512, 2
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert expert_tile_shape(T * k, E, F, D, cus) == "cut to rows"
    g = torch.Generator(device="cuda").manual_seed(8)
    t = lambda s, std: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g)
    x, wg, w1, w2 = t((T, D), 1.0), t((E, D), 10 * D ** -0.5), t((E, F, D), D ** -0.5), t((E, D, F), F ** -0.5)
    bias = torch.zeros(E, device="cuda")
    bias[5] = 25.0   # a hot expert
    m = binding.MoeLayer(T, D, F, E, k, "bf16")
    r = m.empty_routing(T)
    y = to_np(m.moe_layer_forward(x, wg, w1, w2, bias, routing_out=r))
    idx, gw, counts = to_np(r["topk_idx"]), to_np(r["topk_w"]), to_np(r["counts"])
    hot = int(counts.argmax())
    assert counts[hot] > 256
    tok = np.unique(np.concatenate([np.flatnonzero((idx == hot).any(axis=1))[::97], np.arange(0, T, 149)]))
    used, local = np.unique(idx[tok], return_inverse=True)
    sel = torch.from_numpy(used).cuda().long()
    ref = orc.layer_tokens(x[tok].cpu(), w1[sel].cpu(), w2[sel].cpu(), local.reshape(len(tok), k).astype(np.int32), gw[tok])
    assert norm_max_err(y[tok], ref) <= TOL["bf16"]
    assert worst_row_rms_rel_err(y[tok], ref) <= 2.0 ** -7


@pytest.mark.parametrize("shape,D,F,n_rows", [
    ("cut to rows", 128, 8192, 258000),     # hidden rows of 3.94 GiB: the last ones' 32-bit byte offsets
    ("256x256", 128, 8192, 262400),         # ... of more: whole rounds of 256x256 tiles and the rest as 128x128
    ("256x256", 72, 8200, 262500)])         # ... with K that ends inside a K tile in both GEMMs
def test_operands_around_4_gib(shape, D, F, n_rows):
    print("4 GiB", shape, D, F, n_rows, flush=True)
    counts = [70000, 1, 0, n_rows - 70000 - 1 - 300, 300]
    E, offsets = len(counts), np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    assert expert_tile_shape(n_rows, E, F, D, torch.cuda.get_device_properties(0).multi_processor_count) == shape
    g = torch.Generator(device="cuda").manual_seed(9)
    t = lambda s, std: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g)
    xp, w1, w2, b1, b2 = t((n_rows, D), 1.0), t((E, F, D), D ** -0.5), t((E, D, F), F ** -0.5), t((E, F), 0.5), t((E, D), 0.5)
    w1[2], w2[2] = float("nan"), float("nan")
    yp = binding.MoeLayer(n_rows, D, F, E, 1, "bf16").moe_expert_ffn(xp, torch.from_numpy(offsets).cuda(), w1, w2, b1, b2)
    assert bool(torch.isfinite(yp).all())
    # every expert's first and last rows, and some in between
    rows = [np.unique(np.concatenate([np.arange(min(c, 40)), np.arange(max(0, c - 40), c), np.arange(0, c, 1501)])) for c in counts]
    sel = torch.from_numpy(np.concatenate([o + r for o, r in zip(offsets, rows)])).cuda().long()
    ref = orc.expert_ffn(xp[sel].cpu(), np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32),
                         w1.nan_to_num().cpu(), w2.nan_to_num().cpu(), b1.cpu(), b2.cpu())
    got = to_np(yp[sel])
    assert norm_max_err(got, ref) <= TOL["bf16"]
    assert worst_row_rms_rel_err(got, ref) <= 2.0 ** -7
