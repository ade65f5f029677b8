"""The fused gate kernel's tile heights (32, 64, 128 rows with a wave per column block, gate_topk.hip): tokens around them, expert
counts around the 32-column blocks, one K tile and fewer than stages, up to eight experts a token.  Logits against the fp64 oracle,
the selection and its order exactly against the oracle's rule on the kernel's own logits, the histogram through the layer."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as orc
from paper_2303_06182_amd import binding
from helpers import to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,D,E,k,renorm,bias", [
    (257, 64, 1, 1, True, False), (300, 64, 32, 2, True, True), (289, 128, 33, 3, False, True), (1000, 320, 64, 8, True, False),
    (8192, 192, 65, 2, False, False), (500, 1024, 97, 2, True, True), (320, 576, 128, 8, False, True),
    (8193, 64, 7, 2, True, True), (8200, 192, 50, 1, False, False), (12001, 128, 96, 2, True, True), (16384, 320, 126, 2, False, True),
    (16385, 64, 66, 2, True, True), (16500, 192, 100, 4, False, False), (24576, 128, 128, 2, True, True), (24577, 128, 128, 2, True, True),
    # 32 experts and fewer: a wave per 32 rows up to 512 dimensions, 256 from 32 rows per CU on
    (300, 512, 32, 2, True, True), (8192, 512, 31, 8, False, False), (300, 576, 32, 2, True, False), (8193, 256, 32, 2, False, True),
    (8193, 320, 32, 2, True, True), (16384, 256, 5, 1, True, False), (16385, 256, 32, 2, True, True)])
def test_gate(T, D, E, k, renorm, bias):
    print("gate", T, D, E, k, flush=True)
    g = torch.Generator(device="cuda").manual_seed(T + E)
    x = torch.empty((T, D), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    wg = torch.empty((E, D), dtype=torch.bfloat16, device="cuda").normal_(0, D ** -0.5, generator=g)
    if E > 2:
        wg[E - 1] = wg[0]   # equal logits: ties go to the lower expert
    gb = torch.empty(E, device="cuda").normal_(0, 1, generator=g) if bias else None
    m = binding.MoeLayer(T, D, 64, E, k, "bf16", renorm)
    logits, idx, w = m.moe_gate_topk(x, wg, gb)
    got = to_np(logits)
    ref = orc.gate_logits(x.cpu(), wg.cpu(), None if gb is None else gb.cpu())
    assert np.abs(got - ref).max() <= 2e-6 * np.abs(ref).max() + 1e-7
    ridx, rw = orc.topk(got, k, renorm)
    np.testing.assert_array_equal(to_np(idx), ridx)
    np.testing.assert_allclose(to_np(w), rw, rtol=2e-6, atol=1e-9)
    # without the logits in memory the same decision, and the routing that starts from the tiles' histograms
    w1 = torch.zeros((E, 64, D), dtype=torch.bfloat16, device="cuda")
    w2 = torch.zeros((E, D, 64), dtype=torch.bfloat16, device="cuda")
    r = m.empty_routing(T)
    del r["logits"]
    m.moe_layer_forward(x, wg, w1, w2, gb, routing_out=r)
    np.testing.assert_array_equal(to_np(r["topk_idx"]), ridx)
    for name, want in zip(("counts", "offsets", "dst_row", "src_tok"), orc.route(ridx, E)):
        np.testing.assert_array_equal(to_np(r[name]), want)


@pytest.mark.parametrize("T,D,E,k", [
    (257, 72, 24, 1), (300, 120, 47, 2), (3001, 1000, 24, 1), (1137, 1496, 47, 2), (8193, 328, 60, 2), (16385, 136, 66, 2),
    (24577, 200, 128, 2), (24577, 392, 50, 3), (40001, 72, 128, 2), (66000, 104, 7, 2), (300, 2040, 128, 8), (301, 504, 32, 2), (301, 520, 32, 2),
    (9000, 264, 30, 2)])
def test_k_ends_inside_a_tile(T, D, E, k):
    test_gate(T, D, E, k, T % 2 == 0, True)


def test_nothing_past_k_is_multiplied():
    """The last row's chunks past K lie behind the arrays, the other rows' in the next row: infinities there must not reach a sum."""
    T, D, E = 320, 200, 40
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.empty((T, D), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    wg = torch.empty((E, D), dtype=torch.bfloat16, device="cuda").normal_(0, 0.1, generator=g)
    x[1::2, :56] = float("inf")   # what follows an even row
    logits, _, _ = binding.MoeLayer(T, D, 64, E, 2, "bf16").moe_gate_topk(x, wg)
    ref = orc.gate_logits(x[::2].cpu(), wg.cpu(), None)
    assert np.abs(to_np(logits)[::2] - ref).max() <= 2e-6 * np.abs(ref).max() + 1e-7
