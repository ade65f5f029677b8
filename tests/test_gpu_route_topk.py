"""Top-k and routing of a decoder step by one block (route_topk_kernel, route.hip): block sizes of 256, 512 and 1024 threads, expert
counts that are and are not multiples of four, gates of one and of several K slices, one token more than the block takes."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as orc
from paper_2303_06182_amd import binding
from helpers import to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,D,E,k", [
    (1, 2048, 128, 2), (16, 2048, 128, 2), (17, 1024, 128, 2), (64, 2048, 128, 4), (65, 2048, 128, 2), (64, 1024, 8, 8), (1, 128, 4, 1),
    (33, 2048, 512, 2), (32, 2048, 512, 4), (16, 2048, 1024, 8), (17, 1024, 1000, 2), (64, 512, 256, 2), (3, 64, 64, 2), (200, 2048, 512, 3),
    (1, 872, 7, 2), (64, 512, 7, 2), (64, 2048, 3, 3), (64, 512, 15, 2), (32, 1024, 31, 4), (33, 1024, 31, 4), (16, 2048, 63, 2),
    (17, 2048, 63, 2), (16, 512, 127, 8), (5, 128, 33, 1), (9, 1024, 250, 2), (100, 1024, 50, 2), (4, 512, 255, 2),
    # slices added by the lanes and by all threads, batches of more than a block
    (65, 512, 8, 2), (256, 1024, 32, 4), (200, 1024, 64, 2), (201, 2048, 64, 2), (130, 512, 96, 2), (2, 1024, 250, 2), (3, 1024, 250, 2),
    (129, 512, 127, 2), (129, 2048, 127, 2), (66, 1024, 510, 8)])
def test_decoder_step(T, D, E, k):
    print("route_topk", T, D, E, k, flush=True)
    g = torch.Generator(device="cuda").manual_seed(T * 1000 + E)
    x = torch.empty((T, D), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    wg = torch.empty((E, D), dtype=torch.bfloat16, device="cuda").normal_(0, D ** -0.5, generator=g)
    if E > 2:
        wg[E - 1] = wg[0]   # equal logits: ties go to the lower expert
    m = binding.MoeLayer(T, D, 64, E, k, "bf16", T % 2 == 0)
    w1 = torch.zeros((E, 64, D), dtype=torch.bfloat16, device="cuda")
    w2 = torch.zeros((E, D, 64), dtype=torch.bfloat16, device="cuda")
    r = m.empty_routing(T)
    m.moe_layer_forward(x, wg, w1, w2, None, routing_out=r)
    got = to_np(r["logits"])
    ref = orc.gate_logits(x.cpu(), wg.cpu(), None)
    assert np.abs(got - ref).max() <= 2e-6 * np.abs(ref).max() + 1e-7   # fp32 sums of up to 2048 products
    ridx, rw = orc.topk(got, k, T % 2 == 0)
    np.testing.assert_array_equal(to_np(r["topk_idx"]), ridx)
    np.testing.assert_allclose(to_np(r["topk_w"]), rw, rtol=2e-6, atol=1e-9)
    for name, want in zip(("counts", "offsets", "dst_row", "src_tok"), orc.route(ridx, E)):
        np.testing.assert_array_equal(to_np(r[name]), want)
