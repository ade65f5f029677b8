"""Routing by one block (route_small, route.hip) around its rounds of 1024 assignments, its limit, and expert counts around the
bits of the index it ballots on."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as orc
from paper_2303_06182_amd import binding
from helpers import to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E", [1, 2, 3, 64, 65, 1000, 1024])
def test_counts_and_rows(E):
    for n in (1, 63, 64, 65, 1023, 1024, 1025, 2047, 2048, 2049):
        print("route", E, n, flush=True)
        rng = np.random.default_rng(n * 31 + E)
        idx = rng.integers(0, E, (n, 1)).astype(np.int32)
        if n % 2:
            idx[: n // 2] = E - 1   # a hot expert: whole waves of one index
        got = binding.MoeLayer(n, 64, 64, E, 1, "bf16").moe_route_counts(torch.from_numpy(idx).cuda())
        for a, b in zip(got, orc.route(idx, E)):
            assert np.array_equal(to_np(a), b)
