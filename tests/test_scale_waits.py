"""The block scales' way into LDS in the direct-to-LDS loop over 4-bit weights (gemm_bf16.hip): a model of the loop's loads and
waits.  Loads complete in order; a wait leaves the newest n in flight; a group's scales must have landed before its first K tile."""
import ctypes

import pytest

from paper_2303_06182_amd import binding


def late_groups(KT, stages, lps, tiles, drains):
    """Groups (by their number in the block's sequence of tiles) whose scales may still be in flight as the group begins."""
    flight, late = [], []            # loads in flight, oldest first: ("s", group) or ("k", K tile of the sequence)
    requested = 0

    def scales():
        nonlocal requested
        flight.append(("s", requested))
        requested += 1

    def wait(n):
        del flight[:max(0, len(flight) - n)]

    def k_tile(i):
        flight.extend([("k", i)] * lps)

    scales(), scales()
    for i in range(stages - 1):
        k_tile(i)
    wait((stages - 2) * lps)
    loaded, group, done = stages - 1, 0, 0
    for tile in range(tiles):
        for kt in range(KT):
            if kt % 8 == 0 and (kt or tile):
                if drains:
                    wait(0)
                group += 1
                scales()
            if kt % 8 == 0 and ("s", group) in flight:
                late.append(group)
            assert ("k", done) not in flight
            k_tile(loaded)
            loaded, done = loaded + 1, done + 1
            wait((stages - 2) * lps)
    return late


def rule(KT, stages):
    f = binding.load_library()["_ZN6moe35526gemm_bf16_scales_in_flightEii"]
    f.argtypes, f.restype = [ctypes.c_int] * 2, ctypes.c_bool
    return f(KT, stages)


@pytest.mark.parametrize("stages", [3, 4, 5, 6])
def test_scales_have_landed(stages):
    for KT in range(1, 70):
        for lps in (2, 3, 5):        # a wave's loads per K tile
            assert late_groups(KT, stages, lps, 5, rule(KT, stages)) == []
            # and the loop waits only where it has to
            assert bool(late_groups(KT, stages, lps, 5, False)) == rule(KT, stages)


def test_the_model_sees_a_short_last_group():
    assert late_groups(9, 4, 3, 3, False) == [2, 4]   # each tile's second group is one K tile long: the next tile's first is late
