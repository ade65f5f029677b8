"""The ring kernel's schedule (csrc/ring_schedule.h), run on the host: every 32-row unit of every expert belongs to exactly
one part, whatever the batch, and the parts cost about the same."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2303_06182_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = tmp_path_factory.mktemp("ring") / "ring_schedule.so"
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__host__=", "-D__device__=", "-D__forceinline__=inline",
                    "-I", CSRC, os.path.join(HERE, "ring_schedule_host.cpp"), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so))


def check(lib, counts):
    rows = np.asarray(counts, dtype=np.int32)
    units = int(((rows + 31) // 32).sum())
    covered, cost = np.zeros(units, dtype=np.int32), np.zeros(8, dtype=np.int32)
    ptr = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    assert lib.ring_cover(ptr(rows), len(rows), ptr(covered), ptr(cost)) == units, counts
    assert np.all(covered == 1), counts
    assert cost.max() <= cost.sum() / 8 + 2 * 14, counts   # a tile of 256 rows, which costs 14, too many at either end


@pytest.mark.parametrize("counts", [[n] for n in (1, 32, 257, 512, 1000, 1024, 1400, 100000)]
                         + [[513, 513], [512, 0, 512], [512, 300, 212], [0] * 127 + [1024], [1024] + [0] * 7])
def test_few_active_experts(lib, counts):
    check(lib, counts)


def test_random_batches(lib):
    rng = np.random.default_rng(3)
    for _ in range(3000):
        E = int(rng.choice([1, 2, 8, 24, 128, 512, 1024]))
        counts = np.zeros(E, dtype=np.int64)
        active = rng.permutation(E)[: int(rng.integers(1, 13)) if rng.random() < 0.5 else E]
        n = int(2 ** rng.uniform(0, 15))
        weight = 1.0 / np.arange(1, len(active) + 1) ** rng.choice([0.0, 0.8, 1.2])
        counts[active] = rng.multinomial(n, weight / weight.sum())
        check(lib, counts)


def test_shared_list(lib):
    first = np.zeros(9, dtype=np.int32)
    for tiles in list(range(0, 300)) + [32 * 112, 32 * 4096 + 1]:
        lib.ring_shares(tiles, first.ctypes.data_as(ctypes.c_void_p))
        assert first[0] == 0 and first[8] == tiles and np.all(np.diff(first) >= 0)
        assert np.diff(first).max() == -(-tiles // 8)
