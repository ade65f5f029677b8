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


@pytest.mark.parametrize("counts,n1,n2,shared", [
    # fewer row tiles than XCDs, or a part with twice the others' tiles
    ([0, 1024] + [0] * 6, 56, 16, True), ([256, 0, 256, 0, 256, 0, 0, 256], 56, 16, True), ([200, 200, 0, 0], 112, 32, True),
    ([260, 237, 257, 265, 231, 256, 228, 226], 56, 16, True), ([372] * 42, 6, 3, True),
    # parts that come out as well as eighths of one list, or better: two row tiles each but for one, one row tile each
    ([268, 280, 271, 264, 246, 272, 282, 301], 56, 16, False), ([284, 311, 258, 258, 278, 290, 285, 276], 56, 16, False),
    ([250, 231, 242, 247, 261, 218, 227, 238, 241, 269, 240, 243, 239, 273, 246, 255], 32, 8, False),
    ([256] * 32, 32, 8, False), ([0] * 8, 32, 8, False)])
def test_when_all_share(lib, counts, n1, n2, shared):
    rows = np.asarray(counts, dtype=np.int32)
    assert bool(lib.ring_is_shared(rows.ctypes.data_as(ctypes.c_void_p), len(rows), n1, n2)) == shared
