"""Expert GEMMs whose K loop goes round K from a place of the tile's own (turned_k: weight rows of a multiple of 4 KB), in every
tile shape that does so, at row counts around the tiles' edges and with columns that end inside a tile; with biases and idle
experts."""
import pytest

from test_gpu_tile_shapes import ragged, run

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 31, 32, 33, 0, 63, 64, 65, 127, 128, 129]


@pytest.mark.parametrize("shape,E,D,F,lo,hi", [
    ("cut to rows", 40, 2048, 1096, 120, 260),    # the first GEMM turns: 32 K tiles
    ("cut to rows", 40, 1096, 4096, 120, 260),    # the second one: 64
    ("128x128", 14, 2048, 776, 100, 120), ("128x128", 14, 776, 2048, 100, 120),
    ("64x128", 80, 2048, 320, 25, 50), ("64x128", 80, 320, 4096, 25, 50),
    ("32x128", 120, 2048, 320, 5, 15), ("32x128", 120, 320, 2048, 5, 15)])
def test_tiles(shape, E, D, F, lo, hi):
    run(shape, ragged(E, EDGES, lo, hi, 4), D, F)


@pytest.mark.parametrize("D,F", [(4096, 544), (544, 8192)])   # the streaming kernel: 4096 and 8192 in parts of a wave each
def test_streams(D, F):
    run("32x128", [0, 1, 3, 0, 16, 17, 2, 33], D, F)
