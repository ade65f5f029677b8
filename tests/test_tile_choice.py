"""Which tile shape the library chooses for the bf16 expert GEMMs, around the lines of its rule."""
import pytest

from helpers import expert_tile_shape


@pytest.mark.parametrize("E,D,F,rows,shape", [
    # few rows per expert: 2^29 weights and two 256-column panels per CU, or the small tiles
    (128, 2048, 8192, 8, "cut to rows"), (128, 2048, 8192, 7, "32x128"), (512, 1024, 4096, 8, "cut to rows"),
    (128, 512, 2048, 24, "32x128"), (64, 2048, 8192, 30, "cut to rows"),
    (512, 512, 2048, 8, "32x128"), (512, 512, 2048, 40, "64x128"), (512, 512, 2048, 100, "128x128"),
    (32, 2048, 8192, 29, "32x128"), (32, 2048, 8192, 64, "128x128"), (16, 4096, 14336, 32, "128x128"),
    (16, 4096, 14336, 100, "128x128"), (8, 6144, 16384, 8, "32x128"), (8, 6144, 16384, 100, "128x128"),
    (4, 8192, 28672, 8, "32x128"), (4, 8192, 28672, 100, "128x128"), (8, 4096, 14336, 100, "128x128"),
    # from 116 rows, given 96 tiles, 120 with fewer than 112
    (32, 1024, 4096, 115, "128x128"), (32, 1024, 4096, 116, "cut to rows"), (8, 4096, 14336, 128, "cut to rows"),
    (24, 1000, 4000, 119, "128x128"), (24, 1000, 4000, 120, "cut to rows"), (28, 1000, 4000, 116, "cut to rows"),
    (11, 2048, 8192, 200, "128x128"), (12, 2048, 8192, 200, "cut to rows"), (8, 2048, 8192, 240, "128x128"),
    (8, 2048, 8192, 250, "cut to rows"),
    # a dimension of 768 and less: from 192 rows, given 144 tiles and 1024 as the other dimension
    (128, 512, 2048, 191, "128x128"), (128, 512, 2048, 192, "cut to rows"), (66, 768, 768, 124, "128x128"),
    (48, 768, 1016, 1000, "128x128"), (48, 768, 1024, 1000, "cut to rows"), (47, 768, 3072, 200, "128x128"),
    (48, 3072, 768, 200, "cut to rows"), (191, 256, 256, 228, "128x128"), (8, 256, 3328, 1500, "128x128"),
    (8, 256, 3328, 5000, "cut to rows"),
    # a dimension of 64 and less: one K tile
    (64, 64, 256, 800, "128x128"), (64, 72, 1024, 800, "cut to rows"), (16, 4096, 64, 1000, "128x128"), (128, 40, 512, 1000, "128x128"),
])
def test_choice(E, D, F, rows, shape):
    assert expert_tile_shape(E * rows, E, F, D) == shape


def test_operands_past_32_bit_offsets():
    assert expert_tile_shape(1 << 18, 8, 8192, 2048) == "256x256"      # 4 GiB of hidden rows
    assert expert_tile_shape(258000, 8, 8192, 2048) == "cut to rows"
