"""GPU parity of the linear for contraction lengths that are not multiples of 64 on the tile that the library takes, which it is asked for: row,
column and K remainders on each, and both sides of the lines between them."""
from __future__ import annotations

import pytest

from tests.dispatch import anyk_tile
from tests.test_gpu_anyk_linear import test_any_contraction_length as check

pytestmark = pytest.mark.gpu

TILES = {(256, 128, 8): (2900, 2200), (128, 128, 8): (1000, 2050), (128, 128, 4): (4100, 4200), (64, 128, 8): (1000, 2040),
         (64, 128, 4): (300, 7300), (64, 64, 4): (700, 1500), (32, 64, 4): (333, 700)}


@pytest.mark.parametrize("fmt", ["int8", "int4"])
@pytest.mark.parametrize("k", [81, 130, 400, 650, 1030])
@pytest.mark.parametrize("tile", TILES)
def test_tiles(tile, k, fmt):
    assert anyk_tile(*TILES[tile], k) == tile
    check(TILES[tile], k, fmt)


@pytest.mark.parametrize("mn,k,tile", [((4096, 4096), 1030, (256, 128, 8)), ((4096, 4096), 130, (128, 128, 8)), ((2000, 6144), 130, (128, 128, 8)),
                                       ((257, 16385), 130, (64, 128, 4)), ((1500, 3001), 650, (64, 128, 4)), ((1500, 3001), 1030, (256, 128, 8)),
                                       ((1562, 2502), 1030, (64, 128, 4)), ((1100, 1500), 130, (64, 64, 4)), ((1100, 1500), 400, (64, 128, 8))])
def test_lines_of_the_choice(mn, k, tile):
    """Two full rounds of the largest tile, a round and a half, a call with half of a larger tile's rows past the end, and both sides of the
    lines at 257 tiles of 128x128 and 192 of 64x128."""
    assert anyk_tile(*mn, k) == tile
    check(mn, k, "int8")
