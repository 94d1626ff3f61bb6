"""The any-K linear's choice between the few-row kernel and the tiles, and of the tile, host functions: each where it was measured the
faster one."""
from __future__ import annotations

import pytest

from tests.dispatch import anyk_few_rows, anyk_tile


@pytest.mark.parametrize("K,most", [(1000, 64), (1376, 64), (516, 48), (764, 48), (1284, 64), (2500, 64), (777, 32), (638, 16), (514, 32), (2823, 32), (1030, 32), (250, 32), (127, 32),
                                    (1026, 16), (2818, 16), (2814, 16), (1023, 16), (1025, 16), (1027, 24), (2815, 13), (2817, 13), (3841, 13)])
def test_most_rows(K, most):
    assert anyk_few_rows(most, 1000, K) and not anyk_few_rows(most + 1, 1000, K)


@pytest.mark.parametrize("K", [1, 63, 64])
def test_short_rows_keep_the_tiles(K):
    assert not anyk_few_rows(1, 1000, K)


# between them the sizes around 257 tiles of 128x128, 512 and 768 of 64x128, two rounds of 256x128 and 192 to 256 of 64x128
TILES = [((1547, 2459), 368, (64, 128, 4)), ((1562, 2502), 5688, (64, 128, 4)), ((1034, 3759), 3751, (64, 128, 4)), ((1500, 3001), 1023, (64, 128, 4)),
         ((1500, 3001), 1025, (256, 128, 8)), ((838, 6126), 313, (64, 128, 4)), ((806, 7286), 70, (64, 128, 4)), ((806, 7686), 70, (128, 128, 8)), ((1000, 7168), 200, (256, 128, 8)),
         ((1000, 5000), 1376, (256, 128, 8)), ((1000, 4096), 1376, (128, 128, 8)), ((1226, 12421), 347, (128, 128, 8)), ((4096, 4096), 1376, (256, 128, 8)),
         ((4096, 4096), 1000, (128, 128, 8)), ((8192, 16384), 1040, (128, 128, 4)), ((300, 16385), 200, (64, 128, 4)), ((1000, 2048), 130, (64, 128, 8)),
         ((1100, 1500), 255, (64, 64, 4)), ((1100, 1500), 257, (64, 128, 8)), ((333, 700), 1376, (32, 64, 4))]


@pytest.mark.parametrize("mn,K,tile", TILES)
def test_tiles_where_each_was_measured_fastest(mn, K, tile):
    assert anyk_tile(*mn, K) == tile
