"""GPU parity of the linear for contraction lengths that are not multiples of 64 on the tiles of eight waves and beside them: row, column
and K remainders on each tile that the dispatch takes, one factor per tensor and one per row."""
from __future__ import annotations

import pytest

from tests.test_gpu_anyk_linear import test_any_contraction_length as check

pytestmark = pytest.mark.gpu

TILES = {(256, 128, 8): (1500, 3001), (128, 128, 8): (1000, 2050), (128, 128, 4): (4100, 4200), (64, 128, 4): (300, 7300),
         (64, 128, 8): (1100, 1500), (64, 64, 4): (700, 1500), (32, 64, 4): (333, 700)}


def chosen(m, n):
    """The tile and its waves by the number of tiles alone.  Which the library takes, by K too: tests/test_gpu_anyk_choice.py."""
    def tiles(bm, bn):
        return -(-m // bm) * -(-n // bn)
    t256, t128, t64 = tiles(256, 128), tiles(128, 128), tiles(64, 128)
    mid = t128 <= 1024 and t128 * 20 <= t64 * 11
    if mid and t128 > 256 and (t256 <= 256 or t256 * 10 >= -(-t256 // 256) * 2304) and t256 * 20 <= t128 * 11:
        return 256, 128, 8
    if mid and t64 > 256:
        return 128, 128, 8
    if t128 >= 512:
        return 128, 128, 4
    if t64 > 256:
        return 64, 128, 4
    if t64 >= 192:
        return 64, 128, 8
    return (64, 64, 4) if tiles(64, 64) >= 256 else (32, 64, 4)


@pytest.mark.parametrize("fmt", ["int8", "int4"])
@pytest.mark.parametrize("k", [81, 130, 400, 650, 1030])
@pytest.mark.parametrize("tile", TILES)
def test_tiles_of_eight_waves(tile, k, fmt):
    assert chosen(*TILES[tile]) == tile
    check(TILES[tile], k, fmt)


@pytest.mark.parametrize("mn,tile", [((4096, 4096), (256, 128, 8)), ((2000, 6144), (128, 128, 8)), ((257, 16385), (64, 128, 4))])
def test_lines_of_the_choice(mn, tile):
    """Two full rounds of the largest tile, a round and a half, and a call with half of a larger tile's rows past the end."""
    assert chosen(*mn) == tile
    check(mn, 130, "int8")
