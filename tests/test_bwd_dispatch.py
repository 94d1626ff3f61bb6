"""The backward linear's choice of kernels, a host function: calls that take the few-row and row-block kernels stay inside the range of
their 32-bit lane offsets, whatever contraction the entry point accepts."""
from __future__ import annotations

import random

import pytest

from tests.dispatch import bwd_reads_lines, bwd_rows, bwd_tile, bwd_turns

MOST = 2 ** 40                                              # the entry point's limit on each product of two sizes


def largest_offset(rows, N):
    """Largest lane offset in bytes: the last row of a block in dY, the last of its 64 columns' weight blocks, the last K tile."""
    return max((max(rows, 64) - 1) * 2 * N, 3 * (N // 32) * 1024) + N // 32 * 1024 + 1024


def test_no_call_wraps_its_offsets():
    rng = random.Random(11)
    shapes = [(1025, 23068672, 1024), (1025, 34603008, 512), (600, 45088768, 512), (1056, 36 << 20, 512), (16, 1 << 27, 16), (32, 1 << 26, 4096)]
    for _ in range(20000):
        M, N, K = (int(2 ** rng.uniform(0, top)) for top in (14, 29.9, 16))
        N = max(N // 32, 1) * 32
        if max(M * N, M * K, N * K) <= MOST:
            shapes.append((M, N, K))
    taken = [(s, bwd_rows(*s)) for s in shapes]
    wrapped = [(s, rows) for s, rows in taken if rows and largest_offset(rows, s[1]) >= 2 ** 32]
    assert not wrapped, wrapped[:5]
    assert sum(rows != 0 for _, rows in taken) > 1000


def test_tiles_where_each_was_measured_fastest():
    for shape in ((2920, 3904, 8448), (1926, 4288, 11008), (3000, 2304, 3328), (4096, 4096, 11008)):
        assert bwd_tile(*shape) == (256, 256), shape
    for shape in ((409, 8576, 15808), (674, 6016, 10560), (2439, 10272, 2753), (2000, 3904, 3904), (3500, 1920, 1920)):
        assert bwd_tile(*shape) == (128, 256), shape
    for shape in ((537, 128, 6720), (376, 96, 10944), (1647, 96, 19008), (3379, 320, 9280), (2218, 160, 2112), (1000, 2304, 2816),
                  (1023, 4416, 4416), (895, 4800, 4800), (2429, 8640, 2176), (1007, 12928, 4224), (1400, 4416, 4416), (1144, 1568, 4928)):
        assert bwd_tile(*shape) == (128, 128), shape


def test_few_rows_and_row_blocks_where_each_was_measured_fastest():
    """On the tiles: many columns of 17 to 64 rows, short contractions of large small blocks; off them: fewer columns, long contractions."""
    for shape in ((30, 4480, 24768), (28, 2400, 25216), (40, 4224, 17792), (51, 960, 24960), (53, 160, 16392), (198, 64, 1984),
                  (643, 2688, 1216), (342, 3200, 3968), (838, 544, 9168)):
        assert bwd_rows(*shape) == 0, shape
    for shape, rows in (((1, 4096, 4096), 64), ((16, 4096, 27456), 64), ((17, 9696, 9728), 64), ((25, 13248, 8896), 64), ((64, 256, 256), 32),
                        ((334, 11072, 1536), 64), ((198, 128, 1984), 32)):
        assert bwd_rows(*shape) == rows, shape


# (rows, outputs, the first even and the first odd number of contraction tiles that turn), None: none does
TURNS = [(1, 1000, None, None), (8, 9000, None, None), (12, 1000, 10, 65), (16, 9000, 64, 65), (40, 500, 8, 33), (64, 1500, 8, 33), (100, 4000, 14, 65),
         (30, 6000, 16, None), (50, 9000, 32, 65), (200, 9000, 2, 33)]


@pytest.mark.parametrize("M,K,even,odd", TURNS)
def test_short_contractions_keep_the_order_of_the_matrix_units(M, K, even, odd):
    for first, parity in ((even, 0), (odd, 1)):
        for tiles in range(2 - parity, 400, 2):
            assert bwd_turns(M, 32 * tiles, K) == (first is not None and tiles >= first), (M, tiles, K)


@pytest.mark.parametrize("tile_rows,first", [(128, 32), (256, 64)])
def test_short_contractions_read_half_lines(tile_rows, first):
    for tiles in range(1, 300):
        assert bwd_reads_lines(32 * tiles, tile_rows) == (tiles % 2 == 0 and tiles >= first), tiles
