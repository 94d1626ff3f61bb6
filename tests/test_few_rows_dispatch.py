"""The few-row linear's choices, host functions of the library: each where it was measured the faster one."""
from __future__ import annotations

import pytest

from paper_2512_14481_amd import binding as B
from tests.dispatch import linear_block_rows, linear_long_rows, linear_quantizes, linear_streams, linear_takes_few_rows, linear_turns

ROW_MAJOR, BLOCKED8, BLOCKED4 = B.SASQ_W_INT8, B.SASQ_W_INT8_BLOCKED, B.SASQ_W_INT4_BLOCKED


def test_weights_that_the_caches_hold_are_not_streamed():
    assert not linear_streams([(8, 11008, 4096)], ROW_MAJOR) and not linear_streams([(32, 16384, 8192)], ROW_MAJOR)
    assert linear_streams([(8, 22016, 8192)], ROW_MAJOR) and linear_streams([(8, 16385, 8192)], ROW_MAJOR)
    assert linear_streams([(1, 256, 256)], BLOCKED8) and linear_streams([(1, 256, 256)], BLOCKED4)


def test_rows_off_whole_lines_are_not_streamed():
    """K an odd multiple of 64: two pieces of a row share most cache lines."""
    assert not linear_streams([(8, 22016, 8256)], ROW_MAJOR) and not linear_streams([(40, 28672, 7232)], ROW_MAJOR)
    assert not linear_streams([(8, 16384, 8192), (8, 11008, 4160)], ROW_MAJOR)
    assert linear_streams([(8, 22016, 8320)], ROW_MAJOR) and linear_streams([(8, 22016, 8256)], BLOCKED8)


def test_long_rows_whatever_the_columns():
    for n in (8192, 9001, 16383, 28671):
        assert linear_long_rows([(8, n, 8192)]) and not linear_long_rows([(8, n, 8128)]), n
    assert linear_long_rows([(8, 8191, 4096), (8, 8191, 12288)]) and not linear_long_rows([(8, 8192, 4096), (8, 8191, 12288)])


# (rows, columns, the first K tiles of a row that turn, whether the call quantizes in the kernel there): even and odd lengths for row-major
TURNS = {ROW_MAJOR: [(1, 3000, 8, 11, True), (16, 5000, 8, 11, True), (8, 9001, 6, 11, True), (20, 4200, 8, 11, True), (40, 1000, 8, 11, True),
                     (30, 8200, 12, 29, False), (40, 8200, 12, 17, False), (64, 9001, 12, 17, False)],
         BLOCKED8: [(8, 3000, 16, 17, True), (16, 3000, 32, 33, True), (3, 9001, 32, 33, True), (40, 500, 8, 9, True), (64, 2000, 12, 13, True),
                    (32, 4200, 8, 9, True)],
         BLOCKED4: [(8, 3000, 10, 9, True), (16, 9001, 32, 33, True), (40, 500, 8, 9, True), (64, 4000, 12, 13, True)]}


@pytest.mark.parametrize("wf", TURNS)
def test_short_contractions_keep_the_order_of_the_matrix_units(wf):
    for rows, columns, even, odd, quantizes in TURNS[wf]:
        for first in (even, odd):
            item = (rows, columns, 64 * first)
            assert linear_takes_few_rows([item], wf) and linear_quantizes([item], wf) == quantizes, item
            assert linear_turns([item], wf), item
            assert not linear_turns([(rows, columns, 64 * (first - 2))], wf), item


def test_forms_that_never_turn():
    """33 to 64 rows quantized in row tiles, which hold two registers' worth of activations; int4 of 9 to 16 rows in narrow workgroups."""
    for item in ((40, 3000, 192), (64, 3000, 448), (64, 4200, 512), (33, 8100, 384)):
        assert linear_quantizes([item], ROW_MAJOR) and not linear_turns([item], ROW_MAJOR), item
    for wf in (BLOCKED8, BLOCKED4):
        items = [(64, 2600, 512)] * 3
        assert linear_quantizes(items, wf) and not linear_turns(items, wf)
    for k in (64, 1024, 8192, 16384):
        assert not linear_turns([(9, 3000, k)], BLOCKED4) and not linear_turns([(16, 500, k)], BLOCKED4)


@pytest.mark.parametrize("rows,dims,want", [
    ((96, 70), [(8200, 128), (8501, 192)], (0, 0, 0)),
    ((66, 80, 96), [(6000, 128), (6500, 64), (5111, 192)], (0, 0, 0)),
    ((97, 66), [(8200, 128), (8501, 192)], (0, 0, 0)),
    ((100, 128), [(8200, 2048), (8501, 2112)], (0, 0, 64)),
    ((70, 96), [(17000, 128), (17000, 128)], (0, 0, 0)),                       # 134 tiles, more than half of a round
    ((90, 65), [(20000, 2048), (20000, 2048)], (0, 0, 96))])
def test_batches_of_many_columns(rows, dims, want):
    """65 to 128 rows: most on the GEMM's tiles, int4's longest on row blocks."""
    items = [(m, n, k) for m, (n, k) in zip(rows, dims)]
    assert tuple(linear_block_rows(items, wf) for wf in (ROW_MAJOR, BLOCKED8, BLOCKED4)) == want
