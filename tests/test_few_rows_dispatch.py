"""The few-row linear's choices, host functions of the library: each where it was measured the faster one."""
from __future__ import annotations

from paper_2512_14481_amd import binding as B
from tests.dispatch import linear_long_rows, linear_streams

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
