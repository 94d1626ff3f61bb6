"""The grouped linear's choice between the split kernel and the others, a host function: each where it was measured the faster one."""
from __future__ import annotations

from tests.dispatch import grouped_form


def test_a_round_counts_the_columns_of_the_fullest_xcd():
    """Groups of 4, one workgroup a CU: 35 columns' runs go round eight XCDs, five to some, so 7 rows of 245 workgroups fill 280 places."""
    assert grouped_form(64, 1024, 1024, 4, False) and grouped_form(24, 1854, 576, 4, False)
    for M, K, N in ((94, 1920, 664), (98, 1728, 548), (79, 2816, 812), (44, 2752, 1305)):
        assert grouped_form(M, N, K, 4, False) == 0, (M, K, N)


def test_short_contractions_of_many_tiles_keep_the_other_kernels():
    for M, K, N, group in ((443, 512, 920, 16), (264, 512, 1559, 16), (476, 512, 827, 16), (18, 192, 10368, 8), (128, 64, 1176, 16), (300, 128, 400, 4),
                           (17, 64, 66, 16), (737, 64, 1280, 64)):
        assert grouped_form(M, N, K, group, False) == 0, (M, K, N, group)
    for M, K, N, group in ((110, 512, 2000, 16), (154, 1408, 2725, 16), (16, 1024, 1024, 16), (185, 768, 3855, 32), (64, 64, 1024, 64)):
        assert grouped_form(M, N, K, group, False) != 0, (M, K, N, group)


def test_few_groups_and_second_rounds():
    for M, K, N, group, blocked in ((290, 6656, 1664, 128, False), (485, 4096, 1568, 64, False), (323, 5120, 1104, 256, False), (1031, 4096, 304, 512, False),
                                    (315, 6144, 1144, 1024, False), (1094, 1024, 384, 1024, True), (1030, 1024, 392, 1024, True)):
        assert grouped_form(M, N, K, group, blocked) in ((0, 2) if group == 1024 or group == 256 else (0,)), (M, K, N, group)
    for M, K, N, group, blocked in ((128, 512, 2048, 512, True), (128, 2048, 1024, 1024, False), (64, 1024, 1024, 1024, True), (128, 4096, 4096, 64, True)):
        assert grouped_form(M, N, K, group, blocked) != 0, (M, K, N, group)
