"""The any-K linear's choice between the few-row kernel and the tiles, a host function: each where it was measured the faster one."""
from __future__ import annotations

import pytest

from tests.dispatch import anyk_few_rows


@pytest.mark.parametrize("K,most", [(1000, 64), (1376, 64), (516, 48), (764, 48), (1284, 64), (2500, 64), (777, 32), (638, 16), (514, 32), (2823, 32), (1030, 32), (250, 32), (127, 32),
                                    (1026, 16), (2818, 16), (2814, 16), (1023, 16), (1025, 16), (1027, 24), (2815, 13), (2817, 13), (3841, 13)])
def test_most_rows(K, most):
    assert anyk_few_rows(most, 1000, K) and not anyk_few_rows(most + 1, 1000, K)


@pytest.mark.parametrize("K", [1, 63, 64])
def test_short_rows_keep_the_tiles(K):
    assert not anyk_few_rows(1, 1000, K)
