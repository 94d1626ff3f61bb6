"""GPU parity of the grouped linear's matrix-unit loops at the edges of their forms: groups of one, two, four, other even and other odd
numbers of K tiles; contractions of one to a few tiles, shorter than the four that are requested ahead; an odd number of groups."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from tests.gpu_util import assert_same_values
from tests.test_gpu_grouped_linear import problem, run_grouped

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles,groups", [(1, 1), (1, 2), (1, 3), (1, 9), (1, 12), (2, 1), (2, 2), (2, 5), (3, 1), (3, 2), (3, 3), (4, 1),
                                          (4, 3), (5, 3), (6, 1), (6, 3), (8, 2), (12, 1)])
@pytest.mark.parametrize("dtype,fmt,blocked", [("f16", "int8", False), ("bf16", "int8", True), ("f16", "int4", True)])
def test_groups_of_whole_tiles_match_oracle(tiles, groups, dtype, fmt, blocked):
    shape, group = (70, 136, 64 * tiles * groups), 64 * tiles
    xb, wq, s_w, bias, s_g = problem(57, shape, group, dtype, fmt)
    ref = oracle.static_linear_grouped(xb, s_g, wq, s_w, bias, group, 8, fmt, dtype)
    y, f, _ = run_grouped(xb, s_g, wq, s_w, bias, group, fmt, dtype, blocked, tile="128")
    assert np.array_equal(f, ref["f"])
    assert_same_values(y, ref["y"], dtype, "Y")
