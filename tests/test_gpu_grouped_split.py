"""Grouped linear, calls of few output tiles: the contraction split over the waves (grouped_split.hip), each of its forms at
remainders of rows, columns, K tiles and phases, and the per-channel kernel's one- and two-row forms.  Bit for bit against the
oracle, as the chain of fused multiply-adds is part of the contract; the general kernels, asked for by a knob, give the same."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import assert_same_values, set_tuning
from tests.test_gpu_grouped_linear import problem, run_grouped

pytestmark = pytest.mark.gpu


def check(shape, group, dtype, blocked):
    xb, wq, s_w, bias, s_g = problem(71, shape, group, dtype, "int8")
    s_g[0] *= 1e-3                                                 # the first group saturates: codes -128 and 127
    ref = oracle.static_linear_grouped(xb, s_g, wq, s_w, bias, group, 8, "int8", dtype)
    y, f, _ = run_grouped(xb, s_g, wq, s_w, bias, group, "int8", dtype, blocked)
    assert np.array_equal(f, ref["f"]), "fp32 group sums"
    assert_same_values(y, ref["y"], dtype, "y")
    y2, _, _ = run_grouped(xb, s_g, wq, s_w, None, group, "int8", dtype, blocked, want_debug=False)
    ref2 = oracle.static_linear_grouped(xb, s_g, wq, s_w, None, group, 8, "int8", dtype)
    assert_same_values(y2, ref2["y"], dtype, "y without bias")


# (rows, columns, K): fewer K tiles than waves, a last phase that is not full, several phases
@pytest.mark.parametrize("blocked", [False, True])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("shape,group", [
    ((5, 33, 704), 32), ((17, 66, 64), 32), ((16, 128, 1024), 32), ((387, 395, 576), 32),               # 16 x 16 and 16 x 32 outputs
    ((5, 33, 704), 64), ((1, 1, 64), 64), ((129, 501, 576), 64), ((390, 970, 192), 64),                 # and 32 x 32, row-major
    ((33, 100, 576), 192), ((100, 300, 1152), 128), ((16, 16, 4096), 128), ((390, 970, 256), 128), ((70, 1100, 1024), 512)])
def test_split(shape, group, dtype, blocked):
    check(shape, group, dtype, blocked)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("shape,group", [
    ((5, 33, 320), 4), ((16, 300, 64), 4), ((33, 70, 576), 4), ((5, 33, 704), 8), ((33, 130, 64), 8), ((16, 512, 1024), 8),
    ((5, 33, 704), 16), ((17, 66, 64), 16), ((40, 333, 1088), 16), ((16, 4, 4096), 16),
    ((1, 1, 64), 1), ((3, 100, 130), 1), ((64, 1000, 80), 1), ((40, 1700, 80), 1), ((16, 4090, 144), 1), ((128, 2500, 65), 1)])
def test_split_small_groups(shape, group, dtype):
    check(shape, group, dtype, False)


# either side of the lines of the dispatch: the general kernel's result is the split one's
@pytest.mark.parametrize("rows,cols,k,group", [(256, 256, 128, 4), (257, 256, 128, 4), (512, 256, 128, 8), (513, 256, 128, 8),
                                               (480, 960, 64, 16), (481, 960, 64, 16), (800, 1120, 64, 32), (801, 1120, 64, 32),
                                               (760, 1024, 128, 64), (780, 1024, 128, 64)])
def test_lines(rows, cols, k, group):
    xb, wq, s_w, bias, s_g = problem(72, (rows, cols, k), group, "bf16", "int8")
    y, f, xq = run_grouped(xb, s_g, wq, s_w, bias, group, "int8", "bf16", False)
    set_tuning(path="twopass")
    try:
        y2, f2, xq2 = run_grouped(xb, s_g, wq, s_w, bias, group, "int8", "bf16", False)
    finally:
        set_tuning()
    assert np.array_equal(f, f2) and np.array_equal(y, y2) and np.array_equal(xq, xq2)
