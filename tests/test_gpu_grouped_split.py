"""Grouped linear, calls of few output tiles: the contraction split over the waves (grouped_split.hip), each of its forms at
remainders of rows, columns, K tiles and phases, and the per-channel kernel's one- and two-row forms.  Bit for bit against the
oracle, as the chain of fused multiply-adds is part of the contract; the general kernels, asked for by a knob, give the same."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from tests.dispatch import grouped_form
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


# (rows, columns, K): fewer K tiles than waves, a last phase that is not full, several phases; with the form that row-major and
# pre-arranged weights take: 1: 16 x 16 outputs, 2: 32 x 32, 3: 16 x 32, 0: the other kernels
@pytest.mark.parametrize("blocked", [False, True])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("shape,group,forms", [
    ((5, 33, 704), 32, (1, 1)), ((17, 66, 64), 32, (1, 1)), ((16, 128, 1024), 32, (1, 1)), ((387, 395, 576), 32, (3, 3)),
    ((5, 33, 704), 64, (1, 1)), ((1, 1, 64), 64, (1, 1)), ((129, 501, 576), 64, (3, 3)), ((390, 970, 192), 64, (2, 3)), ((700, 970, 576), 64, (2, 3)),
    ((33, 100, 576), 192, (1, 1)), ((430, 970, 576), 192, (2, 3)), ((300, 970, 576), 192, (3, 3)), ((100, 300, 1152), 128, (1, 1)), ((16, 16, 4096), 128, (1, 1)),
    ((390, 970, 256), 128, (2, 3)), ((70, 1100, 1024), 512, (3, 3)), ((400, 1030, 1024), 512, (0, 3)), ((240, 1030, 1024), 1024, (3, 3))])
def test_split(shape, group, forms, dtype, blocked):
    M, N, K = shape
    assert grouped_form(M, N, K, group, blocked) == forms[blocked]
    check(shape, group, dtype, blocked)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("shape,group", [
    ((5, 33, 320), 4), ((16, 300, 256), 4), ((33, 70, 576), 4), ((5, 33, 704), 8), ((33, 130, 128), 8), ((16, 512, 1024), 8),
    ((5, 33, 704), 16), ((17, 66, 128), 16), ((40, 333, 1088), 16), ((16, 4, 4096), 16),
    ((1, 1, 64), 1), ((3, 100, 130), 1), ((64, 1000, 80), 1), ((40, 1700, 80), 1), ((16, 4090, 144), 1), ((128, 2500, 65), 1)])
def test_split_small_groups(shape, group, dtype):
    M, N, K = shape
    assert group == 1 or grouped_form(M, N, K, group, False) == 1
    check(shape, group, dtype, False)


# the last shape in front of each line of the dispatch: the most workgroups a form is taken for, against the general kernel
@pytest.mark.parametrize("rows,cols,k,group", [(256, 256, 192, 4), (256, 256, 128, 8), (512, 256, 512, 8), (192, 512, 128, 16), (496, 512, 512, 16),
                                               (448, 1024, 1024, 16), (688, 512, 64, 32), (864, 1024, 512, 32), (800, 970, 576, 64), (496, 970, 576, 192)])
def test_lines(rows, cols, k, group):
    assert grouped_form(rows, cols, k, group, False) != 0 and grouped_form(rows + 16, cols, k, group, False) == 0
    xb, wq, s_w, bias, s_g = problem(72, (rows, cols, k), group, "bf16", "int8")
    y, f, xq = run_grouped(xb, s_g, wq, s_w, bias, group, "int8", "bf16", False)
    set_tuning(path="twopass")
    try:
        y2, f2, xq2 = run_grouped(xb, s_g, wq, s_w, bias, group, "int8", "bf16", False)
    finally:
        set_tuning()
    assert np.array_equal(f, f2) and np.array_equal(y, y2) and np.array_equal(xq, xq2)
