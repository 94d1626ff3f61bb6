"""GPU parity of the backward linear's few-row, small-block and row-block kernels in both orders of loading dY (turned in LDS, and in the
MFMA's order) on both sides of the lines between them; the library's host functions say which form each call takes."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2512_14481_amd import workloads as wl
from tests.dispatch import bwd_rows, bwd_turns
from tests.gpu_util import set_tuning
from tests.test_gpu_linear_bwd import check_dx, prepare, problem, run_bwd

pytestmark = pytest.mark.gpu

# (rows, contraction tiles of 32, output columns, turned)
CASES = [(5, 66, 1001, False), (7, 33, 4200, False), (12, 8, 1000, False), (12, 10, 1001, True), (16, 63, 300, False), (16, 65, 300, True),
         (13, 62, 4500, False), (13, 64, 4500, True), (40, 6, 500, False), (40, 8, 501, True), (64, 31, 1500, False), (64, 33, 1500, True),
         (100, 12, 4000, False), (100, 14, 4001, True), (30, 14, 6000, False), (30, 16, 6000, True), (30, 65, 4500, False), (50, 32, 8300, True),
         (50, 30, 8300, False), (130, 65, 2900, True), (200, 31, 4000, False), (200, 33, 4000, True)]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("M,ktiles,K,turns", CASES)
def test_both_orders_match_oracle(M, ktiles, K, turns, dtype):
    set_tuning()
    shape = (M, 32 * ktiles, K)
    assert bwd_rows(*shape) and bwd_turns(*shape) == turns
    dyb, wq, s_w = problem(87, shape, dtype, "int8")
    wt, _ = prepare(wq, s_w, "int8", dtype)
    ref = oracle.linear_bwd_input(dyb, wq, s_w, "int8", dtype)
    got, acc = run_bwd(dyb, wt, K, dtype, want_acc=True)
    check_dx(got, ref, dtype, shape[1], f"{shape} {dtype}")
    err = np.abs(acc.astype(np.float64) - ref["exact"])
    assert (err <= shape[1] * 2.0 ** -24 * ref["sum_abs"] + 1e-45).all(), err.max()
    assert np.array_equal(got, wl.f32_to_storage_bits(acc, dtype))
