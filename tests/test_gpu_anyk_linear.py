"""GPU parity of the linear for contraction lengths that are not multiples of 64 against the CPU oracle: accumulators bit for
bit, Y equal by value, at the edges of its 128-channel stages, of 16-code pieces and rows shorter than one, of its tiles, with
rows at every alignment; one factor per tensor and one per row."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_2512_14481_amd import binding as B
from tests.gpu_util import TDT, assert_same_values, dev_scalar, set_tuning, to_bits, to_dev
from tests.test_gpu_dynamic_linear import run_dynamic
from tests.test_gpu_grouped_linear import WF
from tests.test_gpu_skinny_linear import problem

pytestmark = pytest.mark.gpu

KS = [1, 2, 7, 15, 16, 18, 31, 63, 65, 100, 127, 129, 130, 136, 144, 250, 255, 257, 400, 526, 1376]
ROWS_COLS = [(1, 1), (33, 47), (64, 64), (65, 130), (127, 129)]
WIDE = [((1920, 2050), 130), ((2049, 1925), 81), ((1, 4099), 1030)]      # enough tiles of every shape the dispatch chooses from


@pytest.mark.parametrize("fmt", ["int8", "int4"])
@pytest.mark.parametrize("mn,k", [(mn, k) for k in KS for mn in ROWS_COLS] + WIDE)
def test_any_contraction_length(mn, k, fmt):
    if fmt == "int4" and k % 2:
        pytest.skip("packed int4 rows hold whole bytes")
    set_tuning()
    (M, N), dtype = mn, "bf16" if k % 3 else "f16"
    xb, wq, s_w, bias, s = problem(91, (M, N, k), fmt, dtype)
    wf, wd, swd = WF[(fmt, False)], torch.from_numpy(wq).cuda(), torch.from_numpy(s_w).cuda()
    x, b = to_dev(xb, dtype), bias if N % 2 else None
    ws = B.new_workspace(B.sasq_static_linear_workspace(M, N, k, wf))
    ref = oracle.static_linear(xb, s, wq, s_w, b, 8, fmt, dtype)
    y = torch.full((M, N), float("nan"), dtype=TDT[dtype], device="cuda")
    acc = torch.zeros((M, N), dtype=torch.int32, device="cuda")
    bd = None if b is None else torch.from_numpy(b).cuda()
    B.sasq_static_linear(x, dev_scalar(s), wd, swd, bd, y, wf, ws, acc, None)
    assert np.array_equal(acc.cpu().numpy(), ref["acc"])
    assert_same_values(to_bits(y), ref["y"], dtype, "Y")
    ref = oracle.dynamic_linear(xb, wq, s_w, b, 8, fmt, dtype)
    yd, accd, _, _ = run_dynamic(xb, wq, s_w, b, fmt, dtype, False)
    assert np.array_equal(accd, ref["acc"])
    assert_same_values(yd, ref["y"], dtype, "Y, one factor per row")
