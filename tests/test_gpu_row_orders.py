"""GPU parity of the few-row linears in both orders of loading operands that lie in rows (turned in LDS, and in the MFMA's order) on both
sides of the lines between them: row tiles of 16, 32 and 64, small blocks, narrow and wide workgroups, codes quantized in the kernel and
before it; the library's host functions say which form each call takes."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_2512_14481_amd import binding as B
from tests.dispatch import linear_quantizes, linear_streams, linear_takes_few_rows, linear_turns
from tests.gpu_util import assert_same_values, dev_scalar, set_tuning, to_bits, to_dev
from tests.test_gpu_grouped_linear import WF, device_weights
from tests.test_gpu_row_blocks import LAYOUTS, test_rows_quantized_in_the_kernel_match_oracle as check_quantized
from tests.test_gpu_row_turn import test_rows_turned_in_lds_match_oracle as check_turned
from tests.test_gpu_skinny_linear import problem

pytestmark = pytest.mark.gpu

# (rows, columns, K, quantized in the kernel, turned)
ROW_MAJOR = [(8, 1001, 448, True, False), (8, 1001, 512, True, True), (13, 300, 576, True, False), (13, 300, 704, True, True),
             (16, 8200, 320, True, False), (16, 8200, 384, True, True), (20, 4200, 448, True, False), (32, 4100, 1024, True, True),
             (20, 3000, 320, True, False), (20, 4200, 704, True, True), (40, 3000, 192, True, False), (64, 3000, 448, True, False),
             (64, 4200, 512, True, False), (40, 1000, 448, True, False), (30, 8200, 640, False, False), (30, 8200, 768, False, True),
             (30, 8191, 1728, False, False), (40, 8200, 1088, False, True), (60, 8190, 960, False, False), (60, 3000, 704, False, False),
             (40, 3000, 2112, False, True), (64, 2000, 1728, False, False), (64, 2000, 1856, False, True), (32, 16, 3136, False, True)]
BLOCKED8 = [(8, 1000, 960, True, False), (8, 1000, 1024, True, True), (16, 600, 1984, True, False), (16, 600, 2048, True, True),
            (7, 5000, 1088, True, True), (16, 5000, 128, True, False), (8, 8200, 256, True, False), (8, 8200, 320, True, False),
            (9, 8200, 2112, True, True), (40, 500, 448, True, False), (40, 500, 512, True, True), (64, 2000, 704, True, False),
            (64, 2000, 768, True, True), (32, 4200, 448, True, False), (32, 4200, 512, True, True)]
BLOCKED4 = [(8, 1000, 512, True, False), (8, 1000, 576, True, True), (16, 1000, 2112, True, False), (8, 8200, 192, True, False),
            (16, 8200, 448, True, False), (5, 8200, 2048, True, True), (40, 500, 448, True, False), (40, 500, 512, True, True),
            (64, 4000, 704, True, False), (64, 4000, 768, True, True)]
CASES = ([("int8", False) + c for c in ROW_MAJOR] + [("int8", True) + c for c in BLOCKED8] + [("int4", True) + c for c in BLOCKED4])


@pytest.mark.parametrize("fmt,blocked,M,N,K,quantizes,turns", CASES)
def test_both_orders_match_oracle(fmt, blocked, M, N, K, quantizes, turns):
    set_tuning()
    wf, dtype = WF[(fmt, blocked)], "bf16" if N % 2 else "f16"
    assert linear_takes_few_rows([(M, N, K)], wf)
    assert (linear_quantizes([(M, N, K)], wf), linear_turns([(M, N, K)], wf)) == (quantizes, turns)
    xb, wq, s_w, bias, s = problem(231, (M, N, K), fmt, dtype)
    ref = oracle.static_linear(xb, s, wq, s_w, bias, 8, fmt, dtype)
    x = to_dev(xb, dtype)
    y = torch.full((M, N), float("nan"), dtype=x.dtype, device="cuda")
    acc = torch.zeros((M, N), dtype=torch.int32, device="cuda")
    B.sasq_static_linear(x, dev_scalar(s), device_weights(wq, fmt, blocked), torch.from_numpy(s_w).cuda(), torch.from_numpy(bias).cuda(), y, wf,
                         B.new_workspace(B.sasq_static_linear_workspace(M, N, K, wf)), acc)
    assert np.array_equal(acc.cpu().numpy(), ref["acc"])
    assert_same_values(to_bits(y), ref["y"], dtype, "Y")


@pytest.mark.parametrize("rows,K,turns", [(32, 448, False), (32, 512, True), (64, 512, False)])
@pytest.mark.parametrize("fmt", ["int8", "int4"])
def test_batches_of_pre_arranged_row_tiles(fmt, rows, K, turns):
    """Three projections are more than a round of small blocks: row tiles of 32 and 64, quantized in the kernel."""
    set_tuning()
    wf, dims = WF[(fmt, True)], [2600, 2601, 2575]
    shapes = [(rows - i, n, K) for i, n in enumerate(dims)]
    assert linear_quantizes(shapes, wf) and linear_turns(shapes, wf) == turns
    items, refs = [], []
    for shape in shapes:
        xb, wq, s_w, _, s = problem(241, shape, fmt, "bf16")
        refs.append(oracle.static_linear(xb, s, wq, s_w, None, 8, fmt, "bf16")["y"])
        items.append((to_dev(xb, "bf16"), dev_scalar(s), device_weights(wq, fmt, True), torch.from_numpy(s_w).cuda(), None,
                      torch.full(shape[:2], float("nan"), dtype=torch.bfloat16, device="cuda")))
    B.sasq_static_linear_batch(items, wf, B.new_workspace(B.sasq_static_linear_batch_workspace(items, wf)))
    for it, ref in zip(items, refs):
        assert_same_values(to_bits(it[5]), ref, "bf16", "Y")


@pytest.mark.parametrize("shape,layouts", [
    ((5, 17001, 8064), (("int8", False),)),                                     # 137 MB of row-major weights, read past the caches
    ((20, 16999, 8064), (("int8", False),)),
    ((9, 9000, 11 * 64), (("int8", False),)),                                   # wide: a wave without a step, the third's last one half
    ((8, 8200, 13 * 64), (("int8", False),)),                                   # wide: the fourth wave's only step is half
    ((9, 9000, 33 * 64), (("int8", False), ("int8", True), ("int4", True))),
    ((40, 1000, 11 * 64), (("int8", False),)),                                  # a small block
    ((40, 3000, 33 * 64), (("int8", False),)),                                  # row tiles of 48, codes from the pre-pass
    ((33, 8200, 17 * 64), (("int8", False),))])                                 # the same, wide
def test_half_steps_of_turned_rows(shape, layouts):
    for fmt, blocked in layouts:
        wf = WF[(fmt, blocked)]
        assert linear_takes_few_rows([shape], wf) and linear_turns([shape], wf)
        assert linear_streams([shape], wf) == (blocked or shape[1] * shape[2] > 128 << 20)
    check_turned(shape, layouts)


@pytest.mark.parametrize("fmt,blocked", LAYOUTS)
@pytest.mark.parametrize("shape", [(32, 4200, 1024), (32, 4200, 1088), (64, 3000, 512), (64, 3000, 576), (64, 2000, 1024), (64, 2000, 1088)])
def test_row_tiles_at_the_longest_quantized_rows(shape, fmt, blocked):
    """Row tiles of 32 and 64 and small blocks, at and past the lengths up to which each workgroup quantizes for itself (rows times K of a row
    tile: 32768, the 4200 columns and row-major 3000; K of a small block of 32 rows: 1024, the 2000 columns)."""
    check_quantized(shape, fmt, blocked)
