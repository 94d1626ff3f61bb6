"""GPU parity of the linear's row blocks (more than 64 rows in small blocks of 16 or 32 rows, or 64, 96 or 128 by 64, K over eight waves)
against the CPU oracle: each block form and weight layout, alone and in batches, with waves that have no K tile at all (K = 64),
uneven shares of them, and rows and columns that end inside a block."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_2512_14481_amd import binding as B
from tests.dispatch import linear_block_rows
from tests.gpu_util import assert_same_values, dev_scalar, set_tuning, to_bits, to_dev
from tests.test_gpu_grouped_linear import WF, device_weights
from tests.test_gpu_skinny_linear import LAYOUTS, problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt,blocked", LAYOUTS)
@pytest.mark.parametrize("items,want", [
    ([(65, 1000, 64)], (32, 32, 32)),                                           # 32 x 32: 96 blocks, waves without a K tile
    ([(130, 1003, 704)], (32, 32, 32)),
    ([(130, 100, 576)], (32, 32, 32)),                                          # 16 x 16, quantized in the kernel
    ([(130, 100, 3136)], (32, 32, 32)),                                         # and before it
    ([(300, 250, 1024)], (32, 32, 32)),                                         # 32 x 16, quantized in the kernel
    ([(1024, 256, 576)], (32, 32, 32)),                                         # exactly 256
    ([(500, 700, 576)], (32, 32, 32)),                                          # 384, so 32 x 64
    ([(70, 5120, 640)], (32, 32, 32)),                                          # 240 of 32 x 64
    ([(96, 1000, 1088), (70, 1201, 192), (20, 500, 64)], (32, 32, 32)),
    ([(70, 5121, 64)], (64, 64, 64)),
    ([(190, 2900, 704)], (64, 64, 64)),
    ([(383, 4090, 192)], (96, 0, 96)),
    ([(1500, 1000, 576)], (96, 96, 96)),
    ([(500, 4090, 1088)], (128, 128, 64)),
    ([(500, 4090, 192)], (0, 0, 64)),
    ([(250, 5000, 576)], (96, 96, 96)),
    ([(250, 6000, 2112)], (128, 128, 128)),
    ([(100, 5500, 2112), (80, 5600, 2112)], (128, 128, 128)),
    ([(96, 5000, 1088), (70, 8201, 192), (96, 6000, 64)], (64, 64, 64)),
    ([(96, 9000, 1088), (70, 8201, 192)], (64, 0, 64)),
    ([(96, 4000, 1088), (70, 4201, 192)], (96, 96, 96)),                       # all rows in one block: weights read once
    ([(400, 2000, 64), (400, 3001, 64)], (0, 0, 0)),
    ([(128, 9001, 2112), (100, 8200, 2112)], (0, 0, 64)),
    ([(128, 4001, 1024), (100, 4200, 1024)], (128, 128, 64)),                 # the same at 128 rows
    ([(300, 2000, 1088), (257, 3001, 576)], (64, 64, 64))])
def test_row_blocks_match_oracle(items, want, fmt, blocked):
    set_tuning()
    assert linear_block_rows(items, WF[(fmt, blocked)]) == want[LAYOUTS.index((fmt, blocked))]
    batch, refs = [], []
    for i, (m, n, k) in enumerate(items):
        xb, wq, s_w, bias, s = problem(101 + i, (m, n, k), fmt, "bf16")
        b = bias if i == len(items) - 1 else None
        refs.append(oracle.static_linear(xb, s, wq, s_w, b, 8, fmt, "bf16"))
        batch.append((to_dev(xb, "bf16"), dev_scalar(s), device_weights(wq, fmt, blocked), torch.from_numpy(s_w).cuda(),
                      None if b is None else torch.from_numpy(b).cuda(), torch.full((m, n), float("nan"), dtype=torch.bfloat16, device="cuda")))
    wf = WF[(fmt, blocked)]
    if len(items) == 1:
        x, s, w, s_w, b, y = batch[0]
        acc = torch.zeros(y.shape, dtype=torch.int32, device="cuda")
        B.sasq_static_linear(x, s, w, s_w, b, y, wf, B.new_workspace(B.sasq_static_linear_workspace(*y.shape, x.shape[1], wf)), acc, None)
        assert np.array_equal(acc.cpu().numpy(), refs[0]["acc"])
    else:
        B.sasq_static_linear_batch(batch, wf, B.new_workspace(B.sasq_static_linear_batch_workspace(batch, wf)))
    for it, ref in zip(batch, refs):
        assert_same_values(to_bits(it[5]), ref["y"], "bf16", "Y")


@pytest.mark.parametrize("fmt,blocked", LAYOUTS)
@pytest.mark.parametrize("shape", [(17, 47, 64), (32, 700, 1024), (32, 700, 1088), (33, 701, 512), (64, 700, 512), (64, 700, 576), (20, 8200, 192)])
def test_rows_quantized_in_the_kernel_match_oracle(shape, fmt, blocked):
    """17 to 64 rows around the line up to which each workgroup quantizes for itself (rows in tiles of 32 or 64, times K: 32768)."""
    set_tuning()
    M, N, K = shape
    xb, wq, s_w, bias, s = problem(110, shape, fmt, "f16")
    ref = oracle.static_linear(xb, s, wq, s_w, bias, 8, fmt, "f16")
    wf = WF[(fmt, blocked)]
    y, acc = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda"), torch.zeros((M, N), dtype=torch.int32, device="cuda")
    B.sasq_static_linear(to_dev(xb, "f16"), dev_scalar(s), device_weights(wq, fmt, blocked), torch.from_numpy(s_w).cuda(),
                         torch.from_numpy(bias).cuda(), y, wf, B.new_workspace(B.sasq_static_linear_workspace(M, N, K, wf)), acc, None)
    assert np.array_equal(acc.cpu().numpy(), ref["acc"])
    assert_same_values(to_bits(y), ref["y"], "f16", "Y")


def test_output_over_input_at_thirty_rows():
    set_tuning()
    shape = (30, 1024, 1024)
    xb, wq, s_w, _, s = problem(111, shape, "int8", "f16")
    ref = oracle.static_linear(xb, s, wq, s_w, None, 8, "int8", "f16")
    x = to_dev(xb, "f16")
    B.sasq_static_linear(x, dev_scalar(s), device_weights(wq, "int8", True), torch.from_numpy(s_w).cuda(), None, x, B.SASQ_W_INT8_BLOCKED,
                         B.new_workspace(B.sasq_static_linear_workspace(*shape, B.SASQ_W_INT8_BLOCKED)))
    assert_same_values(to_bits(x), ref["y"], "f16", "Y")
