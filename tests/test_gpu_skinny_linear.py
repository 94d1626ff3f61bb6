"""GPU parity of the few-row linear kernels (M <= 64, and row blocks of 64, 96 and 128) against the CPU oracle: accumulators bit for bit, Y equal by value, for
every weight layout that reaches them, at the edges of their row tiles (16, 32, 48, 64), of the split of K over the waves
(fewer K tiles than waves, remainders), of the column tiles and of the narrow / wide choice; mixed batches; in-place calls."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_2512_14481_amd import binding as B
from paper_2512_14481_amd import workloads as wl
from tests.gpu_util import TDT, assert_same_values, dev_scalar, set_tuning, to_bits, to_dev
from tests.test_gpu_grouped_linear import WF, device_weights

pytestmark = pytest.mark.gpu

LAYOUTS = [("int8", False), ("int8", True), ("int4", True)]
SHAPES = [(1, 1, 64), (3, 47, 576), (15, 130, 128), (16, 512, 1088), (17, 33, 64), (32, 96, 704), (33, 72, 2112), (48, 250, 640),
          (49, 31, 192), (64, 264, 1024), (65, 64, 128), (16, 8200, 192), (2, 8185, 320), (30, 8192, 128), (64, 8189, 192),
          # more than 64 rows: small blocks, row blocks of 64 (int4) and 96, the GEMM's tiles
          (333, 1000, 704), (227, 5504, 128), (270, 4090, 128), (450, 4090, 128), (300, 3500, 192), (96, 16500, 64), (97, 9001, 128), (128, 8200, 320)]


def problem(seed, shape, fmt, dtype):
    M, N, K = shape
    xb = wl.random_bits(seed, f"sx{shape}{dtype}", (M, K), dtype, gain=2.0)
    wq, s_w = oracle.quantize_weight(wl.random_f32(seed, f"sw{shape}", (N, K), 0.02), fmt)
    return xb, wq, s_w, wl.random_f32(seed, f"sb{shape}", (N,), 0.3), np.float32(oracle.absmax_scale(xb, 8, dtype) * 0.4)


@pytest.mark.parametrize("fmt,blocked", LAYOUTS)
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_few_rows_match_oracle(shape, dtype, fmt, blocked):
    set_tuning()
    M, N, K = shape
    xb, wq, s_w, bias, s = problem(61, shape, fmt, dtype)
    wf, wd, swd = WF[(fmt, blocked)], device_weights(wq, fmt, blocked), torch.from_numpy(s_w).cuda()
    x = to_dev(xb, dtype)
    ws = B.new_workspace(B.sasq_static_linear_workspace(M, N, K, wf))
    for b in (None, bias):
        ref = oracle.static_linear(xb, s, wq, s_w, b, 8, fmt, dtype)
        y = torch.full((M, N), float("nan"), dtype=TDT[dtype], device="cuda")
        acc = torch.zeros((M, N), dtype=torch.int32, device="cuda")
        bd = None if b is None else torch.from_numpy(b).cuda()
        B.sasq_static_linear(x, dev_scalar(s), wd, swd, bd, y, wf, ws, acc, None)
        assert np.array_equal(acc.cpu().numpy(), ref["acc"])
        assert_same_values(to_bits(y), ref["y"], dtype, "Y")
        y2 = torch.full_like(y, float("nan"))
        B.sasq_static_linear(x, dev_scalar(s), wd, swd, bd, y2, wf, ws)
        assert np.array_equal(to_bits(y2), to_bits(y))


@pytest.mark.parametrize("rows", [(5, 16, 1), (9, 64, 20), (70, 3, 129)])
@pytest.mark.parametrize("fmt,blocked", LAYOUTS)
def test_batch_of_few_rows_matches_oracle(rows, fmt, blocked):
    set_tuning()
    dims = [(96, 640), (300, 64), (41, 1984)] if max(rows) <= 64 else [(520, 640), (600, 64), (513, 1984)]
    items, refs = [], []
    for i, (m, (n, k)) in enumerate(zip(rows, dims)):
        xb, wq, s_w, bias, s = problem(70 + i, (m, n, k), fmt, "bf16")
        b = bias if i == 1 else None
        refs.append(oracle.static_linear(xb, s, wq, s_w, b, 8, fmt, "bf16")["y"])
        items.append((to_dev(xb, "bf16"), dev_scalar(s), device_weights(wq, fmt, blocked), torch.from_numpy(s_w).cuda(),
                      None if b is None else torch.from_numpy(b).cuda(), torch.empty((m, n), dtype=torch.bfloat16, device="cuda")))
    wf = WF[(fmt, blocked)]
    B.sasq_static_linear_batch(items, wf, B.new_workspace(B.sasq_static_linear_batch_workspace(items, wf)))
    for it, ref in zip(items, refs):
        assert_same_values(to_bits(it[5]), ref, "bf16", "Y")


def test_output_over_input_at_few_rows():
    """An output that is the input's own buffer: the activations are quantized before the first output is written."""
    set_tuning()
    shape = (8, 2048, 2048)
    xb, wq, s_w, _, s = problem(80, shape, "int8", "f16")
    ref = oracle.static_linear(xb, s, wq, s_w, None, 8, "int8", "f16")
    wd, x = device_weights(wq, "int8", True), to_dev(xb, "f16")
    ws = B.new_workspace(B.sasq_static_linear_workspace(*shape, B.SASQ_W_INT8_BLOCKED))
    B.sasq_static_linear(x, dev_scalar(s), wd, torch.from_numpy(s_w).cuda(), None, x, B.SASQ_W_INT8_BLOCKED, ws)
    assert_same_values(to_bits(x), ref["y"], "f16", "Y")


def chosen_rows(rows, dims, fmt):
    """Rows per block for a batch of at most 128 and more than 64 rows (0: the GEMM's tiles) by rounds alone.  What the library takes:
    tests/test_few_rows_dispatch.py."""
    cols = [-(-n // 64) for n, _ in dims]
    if min(cols) < 8:
        return 0
    for block in (64, 96):
        if sum(-(-m // block) * c for m, c in zip(rows, cols)) <= 256:
            return block
    tiles, work, k_max = 0, 0, max(k for _, k in dims)
    for n, k in dims:
        tiles, work = tiles + -(-n // 256), work + -(-n // 256) * k
    fill = work / (256 * max(k_max, -(-tiles // 256) * work / tiles))
    if max(rows) <= 96:
        line = 0.5 if k_max < 2048 else 0.7 if tiles > 256 else 0.8 if fmt == "int4" else 0.5
        return 96 if fill <= line else 0
    return 0 if fill > 0.5 or (fmt != "int4" and k_max < 2048 and tiles > 64) else 128


@pytest.mark.parametrize("rows,dims,want", [
    ((96, 70), [(8200, 128), (8501, 192)], {"int8": 96, "int4": 96}),
    ((66, 80, 96), [(6000, 128), (6500, 64), (5111, 192)], {"int8": 96, "int4": 96}),
    ((97, 66), [(8200, 128), (8501, 192)], {"int8": 0, "int4": 128}),
    ((100, 128), [(8200, 2048), (8501, 2112)], {"int8": 128, "int4": 128}),
    ((70, 96), [(17000, 128), (17000, 128)], {"int8": 0, "int4": 0}),          # 134 tiles, more than half of a round
    ((90, 65), [(20000, 2048), (20000, 2048)], {"int8": 0, "int4": 96})])
@pytest.mark.parametrize("fmt,blocked", LAYOUTS)
def test_batch_of_row_blocks_matches_oracle(rows, dims, want, fmt, blocked):
    """Batches with all rows in one block of 96 or 128, unequal M and ragged N, and their neighbours on the GEMM's tiles."""
    set_tuning()
    assert chosen_rows(rows, dims, fmt) == want[fmt]
    items, refs = [], []
    for i, (m, (n, k)) in enumerate(zip(rows, dims)):
        xb, wq, s_w, bias, s = problem(90 + i, (m, n, k), fmt, "f16")
        b = bias if i == 1 else None
        refs.append(oracle.static_linear(xb, s, wq, s_w, b, 8, fmt, "f16")["y"])
        items.append((to_dev(xb, "f16"), dev_scalar(s), device_weights(wq, fmt, blocked), torch.from_numpy(s_w).cuda(),
                      None if b is None else torch.from_numpy(b).cuda(), torch.full((m, n), float("nan"), dtype=torch.float16, device="cuda")))
    wf = WF[(fmt, blocked)]
    B.sasq_static_linear_batch(items, wf, B.new_workspace(B.sasq_static_linear_batch_workspace(items, wf)))
    for it, ref in zip(items, refs):
        assert_same_values(to_bits(it[5]), ref, "f16", "Y")


@pytest.mark.parametrize("fmt,blocked", LAYOUTS)
@pytest.mark.parametrize("shape", [(64, 32768, 64), (49, 32769, 64), (48, 52480, 64), (33, 52481, 64), (64, 66000, 64), (64, 93000, 64)])
def test_few_rows_many_columns(shape, fmt, blocked):
    """Both sides of the lines between the few-row kernels and the GEMM's tiles (half a round, four fifths, a second round)."""
    set_tuning()
    M, N, K = shape
    xb, wq, s_w, bias, s = problem(95, shape, fmt, "bf16")
    ref = oracle.static_linear(xb, s, wq, s_w, bias, 8, fmt, "bf16")
    y = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    wf = WF[(fmt, blocked)]
    B.sasq_static_linear(to_dev(xb, "bf16"), dev_scalar(s), device_weights(wq, fmt, blocked), torch.from_numpy(s_w).cuda(),
                         torch.from_numpy(bias).cuda(), y, wf, B.new_workspace(B.sasq_static_linear_workspace(M, N, K, wf)))
    assert_same_values(to_bits(y), ref["y"], "bf16", "Y")
