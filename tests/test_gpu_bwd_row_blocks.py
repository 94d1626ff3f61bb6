"""GPU parity of the backward linear's kernels for few rows and row blocks (contraction split over the waves, no tiles) against the CPU
oracle: the row-tile forms (16, 32, 64 rows; narrow and wide), small blocks, blocks of 64 and 96 rows, waves without a contraction tile, ragged
rows and columns.  Bounds as for the tiled kernels: fp32 sums in any order, one rounding."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2512_14481_amd import workloads as wl
from tests.dispatch import bwd_rows, bwd_tile
from tests.test_gpu_linear_bwd import check_dx, prepare, problem, run_bwd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("shape,want", [
    ((1, 32, 2), 64), ((16, 576, 4096), 64), ((15, 96, 4104), 64), ((32, 1088, 5001), 64), ((64, 2048, 8300), 64), ((50, 1024, 9003), 64), ((40, 32, 20000), 0),
    ((17, 64, 70), 32), ((33, 96, 48), 32), ((64, 576, 1024), 32), ((130, 160, 130), 32),                                 # 16 x 16
    ((32, 1088, 4090), 32), ((33, 96, 1300), 32), ((300, 320, 256), 32),                                                  # 32 x 16
    ((64, 1056, 4096), 32), ((64, 2048, 4200), 32), ((50, 1024, 5003), 32),
    ((65, 32, 2), 32), ((65, 1024, 1000), 32), ((130, 1024, 520), 32), ((129, 1600, 449), 32), ((1024, 96, 256), 32),    # 32 x 32
    ((500, 288, 700), 32), ((70, 1056, 5120), 32), ((222, 544, 1530), 32),                                                # 32 x 64
    ((70, 1056, 5121), 64), ((300, 1024, 1700), 64), ((500, 4096, 2000), 64), ((1000, 1024, 520), 0), ((2000, 1024, 448), 0), ((198, 64, 1984), 0),
    ((18, 544, 27456), 0), ((53, 160, 16392), 0), ((380, 4096, 4000), 0),
    ((130, 4096, 7500), 96)])
def test_few_rows_and_row_blocks_match_oracle(shape, want, dtype):
    assert bwd_rows(*shape) == want
    dyb, wq, s_w = problem(83, shape, dtype, "int8")
    wt, K = prepare(wq, s_w, "int8", dtype)
    ref = oracle.linear_bwd_input(dyb, wq, s_w, "int8", dtype)
    got, acc = run_bwd(dyb, wt, K, dtype, want_acc=True)
    check_dx(got, ref, dtype, shape[1], f"{shape} {dtype}")
    err = np.abs(acc.astype(np.float64) - ref["exact"])
    assert (err <= shape[1] * 2.0 ** -24 * ref["sum_abs"] + 1e-45).all(), err.max()
    assert np.array_equal(got, wl.f32_to_storage_bits(acc, dtype))
    assert np.array_equal(run_bwd(dyb, wt, K, dtype), got)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("shape", [(1830, 1024, 3330), (1793, 1056, 3329), (2048, 1024, 3200)])
def test_tiles_of_128_by_256(shape, dtype):
    """390 to 512 tiles of 128x128: they go as 128x256, ragged and whole; the 256x256 tiles sum in the same order."""
    M, N, K = shape
    assert bwd_rows(*shape) == 0 and bwd_tile(*shape) == (128, 256)
    dyb, wq, s_w = problem(84, shape, dtype, "int8")
    wt, K = prepare(wq, s_w, "int8", dtype)
    ref = oracle.linear_bwd_input(dyb, wq, s_w, "int8", dtype)
    got, acc = run_bwd(dyb, wt, K, dtype, want_acc=True)
    check_dx(got, ref, dtype, N, f"{shape} {dtype}")
    assert np.array_equal(got, wl.f32_to_storage_bits(acc, dtype))
    assert np.array_equal(run_bwd(dyb, wt, K, dtype, tile="256"), got)
