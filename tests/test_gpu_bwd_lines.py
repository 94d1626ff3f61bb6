"""GPU parity of the backward GEMM around the ends of its pipeline against the CPU oracle: contractions of a few K tiles of 32, even and
odd, which read dY in half lines, and the first ones that read it in whole cache lines on each tile; ragged rows and columns; both tiles that can
be forced.  Bounds as for the other tiles: fp32 sums in any order, one rounding."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2512_14481_amd import workloads as wl
from tests.dispatch import bwd_reads_lines
from tests.test_gpu_linear_bwd import check_dx, prepare, problem, run_bwd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("tile", ["256", "128"])
@pytest.mark.parametrize("ktiles", [2, 4, 6, 8, 9, 10, 12, 14, 16, 17, 18, 26])
def test_contractions_around_the_pipeline(ktiles, tile, dtype):
    shape = (261, 32 * ktiles, 274)
    dyb, wq, s_w = problem(85, shape, dtype, "int8")
    wt, K = prepare(wq, s_w, "int8", dtype)
    ref = oracle.linear_bwd_input(dyb, wq, s_w, "int8", dtype)
    got, acc = run_bwd(dyb, wt, K, dtype, tile, want_acc=True)
    check_dx(got, ref, dtype, shape[1], f"{shape} {dtype} tile {tile}")
    err = np.abs(acc.astype(np.float64) - ref["exact"])
    assert (err <= shape[1] * 2.0 ** -24 * ref["sum_abs"] + 1e-45).all(), err.max()
    assert np.array_equal(got, wl.f32_to_storage_bits(acc, dtype))


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("tile,ktiles", [(t, k) for t, first in (("128", 32), ("256", 64)) for k in (first - 2, first, first + 1, first + 2, first + 4, first + 6)])
def test_first_contractions_in_whole_lines(ktiles, tile, dtype):
    assert bwd_reads_lines(32 * ktiles, int(tile)) == (ktiles % 2 == 0 and ktiles >= (64 if tile == "256" else 32))
    test_contractions_around_the_pipeline(ktiles, tile, dtype)
