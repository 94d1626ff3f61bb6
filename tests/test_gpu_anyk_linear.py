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
WIDE = [((1920, 2050), 130), ((2049, 1925), 81), ((1, 4099), 1030)]      # tiles of 128x128 and 64x128, and one row
TILES = {(128, 128): (2817, 3001), (64, 128): (1000, 2050), (64, 64): (1100, 1500), (32, 64): (333, 700)}


def chosen(m, n, k, fmt):
    """The tile of four waves by their number, or None for one thread per output.  Which tile the library takes, and with how many waves:
    tests/test_gpu_anyk_choice.py."""
    wlen = k // 2 if fmt == "int4" else k
    if wlen <= 20 and m * n * wlen <= 3 << 19:
        return None
    for (bm, bn), least in (((128, 128), 512), ((64, 128), 256), ((64, 64), 256)):
        if -(-m // bm) * -(-n // bn) >= least:
            return bm, bn
    return 32, 64


@pytest.mark.parametrize("fmt", ["int8", "int4"])
@pytest.mark.parametrize("k", [81, 130, 400, 650])
@pytest.mark.parametrize("tile", TILES)
def test_every_tile(tile, k, fmt):
    """Row, column and K remainders on each tile: one stage of 128 channels, several, and part of one over."""
    assert chosen(*TILES[tile], k, fmt) == tile
    if tile == (128, 128) and k == 650:
        pytest.skip("the other lengths cover this tile's ring of two")
    test_any_contraction_length(TILES[tile], k, fmt)


@pytest.mark.parametrize("fmt", ["int8", "int4"])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 7, 8, 9, 12, 13, 15, 16, 17, 18, 20, 21, 22, 40, 42])
def test_short_rows(k, fmt):
    """Rows shorter than a 16-byte piece, on the tiles and with a thread per output, on both sides of the line between them."""
    if fmt == "int4" and k % 2:
        pytest.skip("packed int4 rows hold whole bytes")
    assert chosen(1100, 1500, k, fmt) == (64, 64)
    assert chosen(64, 999, k, fmt) == (None if (k // 2 if fmt == "int4" else k) <= 20 else (32, 64))
    for mn in ((1100, 1500), (64, 999), (1, 20001)):
        test_any_contraction_length(mn, k, fmt)


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


FEW_K = [65, 79, 100, 127, 200, 333, 516, 1000, 1031, 2095, 2108]
FEW_ROWS = [(1, 1), (15, 130), (16, 250), (17, 33), (32, 96), (33, 72), (48, 250), (49, 31), (64, 264)]
FEW_ROWS_WIDE = [(1, 8200), (16, 8195), (32, 8200), (64, 8189)]             # wide workgroups


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("mn,k", [(mn, k) for k in FEW_K for mn in FEW_ROWS] + [(mn, k) for k in (79, 200, 1031) for mn in FEW_ROWS_WIDE])
def test_few_rows(mn, k, dtype):
    """At most 64 rows: K over the waves, whole K tiles and the rest of a row; quantized in the kernel (at most 16 rows, or few codes)
    and before it; the tiled kernel, asked for by a knob, gives the same."""
    (M, N) = mn
    xb, wq, s_w, bias, s = problem(92, (M, N, k), "int8", dtype)
    wd, swd, x, bd = torch.from_numpy(wq).cuda(), torch.from_numpy(s_w).cuda(), to_dev(xb, dtype), torch.from_numpy(bias).cuda()
    ws = B.new_workspace(B.sasq_static_linear_workspace(M, N, k, B.SASQ_W_INT8))
    ref = oracle.static_linear(xb, s, wq, s_w, bias, 8, "int8", dtype)
    for path in (None, "twopass"):
        set_tuning(path=path)
        y = torch.full((M, N), float("nan"), dtype=TDT[dtype], device="cuda")
        acc = torch.zeros((M, N), dtype=torch.int32, device="cuda")
        B.sasq_static_linear(x, dev_scalar(s), wd, swd, bd, y, B.SASQ_W_INT8, ws, acc, None)
        set_tuning()
        assert np.array_equal(acc.cpu().numpy(), ref["acc"]), path
        assert_same_values(to_bits(y), ref["y"], dtype, "Y")
