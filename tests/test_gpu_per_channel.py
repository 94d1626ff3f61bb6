"""GPU parity of the per-channel fake-quant operator against the CPU oracle."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_2512_14481_amd import binding as B
from paper_2512_14481_amd import workloads as wl
from tests.gpu_util import assert_same_values, to_bits, to_dev

pytestmark = pytest.mark.gpu


def col_absmax_scales(xb, dtype, div=1.0):
    v = np.abs(wl.storage_bits_to_f32(xb, dtype)).max(axis=0)
    return (np.maximum(v, np.float32(1e-3)) / np.float32(127.0 * div)).astype(np.float32)


def run_pc(xb, dyb, s, dtype, bits=8, want_dx=True):
    x, dy = to_dev(xb, dtype), to_dev(dyb, dtype)
    sd = torch.from_numpy(s).cuda()
    y = torch.empty_like(x)
    codes = torch.empty(x.shape, dtype=torch.int8, device="cuda")
    B.sasq_fakequant_fwd_pc(x, sd, y, codes, bits)
    y2 = torch.empty_like(x)
    B.sasq_fakequant_fwd_pc(x, sd, y2, None, bits)
    rows, cols = xb.shape
    ws = B.new_workspace(B.sasq_fakequant_bwd_pc_workspace(rows, cols))
    dx = torch.empty_like(x) if want_dx else None
    ds = torch.full((cols,), 777.0, dtype=torch.float32, device="cuda")
    B.sasq_fakequant_bwd_pc(x, dy, sd, dx, ds, ws, bits)
    ds_b = torch.zeros(cols, dtype=torch.float32, device="cuda")
    B.sasq_fakequant_bwd_pc(x, dy, sd, dx, ds_b, ws, bits)          # same workspace again: tickets were reset
    torch.cuda.synchronize()
    assert torch.equal(y.view(torch.int16), y2.view(torch.int16))
    assert torch.equal(ds.view(torch.int32), ds_b.view(torch.int32)), "per-channel ds is reproducible"
    return to_bits(y), codes.cpu().numpy(), (to_bits(dx) if want_dx else None), ds.cpu().numpy()


def check(xb, dyb, s, dtype, bits=8):
    y, codes, dx, ds = run_pc(xb, dyb, s, dtype, bits)
    y_ref, c_ref = oracle.fakequant_fwd_pc(xb, s, bits, dtype)
    assert np.array_equal(codes, c_ref), "codes"
    assert_same_values(y, y_ref, dtype, "y")
    ref = oracle.fakequant_bwd_pc(xb, dyb, s, bits, dtype)
    assert_same_values(dx, ref["dx"], dtype, "dx")
    err = np.abs(ds.astype(np.float64) - ref["ds64"])
    assert (err <= 1e-4 * np.abs(ref["ds64"]) + 1e-6 * ref["sum_abs"]).all(), (err.max(), np.abs(ref["ds64"]).min())
    tight = np.abs(ref["ds64"]) > 1e-3 * ref["sum_abs"]            # well-conditioned columns: the plain 1e-4 bar
    assert (err[tight] <= 1e-4 * np.abs(ref["ds64"][tight])).all()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("shape", [(1, 8), (5, 16), (33, 512), (64, 256), (257, 1032), (100, 4096),
                                   (7, 13), (40, 1001), (1, 1)])
def test_per_channel_shapes(shape, dtype):
    xb = wl.random_bits(41, f"pcx{shape}{dtype}", shape, dtype, gain=2.5)
    dyb = wl.random_bits(41, f"pcg{shape}{dtype}", shape, dtype)
    for div in (1.0, 4.0):
        s = col_absmax_scales(xb, dtype, div)
        if shape[1] > 2:
            s[1] = -s[1]
        check(xb, dyb, s, dtype)
    check(xb, dyb, col_absmax_scales(xb, dtype, 0.06), dtype, bits=4)


@pytest.mark.parametrize("cfg_name,act_name", [("c1_single", "x"), ("c3_mlp7b", "x_mlp"), ("c3_mlp7b", "x_down"),
                                               ("c4_w4a8_13b", "x_down")])
def test_per_channel_full_size(cfg_name, act_name):
    cfg = wl.CONFIGS[cfg_name]
    xb = wl.activation(cfg, act_name)
    proj = next(p for p in cfg.projs if p.x == act_name)
    dyb = wl.upstream_grad(cfg, proj.name)
    check(xb, dyb, col_absmax_scales(xb, cfg.dtype, 4.0), cfg.dtype)


def test_pc_backward_workspace_reuse_with_different_data():
    """A second call on the same workspace with other data must not see the first call's partials."""
    dtype = "f16"
    shape = (700, 1032)
    ws = B.new_workspace(B.sasq_fakequant_bwd_pc_workspace(*shape))
    s = (np.abs(wl.random_f32(77, "rs", (shape[1],), 0.02)) + np.float32(0.004)).astype(np.float32)
    sd = torch.from_numpy(s).cuda()
    for rep in range(3):
        xb = wl.random_bits(77 + rep, f"rx{rep}", shape, dtype, gain=2.0)
        dyb = wl.random_bits(77 + rep, f"rd{rep}", shape, dtype, gain=1.0 + rep)
        ds = torch.empty(shape[1], dtype=torch.float32, device="cuda")
        B.sasq_fakequant_bwd_pc(to_dev(xb, dtype), to_dev(dyb, dtype), sd, None, ds, ws, 8)
        torch.cuda.synchronize()
        ref = oracle.fakequant_bwd_pc(xb, dyb, s, 8, dtype)
        err = np.abs(ds.cpu().numpy().astype(np.float64) - ref["ds64"])
        assert (err <= 1e-4 * np.abs(ref["ds64"]) + 1e-6 * ref["sum_abs"]).all(), rep


@pytest.mark.parametrize("rows", [15, 16, 31, 32, 33, 47, 63, 64, 65, 129, 2049])
def test_per_channel_row_chunks(rows):
    """Rows around the group of 16, the chunk of 32 and the cap on chunks.  Bound: four rows are summed in fp32 (a product, a
    subtraction and three additions each rounded once), a partial and the result rounded once: 8 2^-24 of the sum of absolute
    terms."""
    dtype, shape = "bf16", (rows, 520)
    xb, dyb = wl.random_bits(43, f"rcx{rows}", shape, dtype, gain=2.5), wl.random_bits(43, f"rcg{rows}", shape, dtype)
    s = col_absmax_scales(xb, dtype, 2.0)
    check(xb, dyb, s, dtype)
    ref = oracle.fakequant_bwd_pc(xb, dyb, s, 8, dtype)
    _, _, _, ds = run_pc(xb, dyb, s, dtype, want_dx=False)
    assert (np.abs(ds - ref["ds64"]) <= 8 * 2.0 ** -24 * ref["sum_abs"]).all()


def test_per_channel_batch_with_long_chunks():
    """A batch large enough for chunks of 64 rows."""
    dtype, shape = "f16", (2113, 4096)
    xb, dyb = wl.random_bits(44, "lcx", shape, dtype, gain=2.5), wl.random_bits(44, "lcg", shape, dtype)
    s = col_absmax_scales(xb, dtype, 2.0)
    ref = oracle.fakequant_bwd_pc(xb, dyb, s, 8, dtype)
    x, dy, sd = to_dev(xb, dtype), to_dev(dyb, dtype), torch.from_numpy(s).cuda()
    items = [(x, dy, sd, torch.empty_like(x), torch.empty_like(sd)) for _ in range(8)]
    B.sasq_fakequant_bwd_pc_batch(items, B.new_workspace(B.sasq_fakequant_bwd_pc_batch_workspace(items)))
    for _, _, _, dx, ds in items:
        assert torch.equal(dx, items[0][3]) and torch.equal(ds, items[0][4])
    assert_same_values(to_bits(items[0][3]), ref["dx"], dtype, "dx")
    assert (np.abs(items[0][4].cpu().numpy() - ref["ds64"]) <= 8 * 2.0 ** -24 * ref["sum_abs"]).all()


# rows per block of 16, 32 and 64 in the backward, at the edges of the rule; launches of few and of thousands of blocks
BATCHES = [[(2113, 4096)] * 8, [(128, 4096), (129, 4096), (1024, 512), (1025, 512), (3, 8)], [(4096, 4096), (4160, 4096), (64, 264), (700, 2048)],
           [(1600, 5120), (1664, 5120), (640, 13824), (704, 13824)], [(128, 4096), (3, 8), (512, 512)]]


@pytest.mark.parametrize("shapes", BATCHES, ids=["many_blocks", "short", "long", "wide", "all_short"])
def test_per_channel_batch_equals_single_calls(shapes):
    """An item's ds (and dx) has the bits of the single-tensor call whatever else is in the launch."""
    g = torch.Generator(device="cuda").manual_seed(45)
    distinct = {}
    for sh in shapes:
        if sh not in distinct:
            x, dy = ((torch.randn(sh, device="cuda", generator=g) * k).half() for k in (2.0, 1.0))
            s = torch.rand(sh[1], device="cuda", generator=g) * 0.05 + 0.01
            dx, ds = torch.empty_like(x), torch.empty_like(s)
            B.sasq_fakequant_bwd_pc(x, dy, s, dx, ds, B.new_workspace(B.sasq_fakequant_bwd_pc_workspace(*sh)))
            distinct[sh] = (x, dy, s, dx, ds)
    items = [(x, dy, s, torch.empty_like(dx), torch.empty_like(ds)) for x, dy, s, dx, ds in (distinct[sh] for sh in shapes)]
    B.sasq_fakequant_bwd_pc_batch(items, B.new_workspace(B.sasq_fakequant_bwd_pc_batch_workspace(items)))
    for sh, (_, _, _, dx, ds) in zip(shapes, items):
        assert torch.equal(ds, distinct[sh][4]), sh
        assert torch.equal(dx, distinct[sh][3]), sh


@pytest.mark.parametrize("rows", [31, 511, 512, 513, 769, 785, 1024, 1025])
def test_per_channel_forward_rows_per_block(rows):
    """Launches around the lines of the forward's rule (256, 384 and 512 blocks of 16 rows x 512 columns): every row comes out
    as in a call on a few rows alone."""
    g = torch.Generator(device="cuda").manual_seed(46)
    x = (torch.randn((rows, 4096), device="cuda", generator=g) * 2).bfloat16()
    s = torch.rand(4096, device="cuda", generator=g) * 0.05 + 0.01
    y, want = torch.empty_like(x), torch.empty_like(x)
    B.sasq_fakequant_fwd_pc(x, s, y)
    for r in range(0, rows, 100):
        B.sasq_fakequant_fwd_pc(x[r:r + 100], s, want[r:r + 100])
    assert torch.equal(y, want)
    y2 = [torch.full_like(x, float("nan")) for _ in range(2)]
    B.sasq_fakequant_fwd_pc_batch([(x, s, t) for t in y2])
    assert all(torch.equal(t, want) for t in y2)
