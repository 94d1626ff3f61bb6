"""The fake-quant backward of small tensors (one workgroup, one to three vectors a thread) at its edges: whole and partial
vectors, a last element run, the first size that goes over several workgroups again."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_2512_14481_amd import binding as B
from paper_2512_14481_amd import workloads as wl
from tests.gpu_util import assert_same_values, dev_scalar, to_bits, to_dev

pytestmark = pytest.mark.gpu

THREAD_VECS = 8 * 1024                                  # elements of one vector a thread


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("n", [1, 7, 8, 9, THREAD_VECS - 1, THREAD_VECS, THREAD_VECS + 7, THREAD_VECS + 8, 2 * THREAD_VECS,
                               2 * THREAD_VECS + 9, 3 * THREAD_VECS - 8, 3 * THREAD_VECS + 7, 3 * THREAD_VECS + 8])
def test_small_backward(dtype, n):
    x = wl.random_bits(31, f"x{n}{dtype}", (1, n), dtype, gain=3.0)
    dy = wl.random_bits(31, f"dy{n}{dtype}", (1, n), dtype)
    s = np.float32(oracle.absmax_scale(x, 8, dtype) / 3)
    ref = oracle.fakequant_bwd(x, dy, s, 8, dtype)
    ws = B.new_workspace(B.sasq_fakequant_bwd_workspace(1, n))
    xd, g, sd = to_dev(x, dtype), to_dev(dy, dtype), dev_scalar(s)
    got = []
    for call in (lambda dx, ds: B.sasq_fakequant_bwd(xd, g, sd, dx, ds, ws, 8), lambda dx, ds: B.sasq_fakequant_bwd_static(xd, g, sd, dx, ds, 8)):
        guard = torch.full((n + 64,), 7.0, dtype=g.dtype, device="cuda")          # nothing past the end is written
        dx, ds = guard[:n].view(1, n), torch.full((1,), float("nan"), dtype=torch.float32, device="cuda")
        call(dx, ds)
        torch.cuda.synchronize()
        assert (guard[n:] == 7.0).all()
        assert_same_values(to_bits(dx), ref["dx"], dtype, "dx")
        # 8 terms are summed in fp32 (relative 8 * 2^-24 of their magnitudes), the rest in fp64, the result rounded once
        assert abs(ds.item() - ref["ds64"]) <= 1e-6 * ref["sum_abs"] + 1e-7 * abs(ref["ds64"])
        got.append(ds.item())
        call(None, ds)
        assert ds.item() == got[0]
    assert got[0] == got[1]
    B.sasq_fakequant_bwd(xd, g, sd, g, ds, ws, 8)                                  # in place
    assert_same_values(to_bits(g), ref["dx"], dtype, "dx over dy")
    assert ds.item() == got[0]
