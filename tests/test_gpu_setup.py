"""GPU parity of the set-up kernels at the edges of their forms: weight quantization by whole 128-bit pieces (K % 4 == 0, up to
256 in one wave, up to 32768) and by the general kernel, the prepared backward weight at ragged sizes and alignments, absmax around its load batches."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_2512_14481_amd import binding as B
from paper_2512_14481_amd import workloads as wl
from tests.gpu_util import to_dev
from tests.test_gpu_linear_bwd import prepare, unblock

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", ["int8", "int4"])
@pytest.mark.parametrize("k", [2, 4, 6, 60, 252, 256, 260, 1020, 1024, 1028, 5120, 8188, 8192, 8196, 11008, 13824, 28672, 32768, 32772])
def test_quantize_weight_rows(k, fmt):
    n = 5
    w = wl.random_f32(31, f"qw{k}", (n, k), 0.02)
    w[1] = 0.0
    w[2, -1] = -3.0                                        # the largest value in the row's last place, and in its first
    w[3, 0] = 3.0
    w[4, k // 2] = np.nan                                  # ignored by the maximum, quantized like the general kernel does
    wq = torch.empty((n, k // 2 if fmt == "int4" else k), dtype=torch.uint8 if fmt == "int4" else torch.int8, device="cuda")
    s_w = torch.empty(n, dtype=torch.float32, device="cuda")
    B.sasq_quantize_weight(torch.from_numpy(w).cuda(), wq, s_w, B.SASQ_W_INT4_PACKED if fmt == "int4" else B.SASQ_W_INT8)
    ref, ref_s = oracle.quantize_weight(np.nan_to_num(w, nan=0.0), fmt)
    assert np.array_equal(s_w.cpu().numpy(), ref_s)
    got, skip = wq.cpu().numpy().view(np.uint8), k // 2 // (2 if fmt == "int4" else 1)
    keep = np.ones(got.shape, bool)
    keep[4, skip] = False
    assert np.array_equal(got[keep], ref.view(np.uint8)[keep])


@pytest.mark.parametrize("fmt,dtype", [("int8", "f16"), ("int4", "bf16")])
@pytest.mark.parametrize("shape", [(1, 2), (31, 14), (32, 16), (33, 18), (64, 510), (40, 512), (65, 514), (7, 1376), (96, 1030),
                                   (33, 126), (17, 128), (65, 130), (20, 258), (900, 4626), (913, 4608)])      # widths of 128 codes, and of 512 (from 256 of those)
def test_prepared_weight(shape, fmt, dtype):
    N, K = shape
    wq, s_w = oracle.quantize_weight(wl.random_f32(33, f"pw{shape}", shape, 0.02), fmt)
    s_w[0] = -s_w[0]                                       # padding stays +0 under any factor
    wt, _ = prepare(wq, s_w, fmt, dtype)
    codes = wq.astype(np.float32) if fmt == "int8" else (((np.stack([wq & 15, wq >> 4], -1).reshape(N, K).astype(np.int32)) ^ 8) - 8).astype(np.float32)
    full = unblock(wt.cpu().numpy(), N, K)
    want = np.zeros(full.shape, np.uint16)
    want[:K, :N] = oracle.encode16((codes * s_w[:, None]).T.astype(np.float32), dtype)
    assert np.array_equal(full, want)


@pytest.mark.parametrize("k", [15, 17, 513])
def test_prepared_weight_odd_rows(k):
    wq, s_w = oracle.quantize_weight(wl.random_f32(35, f"ow{k}", (37, k), 0.02), "int8")
    wt, _ = prepare(wq, s_w, "int8", "f16")
    want = oracle.encode16((wq.astype(np.float32) * s_w[:, None]).T.astype(np.float32), "f16")
    assert np.array_equal(unblock(wt.cpu().numpy(), 37, k)[:k, :37], want)


@pytest.mark.parametrize("n", [1, 7, 8, 9, 8 * 256 * 8 - 8, 8 * 256 * 8 + 11, 8 * 256 * 8 * 600 + 3,
                               8 * 1024 + 9, 8 * 1024 * 128, 8 * 1024 * 128 + 7, 8 * 1024 * 128 + 8])      # one pass of up to 128 blocks, and past it
def test_absmax_sizes(n):
    xb = wl.random_bits(37, f"am{n}", (1, n), "bf16", gain=1.0)
    for at in {0, n - 1, n // 2}:
        b = xb.copy()
        b[0, at] = 0xC2F7                                  # -123.5
        s = torch.zeros(1, dtype=torch.float32, device="cuda")
        B.sasq_absmax_scale(to_dev(b, "bf16"), s, B.new_workspace(B.sasq_absmax_scale_workspace(1, n)))
        assert np.float32(s.item()) == oracle.absmax_scale(b, 8, "bf16")
