"""GPU tests of calls whose workgroups hold 2^32 threads and more, which one launch cannot: they go in parts, or to the kernel
that needs fewer.  The references are torch on the same card (integer sums, one rounding each) and the same entry point on slices."""
from __future__ import annotations

import pytest
import torch

from paper_2512_14481_amd import binding as B

pytestmark = pytest.mark.gpu


def need(gib):
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < gib << 30:
        pytest.skip(f"needs {gib} GiB of device memory")


def row_problem(n, k):
    g = torch.Generator("cuda").manual_seed(71)
    x = torch.linspace(-1.0, 0.9, k, device="cuda").half().reshape(1, k)
    wq = torch.empty((n, k), dtype=torch.int8, device="cuda").random_(-128, 128, generator=g)
    s_w = torch.empty(n, device="cuda").uniform_(0.5e-3, 2e-3, generator=g)
    return x, wq, s_w, torch.empty((1, n), dtype=torch.float16, device="cuda"), torch.full((1,), 0.01, device="cuda")


def check_row(y, xq, wq, s_w, s, grouped):
    n, step = y.shape[1], 1 << 24
    for a in range(0, n, step):
        acc = (wq[a:a + step].float() * xq[0].float()).sum(1)                      # below 2^24: exact
        sw = s_w[a:a + step]
        assert torch.equal(y[0, a:a + step], ((acc * s) * sw if grouped else acc * (s * sw)).half()), a


@pytest.mark.parametrize("group", [1, 2, 3])               # single channels, sums on the matrix units, sums on the VALUs
def test_grouped_one_row_by_two_to_the_thirty_columns(group):
    need(32)
    n = (1 << 30) + 5
    x, wq, s_w, y, s = row_problem(n, group)
    ws = B.new_workspace(B.sasq_static_linear_workspace(1, n, group, B.SASQ_W_INT8))
    xq = torch.empty((1, group), dtype=torch.int8, device="cuda")
    B.sasq_static_linear_grouped(x, s, wq, s_w, None, y, group, B.SASQ_W_INT8, ws, xq_out=xq)
    check_row(y, xq, wq, s_w, s, True)


@pytest.mark.parametrize("n,k,gib", [((1 << 31) - 1, 3, 48), ((1 << 29) + 7, 64, 80)])      # any K; whole K tiles, few rows
def test_linear_one_row_by_very_many_columns(n, k, gib):
    need(gib)
    x, wq, s_w, y, s = row_problem(n, k)
    ws = B.new_workspace(B.sasq_static_linear_workspace(1, n, k, B.SASQ_W_INT8))
    xq = torch.empty((1, k), dtype=torch.int8, device="cuda")
    B.sasq_static_linear(x, s, wq, s_w, None, y, B.SASQ_W_INT8, ws, None, xq)
    check_row(y, xq, wq, s_w, s, False)


def test_prepared_weight_of_two_to_the_twentynine_rows():
    need(48)
    n, step = 1 << 29, 1 << 20
    _, wq, s_w, _, _ = row_problem(n, 1)
    block = 32 * 16 * 2                                    # bytes of 32 rows of one code

    def prepare(a, b):
        wt = torch.empty(B.sasq_bwd_weight_bytes(b - a, 1), dtype=torch.uint8, device="cuda")
        B.sasq_prepare_bwd_weight(wq[a:b], s_w[a:b], wt, b - a, 1, B.SASQ_W_INT8, torch.float16)
        return wt

    whole = prepare(0, n)
    for a in (0, (1 << 28) - step // 2, n - step):
        assert torch.equal(whole[a // 32 * block:(a + step) // 32 * block], prepare(a, a + step)), a


def test_quantize_weight_of_two_to_the_twentytwo_long_rows():
    need(200)
    n, k = 1 << 22, 8196
    w = torch.zeros((n, k), device="cuda")
    for r in (0, n // 2, n - 1):
        w[r] = torch.linspace(-0.5, 0.4 + 1e-7 * r, k, device="cuda")
    wq = torch.empty((n, k), dtype=torch.int8, device="cuda")
    s_w = torch.empty(n, device="cuda")
    B.sasq_quantize_weight(w, wq, s_w, B.SASQ_W_INT8)
    for a in (0, n // 2 - 1, n - 3):
        q, s = torch.empty_like(wq[:3]), torch.empty_like(s_w[:3])
        B.sasq_quantize_weight(w[a:a + 3].clone(), q, s, B.SASQ_W_INT8)
        assert torch.equal(wq[a:a + 3], q) and torch.equal(s_w[a:a + 3], s), a
    assert int((s_w != s_w[1]).sum()) == 3
