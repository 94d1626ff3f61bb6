"""GPU parity of the few-row linears whose operands lie in rows and turn into the MFMA's order in LDS: the forms that the other tests'
sizes do not reach (long rows, weights beyond the cached size), half steps of two K tiles in every wave's place, up to eight rows and more."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_2512_14481_amd import binding as B
from tests.gpu_util import assert_same_values, dev_scalar, set_tuning, to_bits, to_dev
from tests.test_gpu_grouped_linear import WF, device_weights
from tests.test_gpu_skinny_linear import problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,layouts", [
    ((8, 8190, 8256), (("int8", True),)),                                     # wide, six K tiles in flight
    ((5, 17001, 8000), (("int8", False),)),                                     # 136 MB of row-major weights
    ((20, 16999, 8000), (("int8", False),)),
    ((9, 9000, 192), (("int8", False), ("int8", True), ("int4", True))),        # more waves than steps, one of them half
    ((7, 100, 1024 + 64), (("int8", False), ("int8", True), ("int4", True))),   # narrow, the last wave's only step is half
    ((8, 8200, 7 * 64), (("int8", False),)),                                    # wide: four waves, the last step half
    ((40, 1000, 9 * 64), (("int8", False),))])
def test_rows_turned_in_lds_match_oracle(shape, layouts):
    set_tuning()
    M, N, K = shape
    for fmt, blocked in layouts:
        xb, wq, s_w, bias, s = problem(211, shape, fmt, "bf16")
        wf = WF[(fmt, blocked)]
        ref = oracle.static_linear(xb, s, wq, s_w, bias, 8, fmt, "bf16")
        y = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
        acc = torch.zeros((M, N), dtype=torch.int32, device="cuda")
        B.sasq_static_linear(to_dev(xb, "bf16"), dev_scalar(s), device_weights(wq, fmt, blocked), torch.from_numpy(s_w).cuda(),
                             torch.from_numpy(bias).cuda(), y, wf, B.new_workspace(B.sasq_static_linear_workspace(M, N, K, wf)), acc, None)
        assert np.array_equal(acc.cpu().numpy(), ref["acc"])
        assert_same_values(to_bits(y), ref["y"], "bf16", "Y")
