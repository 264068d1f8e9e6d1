"""Compensated bf16 reductions are float64 sums of exact products: sums that
cancel to far below their terms, and terms outside the range of float32."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def _bf16(values):
    return torch.tensor(values, dtype=torch.float64).to(torch.bfloat16).cuda()


# the products below are multiples of 1 whose partial sums, in any order, stay below
# 2^8 2^15 2^10 200002 < 2^51: exact in
# float64, so the results are exact whatever the reduction's shape
@pytest.mark.parametrize("n", [8, 1000, 100001])
def test_cancelling_sums_are_exact(n):
    from paper_1409_0669_amd import ops
    rng = np.random.default_rng(7)
    half = rng.integers(-255, 256, n).astype(np.float64) * 2.0 ** rng.integers(0, 16, n)
    x = np.concatenate([half, half[::-1], [1.0]])
    y = np.concatenate([np.full(n, 2.0 ** 10), np.full(n, -2.0 ** 10), [1.0]])
    xt, yt = _bf16(x), _bf16(y)
    assert float(ops.dot(xt, yt, acc="compensated", out_dtype=torch.float64)) == 1.0
    A = torch.stack([xt, yt, xt]).contiguous()
    want = [1.0, float((y * y).sum()), 1.0]
    got = ops.gemv(A, yt, acc="compensated", out_dtype=torch.float64)
    assert got.tolist() == want
    got = ops.gemv(A.t().contiguous(), yt, trans=True, acc="compensated", out_dtype=torch.float64)
    assert got.tolist() == want
    out = torch.empty(1, dtype=torch.float64, device="cuda")
    rows = torch.empty(3, dtype=torch.float64, device="cuda")
    from paper_1409_0669_amd.batch import BatchPlan
    BatchPlan([(A, yt, rows)], [(xt, yt, out)], acc="compensated", out_dtype=torch.float64).run()
    assert out.item() == want[0] and rows.tolist() == want


def test_terms_outside_float32():
    from paper_1409_0669_amd import ops
    x, y = _bf16([2.0 ** 100, 2.0 ** -100, 1.0]), _bf16([2.0 ** 100, 2.0 ** -100, 0.0])
    assert float(ops.dot(x, y, acc="compensated", out_dtype=torch.float64)) == 2.0 ** 200
    z = _bf16([2.0 ** -100] * 3)
    assert float(ops.dot(z, z, acc="compensated", out_dtype=torch.float64)) == 3 * 2.0 ** -200
    inf = _bf16([float("inf"), 1.0, 0.0])
    assert float(ops.dot(inf, x, acc="compensated")) == float("inf")
    assert np.isnan(float(ops.dot(inf, _bf16([0.0, 1.0, 1.0]), acc="compensated")))
