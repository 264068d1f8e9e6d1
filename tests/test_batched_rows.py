"""Batched GEMV tiles at the edges of their row groups: row lengths around
whole packs and whole trips of 8 to 64 lanes, row counts around a wave's and a
work-group's rows, lines and x on any element, and entries outside a row (NaN)
that its last, overlapping pack must not add."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from tests.criteria import TOL, bitwise_equal, check_vector, plain_reduced
from tests.gpu_util import DT, guarded, host, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("acc", ["plain", "compensated"])
@pytest.mark.parametrize("packs,block", [(0, 0), (1, 64), (32, 512)])
def test_rows_at_the_edges(dtype, acc, packs, block):
    need_gpu()
    from paper_1409_0669_amd.batch import BatchPlan
    V = {"f64": 2, "f32": 4, "bf16": 8}[dtype]
    od = torch.float64 if dtype == "f64" else torch.float32
    g = torch.Generator().manual_seed(41)
    gemvs, checks = [], []
    lengths = sorted({max(1, k * V + d) for k in (1, 8, 9, 64, 128, 520) for d in (-1, 0, 1, V - 1)})
    for i, n in enumerate(lengths):
        m, pad, at = (1, 7, 8, 65, 257)[i % 5], (0, 1, 3, 8)[i % 4], i % (V + 1)
        buf = torch.full((at + m * (n + pad),), float("nan"), dtype=DT[dtype])
        A = buf[at:].view(m, n + pad)[:, :n]
        A.copy_(torch.rand(m, n, generator=g, dtype=torch.float64) - 0.5)
        xb = torch.full((at + n + V,), float("nan"), dtype=DT[dtype])
        xb[at:at + n] = (torch.rand(n, generator=g, dtype=torch.float64) - 0.5).to(DT[dtype])
        if m == 8:  # an infinity under the last pack, met by a zero: NaN in one row, infinite in the others
            A[:, n - 1] = 1.0
            A[3, n - 1] = 0.0
            xb[at + n - 1] = float("-inf")
        bufc, xc = buf.cuda(), xb.cuda()
        y, check = guarded(m, od)
        gemvs.append((bufc[at:].view(m, n + pad)[:, :n], xc[at:at + n], y))
        checks.append(check)
    BatchPlan(gemvs, [], acc=acc, packs=packs, block=block).run()
    torch.cuda.synchronize()
    for (A, x, y), n, check in zip(gemvs, lengths, checks):
        what = "%s %s n=%d m=%d" % (dtype, acc, n, A.shape[0])
        check(what)
        A64, x64 = host(A), host(x)
        with np.errstate(invalid="ignore"):
            ref, scale = oracle.gemv(A64, x64), np.abs(A64) @ np.abs(x64)
        got, fin = host(y), np.isfinite(ref)
        assert bitwise_equal(got[~fin], ref[~fin]), what
        check_vector(got[fin], ref[fin], scale[fin], TOL[dtype], what, plain_f32=plain_reduced(dtype, acc))
