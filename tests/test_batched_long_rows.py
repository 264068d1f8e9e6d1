"""Batched GEMVs with rows that a work-group shares: lengths around the start
of that form, around its changes of rows per work-group, around whole packs
and trips; row counts around its rows; rows on any element; x and A followed by
NaN.  Whole-number sums, exact in every order, and the accuracy of plain sums."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from tests.criteria import TOL, check_vector, plain_reduced
from tests.gpu_util import DT, guarded, host, need_gpu

pytestmark = pytest.mark.gpu


def _rows(m, n, pad, at, dtype, fill):
    buf = torch.full((at + m * (n + pad),), float("nan"), dtype=DT[dtype], device="cuda")
    A = buf[at:].view(m, n + pad)[:, :n]
    A.copy_(fill(m, n))
    return A


@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("acc", ["plain", "compensated"])
@pytest.mark.parametrize("block", [64, 256, 512])
def test_long_rows_are_exact(dtype, acc, block):
    need_gpu()
    from paper_1409_0669_amd.batch import BatchPlan
    g = torch.Generator(device="cuda").manual_seed(67)
    draw = lambda *s: torch.randint(-1, 2, s, generator=g, device="cuda", dtype=torch.int8).to(DT[dtype])
    od = torch.float64 if dtype == "f64" else torch.float32
    gemvs, checks = [], []
    for i, n in enumerate((2816, 2817, 4096, 4097, 4103, 8191, 8192, 8193, 16387, 32768, 32769, 100001, 1 << 20)):
        m, pad, at = (1, 3, 4, 7, 8, 9, 17)[i % 7], (0, 1, 3, 8)[i % 4], i % 9
        y, check = guarded(m, od)
        gemvs.append((_rows(m, n, pad, at, dtype, draw), _rows(1, n, 5, 8 - at, dtype, draw)[0], y))
        checks.append(check)
    plan = BatchPlan(gemvs, [(gemvs[0][1], gemvs[1][1][1:], torch.empty(1, dtype=od, device="cuda"))], acc=acc,
                     block=block)
    stream = torch.cuda.Stream()
    for replay in range(3):
        torch.cuda.synchronize()
        for _, _, y in gemvs:
            y.fill_(float("nan"))
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            if replay == 1:
                plan.capture()
            plan.run() if replay == 0 else plan.replay()
        torch.cuda.synchronize()
        for (A, x, y), check in zip(gemvs, checks):
            assert torch.equal(y.double(), (A.double() * x.double()).sum(1)), (A.shape, replay)
            check(str(A.shape))
    plan.close()


@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
def test_long_rows_and_non_finite_entries(dtype):
    need_gpu()
    from paper_1409_0669_amd.batch import BatchPlan
    g = torch.Generator(device="cuda").manual_seed(68)
    od = torch.float64 if dtype == "f64" else torch.float32
    for acc in ("plain", "compensated"):
        gemvs = []
        for n in (5003, 20001, 40002):
            fill = lambda *s: (torch.rand(s, generator=g, device="cuda", dtype=torch.float64) - 0.5).to(DT[dtype])
            A, x = _rows(11, n, 2, 1, dtype, fill), _rows(1, n, 0, 0, dtype, fill)[0]
            A[2, n - 1], A[5, 17] = float("inf"), float("nan")
            gemvs.append((A, x, torch.empty(11, dtype=od, device="cuda")))
        BatchPlan(gemvs, [], acc=acc).run()
        torch.cuda.synchronize()
        for A, x, y in gemvs:
            A64, x64, got = host(A), host(x), host(y)
            with np.errstate(invalid="ignore"):
                ref, scale = oracle.gemv(A64, x64), np.abs(A64) @ np.abs(x64)
            assert got[2] == ref[2] and np.isinf(ref[2]) and np.isnan(got[5])
            fin = np.isfinite(ref)
            assert fin.sum() == 9
            check_vector(got[fin], ref[fin], scale[fin], TOL[dtype], "%s %s %s" % (dtype, acc, A.shape),
                         plain_f32=plain_reduced(dtype, acc))


def test_long_rows_make_enough_work_groups():
    need_gpu()
    from paper_1409_0669_amd.batch import BatchPlan
    for n, rows in ((3000, 21), (8192, 8), (20000, 4), (100000, 1)):
        A, x, y = torch.zeros(64, n, device="cuda"), torch.zeros(n, device="cuda"), torch.zeros(64, device="cuda")
        assert BatchPlan([(A, x, y)], []).info()["items"] >= 64 // rows, n
