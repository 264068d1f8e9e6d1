"""Tall matrices: the rows GEMV's work-groups fit short lines and a launch's
thread count, and products of more than 2^24 lines are exact on whole
numbers."""
from __future__ import annotations

import ctypes

import pytest
import torch

from tests.gpu_util import DT, guarded, need_gpu

SIZES = {"f64": 8, "f32": 4, "bf16": 2}


@pytest.fixture(autouse=True)
def _defaults():
    from paper_1409_0669_amd import ops
    ops.reset_config()
    yield
    ops.reset_config()


def test_work_groups_fit_the_lines_and_the_launch():
    from paper_1409_0669_amd import _lib as L
    c = L.Config()
    for t, size in enumerate(SIZES.values()):
        for lines in [(1 << e) + d for e in (12, 18, 20, 21, 23, 24, 25, 26, 27, 28) for d in (-1, 0, 1)] + [20_000_000]:
            for k in (1, 2, 4, 7, 8, 13, 64, 100, 300, 1000, 1500, 5000, 30000):
                if lines * k * size > 1 << 38:
                    continue
                for acc in (0, 1):
                    assert L.lib.bwla_get_config(L.OP_GEMV_ROWS, t, acc, lines, k, ctypes.byref(c)) == L.OK
                    what = (t, acc, lines, k, c.block, c.rows, c.split)
                    packs = max(1, k // (16 // size))
                    slice_packs = -(-packs // c.split)
                    assert c.block <= -(-slice_packs // 64) * 64, what
                    assert -(-lines // c.rows) * c.split * c.block < 1 << 32, what
                    if lines * k * size >= 1 << 28 and packs <= 192:
                        assert c.rows >= 4, what


def test_more_threads_than_a_launch_holds_are_refused():
    from paper_1409_0669_amd import _lib as L
    A, x, y = 1 << 40, 1 << 44, 1 << 45
    b = ctypes.c_size_t()
    assert L.lib.bwla_gemv(1, 0, 0, 0, 1 << 32, 1, A, 1, x, 1, y, None, 0, None) == L.ERR_UNSUPPORTED
    assert L.lib.bwla_gemv_ex_workspace_size(1, 1, 0, 0, 1 << 32, 1, ctypes.byref(b)) == L.OK
    assert L.lib.bwla_gemv_ex(1, 0, 0, 0, 1 << 32, 1, 2.0, A, 1, x, 1, 0.0, 1, y, 1, 1 << 50, b.value,
                              None) == L.ERR_UNSUPPORTED


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,lines,k", [("bf16", 1 << 24, 8), ("f64", (1 << 24) + 3, 2), ("f32", 1 << 24, 5),
                                           ("f64", 1 << 20, 64), ("f32", (1 << 20) + 1, 65), ("bf16", 1 << 18, 513)])
def test_tall_products_are_exact(dtype, lines, k):
    need_gpu()
    from paper_1409_0669_amd import ops
    g = torch.Generator(device="cuda").manual_seed(51)
    A = torch.randint(-3, 4, (lines, k), generator=g, device="cuda", dtype=torch.int8).to(DT[dtype])
    x = torch.randint(-3, 4, (k,), generator=g, device="cuda").to(DT[dtype])
    ref = torch.zeros(lines, dtype=torch.float64, device="cuda")
    for j in range(k):
        ref.add_(A[:, j].double(), alpha=float(x[j]))
    for acc in ("plain", "compensated"):
        y, guard = guarded(lines, ops.default_out_dtype(DT[dtype]))
        ops.gemv(A, x, acc=acc, out=y)
        assert torch.equal(y.double(), ref), (dtype, lines, k, acc)
        guard()
