"""The rows GEMV's shape rule: parity on both sides of its lines, and on the
CPU, that it stays within what the kernel and its grid take."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest
import torch

import oracle
from tests.criteria import TOL, check_scalar, check_vector, plain_reduced
from tests.gpu_util import DT, guarded, host, mat, need_gpu, vec

DTYPES = ["f64", "f32", "bf16"]


@pytest.fixture(autouse=True)
def _defaults():
    from paper_1409_0669_amd import ops
    ops.reset_config()
    yield
    ops.reset_config()


# few and many lines (one, two, four per work-group), lines of less than a pack, of
# one wave's packs and past them, many short lines
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("lines,k", [(3, 5), (399, 130), (400, 513), (2049, 70), (8193, 41), (7000, 3), (5, 40001)])
@pytest.mark.parametrize("start", [0, 1])
def test_rows_rule_parity(dtype, lines, k, start):
    need_gpu()
    from paper_1409_0669_amd import ops
    A, A64 = mat(lines, k + start, dtype, 161, pad=start)
    A, A64 = A[:, start:], np.ascontiguousarray(A64[:, start:])
    x, x64 = vec(k, dtype, 162, pad_front=start)
    ref, scale = oracle.gemv(A64, x64), np.abs(A64) @ np.abs(x64)
    for acc in ("plain", "compensated"):
        y, guard = guarded(lines, ops.default_out_dtype(DT[dtype]), start)
        ops.gemv(A, x, acc=acc, out=y)
        what = "%s %dx%d start=%d %s" % (dtype, lines, k, start, acc)
        check_vector(host(y), ref, scale, TOL[dtype], what, plain_f32=plain_reduced(dtype, acc))
        guard(what)
        if dtype != "bf16":
            w, w64 = vec(lines, dtype, 163)
            y2, s = ops.gemv_dot(A, x, w=w, acc=acc)
            assert torch.equal(y2, y), what
            check_scalar(float(s), float(w64 @ ref), 2 * float(np.abs(w64) @ scale), TOL[dtype], "dot " + what)


def test_rows_rule_limits():
    from paper_1409_0669_amd import _lib as L
    lib = L.lib
    c, b = L.Config(), ctypes.c_size_t()
    for t, size in ((0, 8), (1, 4), (2, 2)):
        for lines in (1, 399, 400, 2048, 2049, 8192, 16384, 1 << 20):
            for k in (1, 7, 64, 500, 5000, 16384, 30000, 1 << 20):
                assert lib.bwla_workspace_size(L.OP_GEMV_ROWS, t, 0, L.ROW_MAJOR, 0, lines, k, ctypes.byref(b)) == L.OK
                for acc in (0, 1):
                    assert lib.bwla_get_config(L.OP_GEMV_ROWS, t, acc, lines, k, ctypes.byref(c)) == L.OK
                    assert 64 <= c.block <= 1024 and c.block % 64 == 0 and c.unroll in (1, 2)
                    assert c.vec == 16 // size and c.rows in (1, 2, 4)
                    groups = -(-lines // c.rows)
                    assert c.grid == min(groups * c.split, (1 << 31) - 1)
                    assert c.split == 1 or b.value >= groups * c.split * c.rows * 16
                    if 512 <= lines and lines * k * size < 1 << 28:
                        assert c.split == 1
