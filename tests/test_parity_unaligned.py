"""GPU parity of operands that start on any element: vectors whose packs begin
after a head of single elements, and matrices whose lines (an odd leading
dimension, a slice of a longer buffer) start anywhere in a 16-byte pack."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from tests.criteria import TOL, bitwise_equal, check_scalar, check_vector, cond_scale, plain_reduced
from tests.gpu_util import DT, guarded, host, mat, need_gpu, vec

pytestmark = pytest.mark.gpu

DTYPES = ["f64", "f32", "bf16"]


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()
    from paper_1409_0669_amd import ops
    ops.reset_config()
    ops.load_default_tuning()
    yield
    ops.reset_config()


# lengths around a head alone (a 128-byte line holds 16, 32 or 64 elements),
# a head and one pack, and several packs per thread; starts alike and unlike
@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("starts", [(1, 1, 1), (3, 5, 2), (7, 0, 1), (0, 1, 0)])
@pytest.mark.parametrize("n", [1, 13, 15, 31, 61, 64, 129, 70001])
def test_vectors_from_any_element(dtype, starts, n):
    from paper_1409_0669_amd import ops
    y, y64 = vec(n, dtype, 131, pad_front=starts[0])
    z, z64 = vec(n, dtype, 132, pad_front=starts[1])
    what = "%s n=%d starts=%s" % (dtype, n, starts)
    a, b = 0.75, -1.25
    x, guard = guarded(n, dtype, starts[2])
    ops.axpby(a, y, b, z, out=x)
    assert bitwise_equal(host(x), oracle.axpby(dtype, a, y64, b, z64)), what
    ops.copy(y, out=x)
    assert bitwise_equal(host(x), y64), what
    ops.scal_to(a, z, out=x)
    assert bitwise_equal(host(x), oracle.scal(dtype, a, z64)), what
    guard(what)
    r, guard_r = guarded(n, dtype, starts[2])
    r.copy_(z)
    x.copy_(y)
    rr = ops.cg_update(a, x, y, r, z)
    rref = oracle.axpby(dtype, -a, z64, 1.0, z64)
    assert bitwise_equal(host(x), oracle.axpby(dtype, a, y64, 1.0, y64)), what
    assert bitwise_equal(host(r), rref), what
    check_scalar(float(rr), oracle.dot(rref, rref), 0.0, TOL[dtype], what)
    guard(what)
    guard_r(what)
    for acc in ("plain", "compensated"):
        check_scalar(float(ops.dot(y, z, acc=acc)), oracle.dot(y64, z64),
                     cond_scale(dtype, acc, np.abs(y64 * z64).sum()), TOL[dtype], what)
        check_scalar(float(ops.nrm2(y, acc=acc)), oracle.nrm2(y64), 0.0, TOL[dtype], what)


# line lengths below, at and past one pack and one wave-wide tile, so that the
# last lane's pack is full, ragged or the only one; leading dimensions that
# shift every line
@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("trans", [0, 1])
@pytest.mark.parametrize("vec_width", [1, 4, 8])
@pytest.mark.parametrize("k", [1, 3, 7, 9, 255, 257, 515])
def test_gemv_lines_from_any_element(dtype, trans, vec_width, k):
    from paper_1409_0669_amd import _lib as L
    from paper_1409_0669_amd import ops
    m, start = 67, 3
    for op in (L.OP_GEMV_ROWS, L.OP_GEMV_COLS):
        ops.set_config(op, DT[dtype], -1, vec=vec_width)
    A, A64 = mat(m, k + start, dtype, 133, pad=k % 2)
    A, A64 = A[:, start:], np.ascontiguousarray(A64[:, start:])
    x, x64 = vec(m if trans else k, dtype, 134, pad_front=1)
    B = A64.T if trans else A64
    ref, scale = oracle.gemv(np.ascontiguousarray(B), x64), np.abs(B) @ np.abs(x64)
    for acc in ("plain", "compensated"):
        y, guard = guarded(len(ref), ops.default_out_dtype(DT[dtype]), 1)
        ops.gemv(A, x, trans=bool(trans), acc=acc, out=y)
        what = "%s trans=%d vec=%d k=%d %s" % (dtype, trans, vec_width, k, acc)
        check_vector(host(y), ref, scale, TOL[dtype], what, plain_f32=plain_reduced(dtype, acc))
        guard(what)
    if dtype != "bf16":  # the epilogue's inner product counts every column once
        w, w64 = vec(len(ref), dtype, 135)
        _, s = ops.gemv_dot(A, x, w=w, trans=bool(trans))
        check_scalar(float(s), float(w64 @ ref), 2 * float(np.abs(w64) @ scale), TOL[dtype], "dot " + what)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("k", [1, 7, 9, 257])
def test_rank_one_lines_from_any_element(dtype, k):
    from paper_1409_0669_amd import ops
    m, start = 37, 3
    u, u64 = vec(m, dtype, 136, pad_front=1)
    v, v64 = vec(k, dtype, 137, pad_front=2)
    buf = torch.full((m, k + start + 2), float("nan"), dtype=DT[dtype], device="cuda")
    ops.ger(u, v, buf[:, start:start + k])
    assert bitwise_equal(host(buf[:, start:start + k]), oracle.ger(dtype, u64, v64).reshape(m, k))
    assert bool(torch.isnan(buf[:, :start]).all()) and bool(torch.isnan(buf[:, start + k:]).all())
