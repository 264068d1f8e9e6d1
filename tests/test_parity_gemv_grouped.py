"""GPU parity of the cols GEMV with several lines per wave access: every width,
with the trips, the last lane's pack, the split and the line combine at their
edges, and the library's own choice over shapes; and the sizing of that choice
on the CPU."""
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


def _check(dtype, lines, k, start, what):
    """A row-major matrix of `lines` lines of k entries, transposed product."""
    from paper_1409_0669_amd import ops
    A, A64 = mat(lines, k + start, dtype, 141, pad=3 if start else 0)
    A, A64 = A[:, start:], np.ascontiguousarray(A64[:, start:])
    x, x64 = vec(lines, dtype, 142, pad_front=start)
    ref, scale = oracle.gemv(np.ascontiguousarray(A64.T), x64), np.abs(A64.T) @ np.abs(x64)
    for acc in ("plain", "compensated"):
        y, guard = guarded(k, ops.default_out_dtype(DT[dtype]), start)
        ops.gemv(A, x, trans=True, acc=acc, out=y)
        check_vector(host(y), ref, scale, TOL[dtype], "%s %s" % (what, acc), plain_f32=plain_reduced(dtype, acc))
        guard(what)
        if dtype != "bf16":
            w, w64 = vec(k, dtype, 143)
            y2, s = ops.gemv_dot(A, x, w=w, trans=True, acc=acc)
            assert torch.equal(y2, y), what
            check_scalar(float(s), float(w64 @ ref), 2 * float(np.abs(w64) @ scale), TOL[dtype], "dot " + what)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("rows,unroll,block", [(2, 8, 256), (4, 4, 512), (8, 4, 64), (8, 8, 1024)])
@pytest.mark.parametrize("split", [1, 2, 9])  # no combine, one thread per output, several
@pytest.mark.parametrize("lines,k", [(1, 8), (7, 9), (64, 131), (257, 64), (1025, 33)])
def test_grouped_edges(dtype, rows, unroll, block, split, lines, k):
    need_gpu()
    from paper_1409_0669_amd import _lib as L
    from paper_1409_0669_amd import ops
    vec_width = 16 // torch.empty(0, dtype=DT[dtype]).element_size()
    ops.set_config(L.OP_GEMV_COLS, DT[dtype], -1, block=block, vec=vec_width, unroll=unroll, rows=rows, split=split)
    assert ops.get_config(L.OP_GEMV_COLS, DT[dtype], lines, k)["rows"] == rows
    for start in (0, 1):
        _check(dtype, lines, k, start, "%s rows=%d split=%d %dx%d start=%d" % (dtype, rows, split, lines, k, start))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("lines,k", [(2, 3), (64, 64), (1024, 600), (1025, 600), (5000, 37), (70, 5000), (2300, 1111)])
def test_shape_rule(dtype, lines, k):
    need_gpu()
    for start in (0, 1):
        _check(dtype, lines, k, start, "%s %dx%d start=%d" % (dtype, lines, k, start))


def test_rule_fills_the_chip_and_is_sized():
    """The shape rule on the CPU: one launch for few lines, enough
    work-groups for many, and a workspace that covers lines on and off a
    cache line and both accumulation modes."""
    from paper_1409_0669_amd import _lib as L
    lib = L.lib
    c, b = L.Config(), ctypes.c_size_t()
    for t, size in ((0, 8), (1, 4), (2, 2)):
        for lines in (1, 500, 1024, 4096, 16000, 100000):
            for k in (1, 7, 100, 1500, 4096, 20001):
                assert lib.bwla_workspace_size(L.OP_GEMV_COLS, t, 0, L.ROW_MAJOR, 1, lines, k, ctypes.byref(b)) == L.OK
                for acc in (0, 1):
                    assert lib.bwla_get_config(L.OP_GEMV_COLS, t, acc, lines, k, ctypes.byref(c)) == L.OK
                    tile = 64 // c.rows * c.vec
                    tiles = -(-k // tile)
                    assert c.split >= 1 and c.grid == tiles * c.split
                    assert c.split == 1 or lines // c.split >= 16
                    if c.split > 1:
                        assert b.value >= tiles * c.split * tile * 16
                    if lines * k * size > 1 << 24 and k >= 16:
                        assert c.grid >= 100, (t, lines, k, c.as_dict())
    assert lib.bwla_get_config(L.OP_GEMV_COLS, 1, 0, 300, 300, ctypes.byref(c)) == L.OK
    assert (c.split, c.rows, c.vec) == (1, 8, 4)
