"""The alpha/beta product stores y in the kernel that would store the GEMV's
results: bitwise the composite (the GEMV, then the update of y) on every
store path, with increments of both signs, x repeated (increment 0), entries
of y between the increments untouched, and infinite and NaN results."""
from __future__ import annotations

import ctypes

import pytest
import torch

from tests.criteria import bitwise_equal
from tests.gpu_util import DT, host, mat, need_gpu, vec

pytestmark = pytest.mark.gpu

DTYPES = ["f64", "f32", "bf16"]
# (trans, configuration): rows and cols kernels, one launch, the line
# combine with one and with several threads per output, one and several lines per access
PATHS = [(0, dict(block=64, rows=2, split=1)), (0, dict(block=128, rows=4, split=3)),
         (0, dict(block=64, rows=1, split=11)), (1, dict(block=256, vec=1, unroll=4, split=1)),
         (1, dict(block=128, vec=2, unroll=2, split=5)), (1, dict(block=256, unroll=4, rows=8, split=1)),
         (1, dict(block=128, unroll=8, rows=2, split=12)), (1, dict())]


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()
    from paper_1409_0669_amd import ops
    ops.reset_config()
    yield
    ops.reset_config()


def _strided(values, inc):
    """(buffer, pointer to pass, logical view as a tensor function) of a vector
    with increment inc in the BLAS convention, NaN between its entries."""
    n = values.numel()
    if inc == 0:
        return values[:1].clone(), lambda b: b.expand(n)
    buf = torch.full(((n - 1) * abs(inc) + 1,), float("nan"), dtype=values.dtype, device="cuda")
    view = (lambda b: b[::inc]) if inc > 0 else (lambda b: b.flip(0)[::-inc])
    buf[::abs(inc)] = values if inc > 0 else values.flip(0)
    return buf, view


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("path", range(len(PATHS)))
@pytest.mark.parametrize("beta", [0.0, -0.75])
@pytest.mark.parametrize("incx,incy", [(1, 1), (1, -2), (3, 1), (-2, 3), (0, 2)])
def test_update_is_the_composite(dtype, path, beta, incx, incy):
    from paper_1409_0669_amd import _lib as L
    from paper_1409_0669_amd import ops
    trans, cfg = PATHS[path]
    for op in (L.OP_GEMV_ROWS, L.OP_GEMV_COLS):
        ops.set_config(op, DT[dtype], -1, **cfg)
    m, n, alpha = 131, 203, 0.3
    A, _ = mat(m, n, dtype, 151, pad=1)
    A[5, 7], A[90, 100] = float("inf"), float("nan")
    rows, cols = (n, m) if trans else (m, n)
    x, _ = vec(cols, dtype, 152)
    od = ops.default_out_dtype(DT[dtype])
    y, _ = vec(rows, "f64" if od == torch.float64 else "f32", 153)
    xb, xview = _strided(x, incx)
    xl = xview(xb).contiguous()
    for acc in ("plain", "compensated"):
        s = ops.gemv(A, xl, trans=bool(trans), acc=acc)
        want = ops.scal_to(alpha, s) if beta == 0.0 else ops.axpby(alpha, s, beta, y)
        yb, yview = _strided(y, incy)
        gaps = torch.isnan(yb)
        if beta == 0.0:
            yb.fill_(float("nan"))  # not read
        size = ctypes.c_size_t()
        code, oc = ops.dtype_code(DT[dtype]), ops._DTYPE[od]
        assert L.lib.bwla_gemv_ex_workspace_size(code, oc, L.ROW_MAJOR, trans, m, n, ctypes.byref(size)) == L.OK
        ws = torch.full((max(1, size.value),), 0xA5, dtype=torch.uint8, device="cuda")
        L.check(L.lib.bwla_gemv_ex(code, ops._ACC[acc], L.ROW_MAJOR, trans, m, n, alpha, A.data_ptr(), A.stride(0),
                                   xb.data_ptr(), incx, beta, oc, yb.data_ptr(), incy, ws.data_ptr(), size.value,
                                   ops._stream(A.device)))
        what = "%s path=%d %s beta=%g incx=%d incy=%d" % (dtype, path, acc, beta, incx, incy)
        assert bitwise_equal(host(yview(yb).contiguous()), host(want)), what
        assert bool(torch.isnan(yb[gaps]).all()), what
