"""GPU parity of the reductions around the size up to which one work-group
takes them in one launch."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from tests.criteria import TOL, bitwise_equal, check_scalar, cond_scale
from tests.gpu_util import DT, host, need_gpu, vec

pytestmark = pytest.mark.gpu

DTYPES = ["f64", "f32", "bf16"]


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()
    from paper_1409_0669_amd import ops
    ops.reset_config()
    yield
    ops.reset_config()


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("acc", ["plain", "compensated"])
@pytest.mark.parametrize("past", [-1, 0, 1])
@pytest.mark.parametrize("start", [0, 1])
def test_reductions_around_one_work_group(dtype, acc, past, start):
    """256 KiB over two vectors (the inner product), one (the norms) and six
    (the update): at, below and past it, and lengths of a few elements."""
    from paper_1409_0669_amd import _lib as L
    from paper_1409_0669_amd import ops
    size = torch.empty(0, dtype=DT[dtype]).element_size()
    for streams in (1, 2, 6):
        for n in ((1 << 18) // (size * streams) + past, 3 + past):
            what = "%s %s n=%d start=%d" % (dtype, acc, n, start)
            op = {1: L.OP_NRM2, 2: L.OP_DOT, 6: L.OP_CG}[streams]
            if n * size * streams <= 1 << 18:
                assert ops.get_config(op, DT[dtype], 0, n, acc=acc)["grid"] == 1, what
            x, x64 = vec(n, dtype, 154, pad_front=start)
            y, y64 = vec(n, dtype, 155, pad_front=start)
            if streams == 1:
                check_scalar(float(ops.nrm2(x, acc=acc)), oracle.nrm2(x64), 0.0, TOL[dtype], what)
                check_scalar(float(ops.asum(x, acc=acc)), oracle.asum(x64), 0.0, TOL[dtype], what)
            elif streams == 2:
                got = ops.dot(x, y, acc=acc)
                check_scalar(float(got), oracle.dot(x64, y64), cond_scale(dtype, acc, np.abs(x64 * y64).sum()),
                             TOL[dtype], what)
                assert torch.equal(got, ops.dot_noalloc(x, y, acc=acc)), what
            else:
                r, p = y.clone(), x.clone()
                rref = oracle.axpby(dtype, -0.5, x64, 1.0, y64)
                rr = ops.cg_update(0.5, x, p, r, p, acc=acc)
                assert bitwise_equal(host(r), rref), what
                check_scalar(float(rr), oracle.dot(rref, rref), 0.0, TOL[dtype], what)
