"""Few long lines: the rows GEMV splits them over the chip, the same way with
and without the inner-product epilogue."""
from __future__ import annotations

import ctypes

import pytest
import torch

from tests.gpu_util import DT, guarded, need_gpu


@pytest.fixture(autouse=True)
def _defaults():
    from paper_1409_0669_amd import ops
    ops.reset_config()
    yield
    ops.reset_config()


def test_few_long_lines_fill_the_chip():
    from paper_1409_0669_amd import _lib as L
    c, b = L.Config(), ctypes.c_size_t()
    for t, size in enumerate((8, 4, 2)):
        for lines in (1, 2, 3, 4, 7, 8, 16, 31, 64, 100, 128, 200, 300, 511, 600, 1000):
            for mb in (8, 100, 300, 800, 1600):
                k = mb * 1_000_000 // size // lines
                assert L.lib.bwla_workspace_size(L.OP_GEMV_ROWS, t, 0, L.ROW_MAJOR, 0, lines, k, ctypes.byref(b)) == L.OK
                for acc in (0, 1):
                    assert L.lib.bwla_get_config(L.OP_GEMV_ROWS, t, acc, lines, k, ctypes.byref(c)) == L.OK
                    what = (t, acc, lines, k, c.block, c.rows, c.split)
                    groups = -(-lines // c.rows)
                    assert c.rows <= max(1, lines + lines // 3), what
                    assert c.split == 1 or b.value >= groups * c.split * c.rows * 16, what
                    if lines < 512 or mb >= 300:  # every CU has work, unless the matrix is of a few MB
                        assert groups * c.split >= (90 if mb == 8 else 190), what


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("lines,k", [(1, 4_000_003), (1, 130_001), (2, 1_000_001), (3, 700_000), (4, 9_000_007),
                                     (9, 250_001), (300, 230_001), (600, 60_000), (511, 300_001)])
def test_few_long_lines_are_exact(dtype, lines, k):
    need_gpu()
    from paper_1409_0669_amd import ops
    g = torch.Generator(device="cuda").manual_seed(53)
    draw = lambda *s: torch.randint(-1, 2, s, generator=g, device="cuda", dtype=torch.int8).to(DT[dtype])
    A, x = draw(lines, k + 1)[:, 1:], draw(k)
    ref = torch.stack([(A[i].double() * x.double()).sum() for i in range(lines)])
    od = ops.default_out_dtype(DT[dtype])
    for acc in ("plain", "compensated"):
        y, guard = guarded(lines, od)
        ops.gemv(A, x, acc=acc, out=y)
        assert torch.equal(y.double(), ref), (dtype, lines, k, acc)
        y.fill_(1.0)
        ops.gemv(A, x, acc=acc, out=y, alpha=0.5, beta=2.0)
        assert torch.equal(y.double(), 0.5 * ref + 2.0), (dtype, lines, k, acc)
        guard()
        if dtype != "bf16":
            y2, s = ops.gemv_dot(A, x, w=torch.ones(lines, dtype=od, device="cuda"), acc=acc)
            assert torch.equal(y2.double(), ref) and s.item() == float(ref.sum()), (dtype, lines, k, acc)


@pytest.mark.gpu
@pytest.mark.parametrize("lines,k", [(4, 20_000_003), (300, 300_001), (700, 200_000), (2049, 40_000)])
def test_fused_and_separate_products_have_the_same_bits(lines, k):
    need_gpu()
    from paper_1409_0669_amd import ops
    g = torch.Generator(device="cuda").manual_seed(54)
    for dtype in (torch.float64, torch.float32):
        A = torch.rand(lines, k, generator=g, device="cuda", dtype=dtype)
        x, w = torch.rand(k, generator=g, device="cuda", dtype=dtype), torch.rand(lines, device="cuda", dtype=dtype)
        for acc in ("plain", "compensated"):
            y, _ = ops.gemv_dot(A, x, w=w, acc=acc)
            assert torch.equal(y, ops.gemv(A, x, acc=acc)), (dtype, lines, k, acc)
        del A
