"""The cols GEMV at the ends of its range: lines shorter than a pack or than a
tile, a handful of very long lines, and widths near the thread count that one
launch holds."""
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


def _config(t, acc, lines, k):
    from paper_1409_0669_amd import _lib as L
    c, b = L.Config(), ctypes.c_size_t()
    assert L.lib.bwla_get_config(L.OP_GEMV_COLS, t, acc, lines, k, ctypes.byref(c)) == L.OK
    assert L.lib.bwla_workspace_size(L.OP_GEMV_COLS, t, acc, L.ROW_MAJOR, 1, lines, k, ctypes.byref(b)) == L.OK
    tile = 64 // c.rows * c.vec
    tiles = -(-k // tile)
    assert c.split == 1 or b.value >= tiles * c.split * tile * 16
    return c, tiles


def test_widths_fit_a_launch():
    for t, size in enumerate((8, 4, 2)):
        for lines in (1, 2, 3, 40, 100):
            for k in [1 << e for e in range(24, 33)] + [(1 << 29) + 5, (1 << 30) + 1]:
                if lines * k * size <= 1 << 38:
                    for acc in (0, 1):
                        c, tiles = _config(t, acc, lines, k)
                        assert tiles * c.split * c.block < 1 << 32, (t, acc, lines, k, c.block, c.rows, c.split)


def test_short_lines_keep_loads_in_flight_and_the_chip_full():
    for t, size in enumerate((8, 4, 2)):
        for k in (1, 2, 3, 5, 7, 9, 16, 33, 48):
            for lines in (40_000, 1_000_000, 20_000_000):
                for acc in (0, 1):
                    c, tiles = _config(t, acc, lines, k)
                    what = (t, acc, lines, k, c.block, c.vec, c.rows, c.unroll, c.split)
                    assert c.vec <= max(1, k), what
                    if k < 16 // size:  # one line per access: 16 of them in flight
                        assert c.unroll == 16 and c.rows == 1, what
                    else:
                        assert tiles == 1 or 4 * k > 3 * 64 // c.rows * c.vec, what
                    if lines >= 1_000_000:
                        assert tiles * c.split >= 128, what


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("lines,k", [(300_001, 1), (70_001, 2), (40_003, 3), (900_000, 5), (90_001, 7), (50_000, 9),
                                     (33_333, 17), (20_001, 33), (1, 1_000_003), (2, 500_001), (3, 4_000_003),
                                     (8, 70_001), (33, 9_999), (39, 1_100_000), (100, 300_001), (500, 200_000)])
def test_extremes_are_exact(dtype, lines, k):
    need_gpu()
    from paper_1409_0669_amd import ops
    g = torch.Generator(device="cuda").manual_seed(57)
    draw = lambda *s: torch.randint(-1, 2, s, generator=g, device="cuda", dtype=torch.int8).to(DT[dtype])
    od = ops.default_out_dtype(DT[dtype])
    for start in (0, 1):
        A, x = draw(lines, k + start)[:, start:], draw(3 * lines)
        for acc in ("plain", "compensated"):
            for inc in (1, 3):
                v = x[::3] if inc == 3 else x[:lines]
                ref = torch.zeros(k, dtype=torch.float64, device="cuda")
                for i in range(0, lines, 4096):
                    ref += (A[i:i + 4096].double() * v[i:i + 4096, None].double()).sum(0)
                y, guard = guarded(k, od)
                ops.gemv(A, v, trans=True, acc=acc, out=y)
                assert torch.equal(y.double(), ref), (dtype, lines, k, start, acc, inc)
                guard()
            if dtype != "bf16":
                y2, s = ops.gemv_dot(A, v.contiguous(), w=torch.ones(k, dtype=od, device="cuda"), trans=True, acc=acc)
                assert torch.equal(y2.double(), ref) and s.item() == float(ref.sum()), (dtype, lines, k, start, acc)
