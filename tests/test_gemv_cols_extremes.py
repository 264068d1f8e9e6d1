"""The cols GEMV at the ends of its range: widths near the thread count that one
launch holds."""
from __future__ import annotations

import ctypes

import pytest


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
