"""Small reductions follow a configuration that is set for them, and have a
rule of their own where none is."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from tests.criteria import TOL, check_scalar, cond_scale
from tests.gpu_util import DT, need_gpu, vec


@pytest.fixture(autouse=True)
def _defaults():
    from paper_1409_0669_amd import ops
    ops.reset_config()
    yield
    ops.reset_config()


@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
def test_entries_are_followed_at_every_size(dtype, tmp_path):
    from paper_1409_0669_amd import _lib as L
    from paper_1409_0669_amd import ops, tune
    size = torch.empty(0, dtype=DT[dtype]).element_size()
    want = dict(block=128, vec=2, unroll=2, grid=5, increment=1)
    for op, streams in ((L.OP_DOT, 2), (L.OP_NRM2, 1), (L.OP_CG, 6)):
        for acc in ("plain", "compensated"):
            assert ops.get_config(op, DT[dtype], 0, 1000, acc=acc)["grid"] == 1  # the rule
            for n in (3, 1000, (1 << 18) // (size * streams), (1 << 19) // (size * streams)):
                ops.set_config(op, DT[dtype], 0, acc=acc, **want)
                got = ops.get_config(op, DT[dtype], 0, n, acc=acc)
                assert {k: got[k] for k in want} == want, (op, acc, n)
                ops.set_config(op, DT[dtype], 0, acc=acc, unroll=4)  # one field is an entry too
                assert ops.get_config(op, DT[dtype], 0, n, acc=acc)["unroll"] == 4
                ops.set_config(op, DT[dtype], 0, acc=acc)
    path = str(tmp_path / "t.txt")  # a table saved before the rule
    tune.write_table([(L.OP_DOT, DT[dtype], "plain", 0, want)], path)
    ops.load_tuning(path)
    assert ops.get_config(L.OP_DOT, DT[dtype], 0, 1000)["grid"] == 5
    assert ops.get_config(L.OP_DOT, DT[dtype], 0, 1000, acc="compensated")["grid"] == 1


def test_the_shipped_table_leaves_small_reductions_to_the_rule():
    from paper_1409_0669_amd import _lib as L
    from paper_1409_0669_amd import ops, tune
    ops.load_tuning(tune.DEFAULT_TABLE)
    for dt, size in ((torch.float64, 8), (torch.float32, 4), (torch.bfloat16, 2)):
        for op, streams in ((L.OP_DOT, 2), (L.OP_NRM2, 1), (L.OP_CG, 6)):
            for acc in ("plain", "compensated"):
                assert ops.get_config(op, dt, 0, (1 << 18) // (size * streams), acc=acc)["grid"] == 1
                assert ops.get_config(op, dt, 0, (1 << 18) // (size * streams) + 1, acc=acc)["grid"] > 1


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("acc", ["plain", "compensated"])
def test_above_one_work_group(dtype, acc):
    need_gpu()
    from paper_1409_0669_amd import ops
    size = torch.empty(0, dtype=DT[dtype]).element_size()
    for kb in (257, 600, 1023, 1024):
        n = kb * 1024 // (2 * size) - 1
        x, x64 = vec(n + 1, dtype, 171)
        y, y64 = vec(n + 1, dtype, 172)
        check_scalar(float(ops.dot(x[1:], y[1:], acc=acc)), oracle.dot(x64[1:], y64[1:]),
                     cond_scale(dtype, acc, np.abs(x64 * y64).sum()), TOL[dtype], "dot %d" % n)
        check_scalar(float(ops.nrm2(x[1:], acc=acc)), oracle.nrm2(x64[1:]), 0.0, TOL[dtype], "nrm2 %d" % n)
