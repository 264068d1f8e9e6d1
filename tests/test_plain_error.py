"""Plain sums do not lose accuracy with the terms of a thread: sums of one
repeated value, whose rounding errors all have one sign in a running sum,
against the bound of the short runs they are made of."""
from __future__ import annotations

import pytest
import torch

from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu

# A run of r equal terms c makes errors of at most 2^-p j c at its j-th addition
# (the first term is exact, x being 1): (2 + ... + r) / r of 2^-p, relative.
run = lambda r: (r * (r + 1) / 2 - 1) / r
# float32: runs of four, added up in float64 (and its 2^-53 for a few thousand terms).
F32 = run(4) * 2.0 ** -24 * 1.001
# float32 columns: runs of at most 8 lines, at most 16 of them added up in float32.
COLS = (run(8) + run(16)) * 2.0 ** -24 * 1.001
# float64 rows of 4096 over 64 lanes: runs of four packs (8 terms), 8 of them in a row, 6
# levels of the wave; fewer terms per thread where more share a row.
F64 = (run(8) + run(8) + 6) * 2.0 ** -53


def worst(got, n, c):
    """n is a power of two, n * c exact."""
    exact = n * c.double()
    return float(((got.double() - exact) / exact).abs().max())


@pytest.mark.parametrize("dtype,bound", [(torch.float32, F32), (torch.float64, F64)])
def test_products_of_equal_terms(dtype, bound):
    need_gpu()
    from paper_1409_0669_amd import ops
    from paper_1409_0669_amd.batch import BatchPlan
    ops.reset_config()
    ops.load_default_tuning()
    g = torch.Generator(device="cuda").manual_seed(61)
    for lines, k in ((4096, 4096), (2048, 16384), (64, 1 << 17), (3, 1 << 22), (600, 1 << 13)):
        if dtype == torch.float64 and (lines, k) != (4096, 4096):
            continue  # the bound above is that shape's
        c = torch.rand(lines, generator=g, device="cuda", dtype=dtype) + 1.0
        A, one = c[:, None].expand(lines, k).contiguous(), torch.ones(k, dtype=dtype, device="cuda")
        assert worst(ops.gemv(A, one, out_dtype=torch.float64), k, c) <= bound, ("rows", lines, k)
        if k <= 16384:
            y = torch.empty(lines, dtype=torch.float64, device="cuda")
            BatchPlan([(A, one, y)], [], out_dtype=torch.float64).run()
            torch.cuda.synchronize()
            assert worst(y, k, c) <= bound, ("batch", lines, k)
        if dtype == torch.float32:
            At = A.t().contiguous()  # the same sums down the columns
            assert worst(ops.gemv(At, one, trans=True, out_dtype=torch.float64), k, c) <= COLS, ("cols", k, lines)
        del A


def test_small_dots_of_equal_terms():
    need_gpu()
    from paper_1409_0669_amd import ops
    ops.reset_config()
    g = torch.Generator(device="cuda").manual_seed(62)
    for n in (1024, 8192, 32768, 65536):
        one = torch.ones(n, device="cuda")
        for c in (torch.rand(64, generator=g, device="cuda") + 1.0):
            x = c.expand(n).contiguous()
            assert worst(ops.dot(x, one, out_dtype=torch.float64), n, c) <= F32, n
            assert worst(ops.asum(x, out_dtype=torch.float64), n, c) <= F32, n
