"""Dots of a batch around whole chunks and around the 64 chunks that the
finalize kernel takes one lane each: sums of whole numbers, exact in every
order, next to GEMVs in the same launch, through run and replay."""
from __future__ import annotations

import pytest
import torch

from tests.gpu_util import DT, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("acc", ["plain", "compensated"])
@pytest.mark.parametrize("block", [64, 256, 512])
def test_dots_around_whole_chunks(dtype, acc, block):
    need_gpu()
    from paper_1409_0669_amd.batch import BatchPlan
    chunk = 65536 // torch.empty(0, dtype=DT[dtype]).element_size()
    od = torch.float64 if dtype == "f64" else torch.float32
    # values in {-1, 0, 1}: every partial sum is below 2^24, exact in float32
    g = torch.Generator(device="cuda").manual_seed(43)
    draw = lambda *s: (torch.randint(-1, 2, s, generator=g, device="cuda")).to(DT[dtype])
    sizes = [1, chunk - 1, chunk, chunk + 1, 2 * chunk, 63 * chunk + 5, 64 * chunk, 64 * chunk + 1, 65 * chunk, 0]
    dots = [(draw(n + i % 3)[i % 3:], draw(n), torch.full((1,), float("nan"), dtype=od, device="cuda"))
            for i, n in enumerate(sizes)]
    gemvs = [(draw(m, n), draw(n), torch.full((m,), float("nan"), dtype=od, device="cuda"))
             for m, n in ((65, 3), (300, 129), (9, 5000))]
    plan = BatchPlan(gemvs, dots, acc=acc, block=block)
    s = torch.cuda.Stream()
    plan.run()
    for replay in range(3):
        torch.cuda.synchronize()
        for p, q, out in dots:
            assert out.item() == float((p.double() * q.double()).sum()), (p.numel(), replay)
            out.fill_(float("nan"))
        for A, x, y in gemvs:
            assert torch.equal(y.double().cpu(), A.double().cpu() @ x.double().cpu()), (A.shape, replay)
            y.fill_(float("nan"))
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            if replay == 0:
                plan.capture()
            plan.replay()
    torch.cuda.synchronize()
    plan.close()
