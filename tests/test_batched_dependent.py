"""Plans whose problems depend on each other by kind: a dot of a GEMV's
result, a long-rowed GEMV of a short-rowed one's, a dot that overwrites an
entry of a GEMV's x.  Whole-number sums, exact in every order."""
from __future__ import annotations

import pytest
import torch

from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("acc", ["plain", "compensated"])
def test_results_used_by_a_later_kind(dtype, acc):
    need_gpu()
    from paper_1409_0669_amd.batch import BatchPlan
    g = torch.Generator(device="cuda").manual_seed(47)
    draw = lambda *s: torch.randint(-1, 2, s, generator=g, device="cuda").to(dtype)
    nan = lambda n: torch.full((n,), float("nan"), dtype=dtype, device="cuda")
    A1, x1, y1 = draw(9000, 130), draw(130), nan(9000)
    A2, y2 = draw(70, 9000), nan(70)  # x is y1: rows too long for the first kind
    A3, x3, y3 = draw(500, 257), draw(257), nan(500)
    w, s1, s2 = draw(9000), nan(1), nan(1)
    u, c, d = draw(70), draw(40000), draw(40000)
    # the last dot's result replaces an entry that A3's product reads before
    plan = BatchPlan([(A2, y1, y2), (A1, x1, y1), (A3, x3, y3)],
                     [(y1, w, s1), (y2, u, s2), (c, d, x3[:1])], acc=acc)
    stream = torch.cuda.Stream()
    for replay in range(4):
        x3[0] = 1.0
        r1 = A1.double().cpu() @ x1.double().cpu()
        r2, r3 = A2.double().cpu() @ r1, A3.double().cpu() @ x3.double().cpu()
        for t in (y1, y2, y3, s1, s2):
            t.fill_(float("nan"))
        torch.cuda.synchronize()
        if replay == 0:
            plan.run()
        else:
            with torch.cuda.stream(stream):
                if replay == 1:
                    plan.capture()
                plan.replay()
        torch.cuda.synchronize()
        assert torch.equal(y1.double().cpu(), r1) and torch.equal(y3.double().cpu(), r3), replay
        assert torch.equal(y2.double().cpu(), r2), replay
        assert s1.item() == float(w.double().cpu() @ r1), replay
        assert s2.item() == float(u.double().cpu() @ r2), replay
        assert x3[0].item() == float(c.double().cpu() @ d.double().cpu()), replay
    plan.close()

