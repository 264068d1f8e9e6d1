"""The tuner's choice between the library's shape rule and a fixed entry, and
what it reports of both (no GPU)."""
from __future__ import annotations

import torch


def test_report_has_both_sides():
    from paper_1409_0669_amd import tune
    rule, fixed = tune._gemv_rule(4), dict(block=256, vec=4, unroll=2, split=0, grid=512, rows=2)
    entry, rec = tune.rule_or_fixed(rule, [950.0, 950.0], fixed, 1000.0, {0: 1000.0, 1: 1000.0})
    assert entry == rec["best"] == rule and rec["best_gbs_geomean"] == 950.0
    assert rec["fixed"] == fixed and rec["fixed_gbs_geomean"] == 1000.0  # what the rule gives up
    assert rec["fixed_gbs_per_shape"] == [1000.0, 1000.0] and rec["default_gbs_per_shape"] == [950.0, 950.0]
    entry, rec = tune.rule_or_fixed(rule, [900.0, 900.0], fixed, 1000.0, {0: 1000.0, 1: 1000.0})
    assert entry == rec["best"] == fixed and rec["best_gbs_geomean"] == 1000.0
    assert rec["best_gbs_per_shape"] == [1000.0, 1000.0] and rec["default_gbs_per_shape"] == [900.0, 900.0]


def test_candidates_are_fixed_and_distinct():
    from paper_1409_0669_amd import tune
    key = lambda c: tuple(sorted(c.items()))
    for dt in (torch.float64, torch.float32, torch.bfloat16):
        for quick in (False, True):
            for cands in (tune._rows_candidates(dt, quick), tune._cols_candidates(dt, quick)):
                assert all(c["block"] for c in cands)  # no candidate is the rule
                assert len({key(c) for c in cands}) == len(cands)
    for quick in (False, True):  # a plan takes more than 8 packs per lane as 8
        c = tune._batch_candidates(quick)
        assert len({(d["block"], min(d["unroll"], 8)) for d in c}) == len(c) >= 4
