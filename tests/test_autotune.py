"""The schedule autotuner's choice, on a stand-in plan with given times."""
import pytest
import torch

from paper_2303_02608_amd import autotune
from paper_2303_02608_amd import binding as B


class FakePlan:
    """dense, lists: time by lanes (None: the automatic schedule) and blocks per CU."""

    def __init__(self, dense, lists, F=7, precision=B.GRAM_F64):
        self.dense, self.lists = dense, lists
        self.feats = [torch.zeros((20, F, 2, 2))]
        self.ys = [torch.zeros((20, 2, 2))]
        self.params = [B.Params(r=5, tr=0, C=0.2, precision=precision)]
        self.states = None
        self.npix = self.wl_capacity = 4
        self.F, self.D = F, F + 2
        self.schedule, self.schedule_set = (1, 16, 4), False
        self.tried = []

    def set_schedule(self, *s):
        self.schedule, self.schedule_set = s, True

    def times(self):
        ld, ll, b = self.schedule if self.schedule_set else (None, 16, 1)
        self.tried.append((ld, ll, b))
        return self.dense(ld, b), self.lists(ll, b)


@pytest.fixture
def tuned(monkeypatch):
    def run(plan, **kw):
        trial = FakePlan(plan.dense, plan.lists, plan.F, plan.params[0].precision)
        monkeypatch.setattr(autotune, "_cache", {})
        monkeypatch.setattr(autotune, "_trial", lambda p: trial, raising=False)
        monkeypatch.setattr(autotune, "_time_prefix", lambda p, frames, bufs: p.times())
        got = autotune.tune(plan, **kw)
        return got, trial
    return run


def _cost(plan):
    return sum(plan.times())


def test_small_frames_keep_their_automatic_lanes(tuned):
    """A frame that 16 lanes per item suit: the tuned plan is no slower than before."""
    dense = {None: 0.019, 1: 0.129, 2: 0.080, 4: 0.040, 8: 0.025, 16: 0.019}
    plan = FakePlan(lambda L, b: dense[L], lambda L, b: {4: 0.03, 8: 0.02, 16: 0.011}[L])
    before = _cost(plan)
    got, _ = tuned(plan)
    assert got == plan.schedule
    assert _cost(plan) <= before


def test_mixed_plans_keep_what_suits_each_clip(tuned):
    """Faster than any one number of lanes for all clips."""
    dense = {None: 1.0, 1: 1.3, 2: 1.8, 4: 2.0, 8: 2.0, 16: 1.5}
    plan = FakePlan(lambda L, b: dense[L], lambda L, b: {4: 0.3, 8: 0.2, 16: 0.1}[L])
    tuned(plan)
    assert not plan.schedule_set


def test_faster_candidates_are_applied(tuned):
    plan = FakePlan(lambda L, b: {None: 1.0, 1: 1.0}.get(L, 0.5 if (L, b) == (2, 2) else 0.9),
                    lambda L, b: {4: 0.3, 8: 0.05, 16: 0.1}[L])
    got, _ = tuned(plan)
    assert got == plan.schedule == (2, 8, 2) and plan.schedule_set


@pytest.mark.parametrize("F,precision,blocks", [(7, B.GRAM_F64, {1, 2}), (10, B.GRAM_F64, {1}), (7, B.GRAM_F32C, {1})])
def test_blocks_without_effect_are_not_tried_again(tuned, F, precision, blocks):
    plan = FakePlan(lambda L, b: 1.0, lambda L, b: 1.0, F, precision)
    _, trial = tuned(plan)
    assert {b for ld, _, b in trial.tried if ld in (1, 2)} == blocks
    assert {b for ld, ll, b in trial.tried if ld is not None and ld > 2} == {1}


def test_a_schedule_set_by_hand_is_replaced(tuned):
    plan = FakePlan(lambda L, b: {1: 1.0}.get(L, 2.0), lambda L, b: {16: 0.1}.get(L, 0.2))
    plan.set_schedule(4, 4, 4)
    got, trial = tuned(plan)
    assert got == plan.schedule == (1, 16, 1)
    assert all(ld is not None for ld, _, _ in trial.tried)
