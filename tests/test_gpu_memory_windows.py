"""Instances that read every window from memory: dense frames whose windows do not
fit LDS, one and two lanes per item set by hand, and the condition output, over
feature counts, half precision and every count of frames.

Tolerances: the contract's, 1e-4 * max(1, |.|) on alpha and beta and 1e-6 on R; the
random features keep every window well conditioned."""
import numpy as np
import pytest
import torch

import oracle
from paper_2303_02608_amd import binding as B
from paper_2303_02608_amd import synth
from parity_util import oracle_clip, say, to_dev

pytestmark = pytest.mark.gpu


def _compare(a, b, R, ref, tag):
    th = ref["theta"]
    ea = np.abs(a - th[:, 0]) / np.maximum(1.0, np.abs(th[:, 0]))
    eb = np.abs(b.T - th[:, 1:]) / np.maximum(1.0, np.abs(th[:, 1:]))
    er = np.abs(R - ref["R"])
    say(f"{tag}: alpha {ea.max():.1e} beta {eb.max():.1e} R {er.max():.1e}")
    assert ea.max() <= 1e-4 and eb.max() <= 1e-4 and er.max() <= 1e-6, tag


def _check(W, H, T, F, r, tr, t, f16, schedule, kappa):
    tag = f"memory {W}x{H} T={T} F={F} r={r} tr={tr} t={t} f16={f16} {schedule} kappa={kappa}"
    say(tag)
    d = synth.random_features_clip(W, H, T, F, 400 + F + r, feat_dtype="f16" if f16 else "f32")
    E, feat = d["E"].numpy(), d["feat"].numpy()
    y, fd = to_dev(E, feat)
    plan = B.Plan([y], [fd], [B.Params(r=r, tr=tr, C=0.2, h=1.2)])
    plan.set_schedule(*schedule)
    n = plan.npix
    a, b = torch.full((n,), 7.0, device="cuda"), torch.full((plan.D, n), 7.0, device="cuda")
    R = torch.full((n,), 7.0, device="cuda")
    k = torch.full((n,), -1.0, device="cuda") if kappa else None
    B.regress(plan, t, None, None, n, a, b, R, k)
    torch.cuda.synchronize()
    ref = oracle.regress_items(oracle_clip(E, feat), oracle.Params(r, tr, 0.2, 1.2), t * W * H + np.arange(W * H),
                               kappa=False)
    _compare(a.cpu().numpy(), b.cpu().numpy(), R.cpu().numpy(), ref, tag)
    assert k is None or float(k.min()) >= 1.0


@pytest.mark.parametrize("F,tr,t,f16", [(1, 0, 0, False), (2, 1, 1, True), (3, 2, 2, False), (4, 1, 0, False),
                                        (5, 2, 1, True), (6, 3, 3, False), (7, 1, 1, False), (7, 2, 2, True),
                                        (8, 0, 0, False), (8, 1, 1, True), (8, 2, 2, False), (9, 1, 1, False),
                                        (10, 2, 2, True), (11, 1, 0, False), (12, 2, 2, False), (12, 1, 1, True)])
def test_windows_beyond_lds(F, tr, t, f16):
    """A radius whose rows take more than two turns of a wave: no tiles at any F."""
    _check(23, 9, 7 if tr == 3 else 5, F, 57, tr, t, f16, (1, 16, 2), False)


@pytest.mark.parametrize("lanes,kappa", [(2, False), (1, True)])
@pytest.mark.parametrize("F,r,tr,t,f16", [(1, 4, 2, 2, False), (3, 3, 1, 1, True), (7, 5, 1, 1, False), (7, 5, 2, 2, True),
                                          (8, 4, 0, 0, False), (8, 5, 2, 2, False), (10, 3, 1, 0, True),
                                          (12, 3, 2, 2, False)])
def test_two_lanes_and_condition_output(F, r, tr, t, f16, lanes, kappa):
    _check(31, 17, 5, F, r, tr, t, f16, (lanes, 16, 2), kappa)


@pytest.mark.parametrize("W,H", [(3, 67), (7, 41), (1, 129)])
def test_narrow_images(W, H):
    """Images narrower than half a tile: packed lanes, from memory."""
    _check(W, H, 3, 7, 4, 1, 1, False, (1, 16, 2), False)
