"""Coordinate moments where nothing hides their rounding: no ridge, and windows
narrower than a pixel, whose centre holds nearly all the weight.  Every instance of
the regression against the oracle.

Tolerances: the contract's, 1e-4 * max(1, |.|) on alpha and beta.  The windows hold
five pixels of weight in each of three frames for four unknowns (F = 1); a weight's
own error (an FP32 exponential at an exponent of about -37: 2e-6) moves a beta by
about as much, times the fit's residual.  An error of 1e-16 / (h b)^2 of the moments
would be 1e-13 * 50^2 / 1e-9 > 1e-4 of them at h b = 0.02."""
import numpy as np
import pytest
import torch

import oracle
from paper_2303_02608_amd import binding as B
from paper_2303_02608_amd import synth
from paper_2303_02608_amd.autograd import wlr_alpha
from parity_util import oracle_clip, say, to_dev

pytestmark = pytest.mark.gpu

W, H, T = 37, 23, 3
NARROW = [0.02, 0.02, 2.0]

# schedule, work list, condition output: every instance that a plain regression takes
ROUTES = {"default": (None, False, False), "tiles": ((1, 16, 2), False, False), "two lanes": ((2, 2, 2), False, False),
          "four lanes": ((4, 4, 1), False, False), "list of one lane": ((1, 1, 2), True, False),
          "list of 8 lanes": ((8, 8, 1), True, False), "list": (None, True, False), "condition": (None, False, True)}


def _clip(seed, shape=(W, H, T), f16=False):
    d = synth.random_features_clip(*shape, 1, seed, feat_dtype="f16" if f16 else "f32")
    return d["E"].numpy(), d["feat"].numpy()


def _regress(E, feat, p, route, t):
    schedule, lists, kappa = ROUTES[route]
    y, fd = to_dev(E, feat)
    plan = B.Plan([y], [fd], [p])
    if schedule:
        plan.set_schedule(*schedule)
    n = plan.npix
    items = torch.arange(n, dtype=torch.int64, device="cuda") if lists else None
    cnt = torch.tensor([n, n], dtype=torch.int32, device="cuda") if lists else None
    a, b = torch.full((n,), 7.0, device="cuda"), torch.full((plan.D, n), 7.0, device="cuda")
    k = torch.empty(n, device="cuda") if kappa else None
    B.regress(plan, t, items, cnt, n, a, b, None, k)
    torch.cuda.synchronize()
    return a.cpu().numpy(), b.cpu().numpy().T


def _check(a, b, ref, tag):
    ea = np.abs(a - ref[:, 0]) / np.maximum(1.0, np.abs(ref[:, 0]))
    eb = np.abs(b - ref[:, 1:]) / np.maximum(1.0, np.abs(ref[:, 1:]))
    say(f"{tag}: alpha {ea.max():.1e} beta {eb.max():.1e}")
    assert ea.max() <= 1e-4 and eb.max() <= 1e-4


@pytest.mark.parametrize("r", [5, 7, 9])
@pytest.mark.parametrize("route", sorted(ROUTES))
def test_narrow_windows_without_ridge(route, r):
    E, feat = _clip(60 + r, f16=r == 9)
    b = [v * 7.0 / r for v in NARROW[:2]] + NARROW[2:]        # the same width in pixels
    ref = oracle.regress_items(oracle_clip(E, feat), oracle.Params(r, 1, 0.2, 1.0, b, 0.0), W * H + np.arange(W * H),
                               kappa=False)["theta"]
    got = _regress(E, feat, B.Params(r=r, tr=1, C=0.2, b=b, ridge=0.0), route, 1)
    _check(*got, ref, f"narrow windows, {route} r={r}")


@pytest.mark.parametrize("route", sorted(ROUTES))
@pytest.mark.parametrize("shape", [(40, 1, 3), (1, 40, 3)])
def test_one_row_or_column_without_ridge(route, shape):
    """A coordinate that does not vary leaves a pivot of exactly zero: no solution."""
    say(f"{shape[0]} x {shape[1]} without ridge, {route}")
    E, feat = _clip(7, shape)
    a, b = _regress(E, feat, B.Params(r=5, tr=1, C=0.2, ridge=0.0), route, 1)
    assert np.isnan(a).all() and np.isnan(b).all()


@pytest.mark.parametrize("route", ["default", "tiles", "list"])
def test_bandwidth_selection(route):
    """One candidate, the plan's own: the same regressions."""
    say(f"narrow windows, bandwidth selection, {route}")
    E, feat = _clip(80)
    ref = oracle.regress_items(oracle_clip(E, feat), oracle.Params(7, 1, 0.2, 1.0, NARROW, 0.0),
                               W * H + np.arange(W * H), kappa=False)["theta"]
    schedule, lists, _ = ROUTES[route]
    y, fd = to_dev(E, feat)
    plan = B.Plan([y], [fd], [B.Params(r=7, tr=1, C=0.2, b=NARROW, ridge=0.0)])
    if schedule:
        plan.set_schedule(*schedule)
    n = plan.npix
    items = torch.arange(n, dtype=torch.int64, device="cuda") if lists else None
    cnt = torch.tensor([n, n], dtype=torch.int32, device="cuda") if lists else None
    a, b = torch.full((n,), 7.0, device="cuda"), torch.full((plan.D, n), 7.0, device="cuda")
    B.regress_bandwidth(plan, 1, items, cnt, n, torch.full_like(y, 0.01), [1.0], a, b)
    torch.cuda.synchronize()
    _check(a.cpu().numpy(), b.cpu().numpy().T, ref, f"bandwidth selection, {route}")


def test_gradients():
    """The adjoint's own regressions (tolerances as in the other adjoint tests)."""
    E, feat = _clip(90)
    rng = np.random.default_rng(3)
    items = np.unique(rng.integers(0, T * H * W, size=300))
    ga = rng.standard_normal(items.size)
    y, fd = to_dev(E, feat)
    y = y.clone().requires_grad_(True)
    bt = torch.tensor(NARROW, dtype=torch.float64, requires_grad=True)
    dev = torch.from_numpy(((items // (H * W)) << 44) | (items % (H * W))).cuda()
    alpha = wlr_alpha(y, bt, fd, dev, 7, 1, C=0.2, ridge=0.0)
    (alpha * torch.from_numpy(ga).float().cuda()).sum().backward()
    torch.cuda.synchronize()
    ref_y, ref_b, fails = oracle.backward(oracle_clip(E, feat), oracle.Params(7, 1, 0.2, 1.0, NARROW, 0.0), items, ga)
    assert fails == 0
    ey = np.abs(y.grad.cpu().numpy() - ref_y).max() / np.abs(ref_y).max()
    eb = np.abs(bt.grad.numpy() - ref_b) / np.maximum(1e-3 * np.abs(ref_b).max(), np.abs(ref_b))
    say(f"narrow windows, gradients: gy {ey:.1e} gb {eb.max():.1e}")
    assert ey <= 1e-4 and eb.max() <= 1e-4
