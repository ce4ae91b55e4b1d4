"""A tuned plan is no slower than an untuned one where the automatic schedule is far
ahead of one lane per pixel (4096 pixels, r = 7, three frames: 7 times), and gives the
same regressions to the contract's tolerance, 1e-4 * max(1, |.|)."""
import numpy as np
import pytest
import torch

from paper_2303_02608_amd import autotune
from paper_2303_02608_amd import binding as B
from paper_2303_02608_amd import synth
from parity_util import say, to_dev

pytestmark = pytest.mark.gpu


def _dense(plan):
    """Regression of frame 1 and the least of 20 times, us."""
    a, b = torch.empty(plan.npix, device="cuda"), torch.empty((plan.D, plan.npix), device="cuda")
    best = float("inf")
    for _ in range(20):
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        e[0].record()
        B.regress(plan, 1, None, None, plan.npix, a, b)
        e[1].record()
        torch.cuda.synchronize()
        best = min(best, e[0].elapsed_time(e[1]) * 1e3)
    return a.cpu().numpy(), best


def test_tuned_small_plan():
    d = synth.make_clip(synth.ClipSpec(W=64, H=64, T=8, spp=4, F=7, n_discs=4, seed=41))
    y, f = to_dev(d["E"].numpy(), d["feat"].numpy())
    plans = [B.Plan([y], [f], [B.Params(r=7, tr=1, C=0.2)]) for _ in range(2)]
    sched = autotune.tune(plans[1], frames=4)
    (a0, t0), (a1, t1) = _dense(plans[0]), _dense(plans[1])
    say(f"tuned {sched}: {t1:.1f} us, untuned {t0:.1f} us")
    assert t1 <= 2.0 * t0
    assert np.max(np.abs(a1 - a0) / np.maximum(1.0, np.abs(a0))) <= 1e-4
