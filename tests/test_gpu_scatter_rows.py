"""Every-crossing events of frames whose rows, flag blocks and words do not line
up, in order and with a full event buffer, against the rule in FP64 on the same
FP32 brightness and state.

Tolerances: pixels, frames, polarities and their order exactly; interpolated
times within the FP32 rounding of the result."""
import numpy as np
import pytest
import torch

from paper_2303_02608_amd import binding as B
from paper_2303_02608_amd.simulator import Simulator
from parity_util import say

pytestmark = pytest.mark.gpu


def _rule(y, C):
    T, H, W = y.shape
    ref, last = y[0].reshape(-1).copy(), y[0].reshape(-1).copy()
    out = []
    for t in range(1, T):
        L = y[t].reshape(-1)
        d = L.astype(np.float64) - ref.astype(np.float64)
        n = np.floor(np.abs(d) / C).astype(np.int64)
        for p in np.nonzero(n)[0]:
            step = C if d[p] > 0 else -C
            den = float(L[p]) - float(last[p])
            for k in range(1, n[p] + 1):
                ts = ((t - 1) + (float(ref[p]) + k * step - float(last[p])) / den)
                out.append((p % W, p // W, t, 1 if step > 0 else -1, ts))
            ref[p] = np.float32(float(ref[p]) + n[p] * step)
        last = L.copy()
    return out, ref


@pytest.mark.parametrize("W,H,share", [(5, 70, 0.9), (63, 9, 0.02), (255, 5, 0.3), (256, 5, 0.3), (300, 7, 1.0),
                                       (1030, 2, 0.05)])
def test_every_crossing_in_order(W, H, share):
    T, C = 4, 0.25
    say(f"every crossing {W}x{H} share {share}")
    rng = np.random.default_rng(W)
    # brightness and levels in whole sixteenths: changes, counts and references are exact
    step = rng.integers(-24, 25, (T, H, W)) / 8.0 + 1.0 / 16.0
    y = np.cumsum(np.where(rng.random((T, H, W)) < share, step, 0.0), axis=0).astype(np.float32)
    feat = torch.zeros((T, 3, H, W), device="cuda")
    want, ref = _rule(y, C)
    assert len(want) > 0
    for capacity in (len(want) + 1, 2 * len(want) // 3):
        sim = Simulator(torch.from_numpy(y).cuda(), feat, B.Params(r=2, tr=0, C=C, multi_crossing=True),
                        capacity=capacity)
        got = sim.run("raw")
        assert got["count"] == len(want)
        n = min(capacity, len(want))
        for i, key in enumerate("xytp"):
            assert np.array_equal(got[key][:n], np.array([e[i] for e in want[:n]])), key
        ts = np.array([e[4] for e in want[:n]])
        assert np.max(np.abs(got["ts"][:n] - ts)) <= 2.0 ** -22 * T
        assert np.array_equal(sim.state.alpha.cpu().numpy().reshape(-1), ref)
