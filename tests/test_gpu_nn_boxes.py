"""Nearest-neighbour distances over boxes narrower and wider than the words read
first, with queries at the image's and the bitmap's ends, against every pair of
events in FP64.

Tolerance: the rounding of the FP64 distance."""
import numpy as np
import pytest
import torch

from paper_2303_02608_amd import binding as B
from paper_2303_02608_amd import quality as Q
from parity_util import say

pytestmark = pytest.mark.gpu


def _events(rng, W, H, T, n):
    return {"x": rng.integers(0, W, n), "y": rng.integers(0, H, n), "t": rng.integers(0, T, n),
            "p": rng.choice([-1, 1], n)}


@pytest.mark.parametrize("W,H,T,n,rmax", [(31, 5, 2, 6, 0.9), (32, 3, 1, 3, 1.5), (33, 40, 3, 12, 0.5),
                                          (64, 9, 4, 40, 0.2), (300, 7, 3, 9, 0.4), (300, 7, 3, 60, 0.1),
                                          (1300, 6, 2, 10, 0.3)])
def test_boxes_against_every_pair(W, H, T, n, rmax):
    say(f"nn boxes {W}x{H}x{T} n={n} rmax={rmax}")
    rng = np.random.default_rng(W + n)
    src, qry = _events(rng, W, H, T, n), _events(rng, W, H, T, 3000)
    for key, top in (("x", W), ("y", H), ("t", T)):           # the ends of every extent
        qry[key][:400] = rng.choice([0, top - 1], 400)
    # sources and queries outside are ignored: no neighbour, no distance
    src["x"][0], qry["y"][7] = W, -1
    got = B.nn_distances(Q.to_device(src), Q.to_device(qry), W, H, T, rmax).cpu().numpy()
    s = {k: v[1:].astype(np.float64) for k, v in src.items()}
    q = {k: v[:, None].astype(np.float64) for k, v in qry.items()}
    d = np.sqrt(((q["x"] - s["x"]) / W) ** 2 + ((q["y"] - s["y"]) / H) ** 2 + ((q["t"] - s["t"]) / T) ** 2)
    d = np.where(q["p"] == s["p"], d, np.inf).min(axis=1)
    d[7] = np.inf
    edge = np.abs(d - rmax) <= 1e-12
    want = np.where(d <= rmax, d, np.inf)
    assert np.array_equal(np.isinf(got[~edge]), np.isinf(want[~edge]))
    fin = np.isfinite(want) & ~edge
    assert fin.any() and np.max(np.abs(got[fin] - want[fin])) <= 1e-14
