"""Nearest-neighbour distances over bitmaps below and above 4 GiB (32-bit offsets, and
the kernel with 64-bit rows), with events at the far end of the map, against every
pair of events in FP64.

Tolerance: the rounding of the FP64 distance."""
import numpy as np
import pytest
import torch

from paper_2303_02608_amd import binding as B
from paper_2303_02608_amd import quality as Q
from parity_util import say

pytestmark = pytest.mark.gpu

W, RMAX = 65536, 0.004


@pytest.mark.parametrize("H,T", [(16383, 16), (16384, 16), (16390, 17)])
def test_large_bitmaps(H, T):
    nbytes = B.load().esim_nn_scratch_bytes(W, H, T)
    say(f"nn {W}x{H}x{T}: bitmaps of {nbytes} bytes")
    assert (nbytes >= 2 ** 32 - 4) == (H >= 16384)
    rng = np.random.default_rng(H)
    n, k = 150, 20
    src = {"x": rng.integers(0, W, n), "y": rng.integers(0, H, n), "t": rng.integers(0, T, n),
           "p": rng.choice([-1, 1], n)}
    for key, top in (("x", W), ("y", H), ("t", T)):           # the last words of the map
        src[key][:30] = top - 1 - rng.integers(0, 2 if key == "t" else 40, 30)
    # queries around the sources, within and beyond the radius (262 columns, 65 rows)
    qry = {"x": np.repeat(src["x"], k) + rng.integers(-300, 301, n * k),
           "y": np.repeat(src["y"], k) + rng.integers(-70, 71, n * k),
           "t": np.repeat(src["t"], k), "p": np.repeat(src["p"], k) * rng.choice([-1, 1, 1, 1], n * k)}
    qry["x"], qry["y"] = np.clip(qry["x"], 0, W - 1), np.clip(qry["y"], 0, H - 1)
    got = B.nn_distances(Q.to_device(src), Q.to_device(qry), W, H, T, RMAX).cpu().numpy()
    s = {c: v.astype(np.float64) for c, v in src.items()}
    q = {c: v[:, None].astype(np.float64) for c, v in qry.items()}
    d = np.sqrt(((q["x"] - s["x"]) / W) ** 2 + ((q["y"] - s["y"]) / H) ** 2 + ((q["t"] - s["t"]) / T) ** 2)
    d = np.where(q["p"] == s["p"], d, np.inf).min(axis=1)
    edge = np.abs(d - RMAX) <= 1e-12
    want = np.where(d <= RMAX, d, np.inf)
    assert np.array_equal(np.isinf(got[~edge]), np.isinf(want[~edge]))
    fin = np.isfinite(want) & ~edge
    assert fin.any() and np.isinf(want).any() and np.max(np.abs(got[fin] - want[fin])) <= 1e-14
    torch.cuda.empty_cache()
