"""The dense instances of the bandwidth selection, by one lane per pixel: tiles from
LDS and, for windows too wide for it, from memory; every default small frame of the
other bandwidth tests runs 16 lanes per item.  Compared with the oracle as there:
alpha and beta of the chosen candidate to 1e-4 max(1, |.|); where the choice differs
from the oracle's, the oracle's SURE at it within 1e-5 + 1e-4 |SURE_min| of the
minimum, and rarely."""
import numpy as np
import pytest
import torch

import oracle
from paper_2303_02608_amd import binding as B
from paper_2303_02608_amd import synth
from parity_util import say

pytestmark = pytest.mark.gpu

HS = [0.5, 0.75, 1.0, 1.5, 2.0]
HS8 = [1.0, 0.4, 2.5, 0.7, 1.8, 0.55, 1.25, 3.2]


def _clip(W, H, T, F, f16, seed):
    d = synth.random_features_clip(W, H, T, F, seed=seed, feat_dtype="f16" if f16 else "f32")
    rng = np.random.default_rng(seed)
    E = d["E"].numpy()
    return E, (E ** 2 * rng.uniform(0.2, 2.0, size=E.shape)).astype(np.float32), d["feat"].numpy()


def _gpu(E, var, feat, p, t, hs, schedule, items=None):
    y = B.log_brightness(torch.from_numpy(E).cuda())
    vy = B.log_variance(torch.from_numpy(E).cuda(), torch.from_numpy(var).cuda(), 4)
    plan = B.Plan([y], [torch.from_numpy(feat).cuda()], [p])
    if schedule:
        plan.set_schedule(*schedule)
    n = plan.npix if items is None else len(items)
    a, h, s = (torch.full((n,), 7.0, device="cuda") for _ in range(3))
    b = torch.full((plan.D, n), 7.0, device="cuda")
    wl = cnt = None
    if items is not None:
        wl = torch.from_numpy(np.asarray(items, np.int64)).cuda()
        cnt = torch.tensor([n, n], dtype=torch.int32, device="cuda")
    B.regress_bandwidth(plan, t, wl, cnt, n, vy, hs, a, b, h, s)
    torch.cuda.synchronize()
    return [v.cpu().numpy() for v in (a, b, h, s)]


def _compare(got, o, hs, tag):
    a, b, h, s = got
    hs = np.asarray(hs)
    kg = np.argmin(np.abs(hs[None, :] - h.astype(np.float64)[:, None]), axis=1)
    assert np.all(np.abs(hs[kg] - h) <= 1e-6 * hs[kg])
    rows = np.arange(len(a))
    so, sm = o["sure"][rows, kg], o["sure"].min(axis=1)
    flips = kg != np.argmin(o["sure"], axis=1)
    say(f"{tag}: {flips.sum()} of {len(a)} choices differ")
    assert np.all(so - sm <= 1e-5 + 1e-4 * np.abs(sm)) and flips.mean() <= 0.01
    ao = o["alpha_k"][rows, kg]
    assert np.max(np.abs(a - ao) / np.maximum(1, np.abs(ao))) <= 1e-4
    assert np.max(np.abs(s - so) / np.maximum(1e-3, np.abs(so))) <= 1e-3
    bo, bg = o["theta"][~flips, 1:], b.T[~flips]
    assert np.max(np.abs(bg - bo) / np.maximum(1, np.abs(bo))) <= 1e-4


@pytest.mark.parametrize("W,H,T,F,r,tr,t,f16,hs,precision", [
    (64, 20, 3, 7, 7, 1, 1, False, HS, B.GRAM_F64),       # whole 64 x 1 tiles
    (65, 7, 3, 7, 5, 1, 0, True, HS, B.GRAM_F64),         # partial tiles, the clip's first frame
    (41, 23, 5, 3, 3, 2, 4, False, HS8, B.GRAM_F64),      # eight candidates, its last frame
    (33, 17, 1, 1, 4, 0, 0, False, HS, B.GRAM_F64),       # one frame
    (50, 11, 5, 8, 5, 2, 1, False, HS, B.GRAM_F64),       # four frames
    (47, 19, 5, 10, 4, 2, 2, True, HS, B.GRAM_F64),       # one wave per SIMD: rows loaded ahead
    (35, 13, 3, 12, 3, 1, 1, False, HS, B.GRAM_F64),      # frame by frame
    (34, 12, 3, 12, 3, 1, 1, True, HS8, B.GRAM_F64),
    (38, 14, 3, 7, 4, 1, 1, False, HS, B.GRAM_F32C),      # the selection's Gram is FP64 whatever the plan's
    (23, 9, 3, 7, 57, 1, 1, False, HS, B.GRAM_F64),       # rows of more than two turns of a wave: from memory
    (21, 8, 5, 8, 57, 2, 2, True, HS, B.GRAM_F64),
    (19, 9, 3, 12, 60, 0, 1, False, HS8, B.GRAM_F64),
    (5, 61, 3, 7, 4, 1, 1, False, HS, B.GRAM_F64),        # narrow: from memory
])
def test_dense_one_lane_per_pixel(W, H, T, F, r, tr, t, f16, hs, precision):
    tag = f"dense bandwidth {W}x{H} F={F} r={r} tr={tr} t={t} f16={f16} K={len(hs)}"
    say(tag)
    E, var, feat = _clip(W, H, T, F, f16, 700 + F + r)
    p = B.Params(r=r, tr=tr, C=0.1, precision=precision)
    schedule = (1, 16, 2) if precision == B.GRAM_F64 else (4, 16, 4)
    got = _gpu(E, var, feat, p, t, hs, schedule)
    vy = oracle.log_variance(E, var, 4)
    o = oracle.regress_bandwidth(oracle.Clip(oracle.log_brightness(E), feat), oracle.Params(r, tr, 0.1), np.asarray(hs),
                                 vy, t * W * H + np.arange(W * H))
    order = np.argsort(hs)
    o = dict(o, sure=o["sure"][:, order], alpha_k=o["alpha_k"][:, order])
    _compare(got, o, np.asarray(hs)[order], tag)


@pytest.mark.parametrize("r", [5, 8])
def test_lists_agree_with_dense(r):
    """Two instances with sums of another order: the same choices and values to
    summation-order rounding."""
    say(f"bandwidth lists and dense tiles r={r}")
    E, var, feat = _clip(70, 31, 3, 7, False, 750 + r)
    p = B.Params(r=r, tr=1, C=0.1)
    pix = np.arange(3, 70 * 31, 7)
    d = _gpu(E, var, feat, p, 1, HS, (1, 16, 2))
    g = _gpu(E, var, feat, p, 1, HS, None, items=pix)
    same = g[2] == d[2][pix]
    assert same.mean() >= 0.99
    assert np.allclose(g[0][same], d[0][pix][same], rtol=1e-5, atol=1e-5)
