"""GPU parity of the regression's work distribution: dense tiles (their widths,
partial tiles, frame groups and the windows that do not fit), and the work-list
instances (groups, rounds, lanes per item, items of different frames in a wave).

Tolerances: the contract's, 1e-4 * max(1, |.|) on alpha and beta and 1e-6 on R;
the random features keep every window well conditioned."""
import numpy as np
import pytest
import torch

import oracle
from paper_2303_02608_amd import binding as B
from paper_2303_02608_amd import synth
from parity_util import oracle_clip, say, to_dev

pytestmark = pytest.mark.gpu


def _clip(W, H, T, F, seed, f16=False):
    d = synth.random_features_clip(W, H, T, F, seed, feat_dtype="f16" if f16 else "f32")
    return d["E"].numpy(), d["feat"].numpy()


def _compare(a, b, R, ref, tag):
    th = ref["theta"]
    ea = np.abs(a - th[:, 0]) / np.maximum(1.0, np.abs(th[:, 0]))
    eb = np.abs(b.T - th[:, 1:]) / np.maximum(1.0, np.abs(th[:, 1:]))
    er = np.abs(R - ref["R"])
    say(f"{tag}: alpha {ea.max():.1e} beta {eb.max():.1e} R {er.max():.1e}")
    assert ea.max() <= 1e-4 and eb.max() <= 1e-4 and er.max() <= 1e-6, tag


def _run(plan, t, items, n, cnt=None):
    a = torch.full((n,), 7.0, device="cuda")
    b = torch.full((plan.D, n), 7.0, device="cuda")
    R = torch.full((n,), 7.0, device="cuda")
    B.regress(plan, t, items, cnt, n, a, b, R)
    torch.cuda.synchronize()
    return a.cpu().numpy(), b.cpu().numpy(), R.cpu().numpy()


@pytest.mark.parametrize("W,H,T,F,r,tr,t,f16", [
    (64, 9, 3, 7, 7, 1, 1, False),      # one column of whole 64 x 1 tiles
    (65, 7, 3, 7, 3, 1, 1, False),      # 16 x 4 tiles, partly outside both ways
    (33, 20, 1, 5, 2, 0, 0, False),     # one frame
    (97, 11, 3, 4, 5, 1, 0, True),      # 32 x 2 tiles, two frames
    (17, 19, 5, 7, 4, 2, 2, False),     # five frames
    (48, 5, 5, 8, 5, 2, 1, False),      # four frames, three quads of channels
    (80, 6, 5, 10, 6, 2, 2, True),      # one wave per SIMD: rows loaded ahead
    (40, 21, 7, 3, 2, 3, 3, False),     # seven frames: groups of five and two
    (33, 9, 5, 11, 3, 2, 2, False),     # eleven channels: three frames at a time, here one by one
    (34, 8, 3, 12, 2, 1, 1, True),      # twelve: always one
    (30, 34, 2, 7, 33, 0, 1, False),    # rows wider than two turns of a wave: no tiles
])
def test_dense_tiles(W, H, T, F, r, tr, t, f16):
    tag = f"tiles {W}x{H} T={T} F={F} r={r} tr={tr} t={t} f16={f16}"
    say(tag)
    E, feat = _clip(W, H, T, F, 70 + W, f16)
    p = B.Params(r=r, tr=tr, C=0.2, h=1.2)
    y, fd = to_dev(E, feat)
    plan = B.Plan([y], [fd], [p])
    plan.set_schedule(1, 16, 2)          # a frame this small takes 16 lanes per item by itself
    got = _run(plan, t, None, W * H)
    ref = oracle.regress_items(oracle_clip(E, feat), oracle.Params(r, tr, 0.2, 1.2), t * W * H + np.arange(W * H),
                               kappa=False)
    _compare(*got, ref, tag)


def test_dense_tiles_of_several_clips():
    """Tiles of clips of different widths, radii and lengths in one launch; the
    clip that has ended writes nothing."""
    say("tiles of three clips")
    shapes = [(70, 9, 4, 3), (31, 12, 2, 5), (20, 33, 4, 2)]
    clips = [_clip(W, H, T, 7, 300 + i) for i, (W, H, T, _) in enumerate(shapes)]
    devs = [to_dev(*c) for c in clips]
    plan = B.Plan([y for y, _ in devs], [f for _, f in devs],
                  [B.Params(r=r, tr=1, C=0.2) for *_, r in shapes])
    plan.set_schedule(1, 16, 2)
    a, b, R = _run(plan, 2, None, plan.npix)
    for k, (W, H, T, r) in enumerate(shapes):
        s = slice(plan.offsets[k], plan.offsets[k] + W * H)
        if T <= 2:
            assert np.all(a[s] == 7.0) and np.all(b[:, s] == 7.0)
            continue
        ref = oracle.regress_items(oracle_clip(*clips[k]), oracle.Params(r, 1, 0.2), 2 * W * H + np.arange(W * H),
                                   kappa=False)
        _compare(a[s], b[:, s], R[s], ref, f"clip {k}")


@pytest.mark.parametrize("lanes", [4, 8, 16])
@pytest.mark.parametrize("r,tr", [(7, 1), (8, 1), (3, 2), (1, 1), (12, 0)])
def test_work_lists(lanes, r, tr):
    """Lists shorter than a group, around a wave's and a block's share and longer
    than one round of every CU, each item at a frame of its own (windows cut by
    both clip ends among them)."""
    W, H, T = 41, 23, 4
    E, feat = _clip(W, H, T, 7, 500 + r)
    y, fd = to_dev(E, feat)
    plan = B.Plan([y], [fd], [B.Params(r=r, tr=tr, C=0.2)])
    plan.set_schedule(lanes, lanes, 2)
    ref = oracle.regress_items(oracle_clip(E, feat), oracle.Params(r, tr, 0.2), np.arange(T * W * H), kappa=False)
    rng = np.random.default_rng(lanes)
    for n in (1, 3, 64 // lanes + 1, 129, 1025, 70001):
        t, pix = rng.integers(0, T, n), rng.integers(0, W * H, n)
        items = torch.from_numpy((t << 44) | pix).cuda()
        cnt = torch.tensor([n, n], dtype=torch.int32, device="cuda")
        got = _run(plan, -1, items, n, cnt)
        k = t * W * H + pix
        _compare(*got, {"theta": ref["theta"][k], "R": ref["R"][k]}, f"list of {n}, lanes {lanes}, r={r} tr={tr}")


@pytest.mark.parametrize("r,tr,f16", [(1, 1, False), (2, 1, True), (7, 0, False), (8, 2, False), (9, 1, True),
                                      (11, 1, False), (16, 0, False), (23, 1, False)])
def test_small_dense_frames(r, tr, f16):
    """Frames that would not fill the chip with tiles, by the default schedule:
    whole columns, and leftover columns cut into 16, 5, 3, 2 and 1 parts."""
    W, H, T = 23, 14, 3
    tag = f"dense {W}x{H} r={r} tr={tr} f16={f16}"
    say(tag)
    E, feat = _clip(W, H, T, 4, 40 + r, f16)
    p = B.Params(r=r, tr=tr, C=0.2)
    y, fd = to_dev(E, feat)
    got = _run(B.Plan([y], [fd], [p]), 1, None, W * H)
    ref = oracle.regress_items(oracle_clip(E, feat), oracle.Params(r, tr, 0.2), W * H + np.arange(W * H), kappa=False)
    _compare(*got, ref, tag)


def test_work_list_longer_than_its_outputs():
    """The device count is clamped to the outputs; an empty list writes nothing."""
    say("clamped and empty lists")
    E, feat = _clip(40, 20, 3, 7, 9)
    y, fd = to_dev(E, feat)
    plan = B.Plan([y], [fd], [B.Params(r=5, tr=1, C=0.2)])
    items = torch.arange(700, dtype=torch.int64, device="cuda")
    full = _run(plan, 1, items, 700, torch.tensor([700, 0], dtype=torch.int32, device="cuda"))
    cut = _run(plan, 1, items, 333, torch.tensor([700, 0], dtype=torch.int32, device="cuda"))
    assert np.array_equal(cut[0], full[0][:333]) and np.array_equal(cut[1], full[1][:, :333])
    none = _run(plan, 1, items, 333, torch.tensor([0, 0], dtype=torch.int32, device="cuda"))
    assert np.all(none[0] == 7.0) and np.all(none[1] == 7.0) and np.all(none[2] == 7.0)
