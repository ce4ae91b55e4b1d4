"""A clip's regressions, events and state do not depend on the other clips of its
plan: whatever instance it takes alone (tiles, 16 lanes per item with whole or cut
columns, windows from memory), it takes in a batch, so that every output is equal
bit for bit, by the default schedule and by the ones set by hand."""
import numpy as np
import pytest
import torch

from paper_2303_02608_amd import binding as B
from paper_2303_02608_amd import synth
from paper_2303_02608_amd.simulator import BatchSimulator, Simulator
from parity_util import say, to_dev

pytestmark = pytest.mark.gpu

# W, H, T, r, tr: small and large frames, windows of cut and of whole columns, of
# five frames, of 16-column tiles, and from memory (too wide for LDS; narrow images)
SHAPES = {
    "sizes": [(240, 200, 3, 5, 1), (300, 260, 3, 5, 1), (64, 9, 2, 5, 0)],
    "radii": [(60, 50, 3, 3, 1), (240, 200, 3, 7, 1), (133, 140, 3, 9, 1)],
    "narrow": [(240, 200, 3, 3, 1), (52, 31, 3, 7, 1)],
    "frames": [(140, 130, 5, 5, 2), (240, 200, 5, 5, 1), (52, 31, 2, 5, 0)],
    "tile widths": [(300, 260, 1, 5, 0), (300, 240, 1, 33, 0), (290, 250, 1, 6, 0)],
    "memory": [(300, 260, 1, 5, 0), (300, 240, 1, 57, 0), (5, 14000, 1, 6, 0), (70, 60, 1, 8, 0)],
}


def _clips(name, f16=False):
    out = []
    for i, (W, H, T, r, tr) in enumerate(SHAPES[name]):
        d = synth.make_clip(synth.ClipSpec(W=W, H=H, T=T, spp=4, F=7, n_discs=8, speed=(0.5, 2.0), seed=900 + i,
                                           feat_dtype="f16" if f16 else "f32"))
        out.append(to_dev(d["E"].numpy(), d["feat"].numpy()) + (B.Params(r=r, tr=tr, C=0.05),))
    return out


def _regress(clips, t, lists, schedule):
    plan = B.Plan([y for y, *_ in clips], [f for _, f, _ in clips], [p for *_, p in clips])
    if schedule:
        plan.set_schedule(*schedule)
    items = cnt = None
    n = plan.npix
    if lists:
        items = torch.cat([(c << 32) + torch.arange(y[0].numel()) for c, (y, *_) in enumerate(clips)]).cuda()
        n = items.numel()
        cnt = torch.tensor([n, n], dtype=torch.int32, device="cuda")
    a, b, R = torch.full((n,), 7.0, device="cuda"), torch.full((plan.D, n), 7.0, device="cuda"), \
        torch.full((n,), 7.0, device="cuda")
    B.regress(plan, t, items, cnt, n, a, b, R)
    torch.cuda.synchronize()
    return [v.cpu().numpy() for v in (a, b, R)]


@pytest.mark.parametrize("schedule", [None, (1, 16, 2), (16, 4, 1)])
@pytest.mark.parametrize("lists", [False, True])
@pytest.mark.parametrize("name", sorted(SHAPES))
def test_regressions(name, lists, schedule):
    say(f"bits of {name} lists={lists} schedule={schedule}")
    clips = _clips(name, f16=name == "frames")
    t = min(y.shape[0] for y, *_ in clips) - 1
    got = _regress(clips, t, lists, schedule)
    off = 0
    for clip in clips:
        alone = _regress([clip], t, lists, schedule)
        n = alone[0].size
        for g, w in zip(got, alone):
            assert np.array_equal(g[..., off:off + n], w)
        off += n


@pytest.mark.parametrize("threshold", [B.THRESHOLD_CLOSED, B.THRESHOLD_LAST_WINDOW])
def test_conversion(threshold):
    """Events and final state of the steps (frame 0, then split or filtered lists)."""
    say(f"bits of a batch conversion, threshold {threshold}")
    clips = []
    for i, (W, H, T, r, tr) in enumerate([(64, 48, 6, 3, 1), (280, 250, 6, 5, 1), (70, 64, 5, 9, 1), (64, 50, 6, 7, 2)]):
        d = synth.make_clip(synth.ClipSpec(W=W, H=H, T=T, spp=4, F=7, n_discs=5, speed=(0.5, 2.0), seed=950 + i))
        clips.append(to_dev(d["E"].numpy(), d["feat"].numpy()) + (B.Params(r=r, tr=tr, C=0.2, threshold=threshold),))
    bs = BatchSimulator([y for y, *_ in clips], [f for _, f, _ in clips], [p for *_, p in clips])
    got = bs.run()
    assert got["count"] > 0
    for c, (y, f, p) in enumerate(clips):
        sim = Simulator(y, f, p)
        one = sim.run("thresholded")
        m = got["clip"] == c
        for k in ("x", "y", "t", "p"):
            assert np.array_equal(got[k][m], one[k]), (c, k)
        for k in ("alpha", "beta", "xref", "tref"):
            assert torch.equal(getattr(bs.plan.states[c], k), getattr(sim.state, k)), (c, k)
