"""The performance cases of the event simulator: what a program that uses it
has it do, through its public entry points, on seeded synthetic clips.

A case is a dict of plain values.  Its ``kind`` names the call:

* ``convert``   one conversion of a clip by ``Simulator.enqueue`` (thresholded,
                exhaustive or raw; eager, or replayed from ``Simulator.capture``)
* ``batch``     the thresholded conversion of several clips in one plan
                (``BatchSimulator.enqueue``)
* ``regress``   one regression call: every pixel of a frame, or a work list of
                scattered pixels
* ``bandwidth`` the regression with the bandwidth chosen per pixel
* ``adjoint``   ``wlr_alpha`` and its gradients with respect to y and b
* ``compare``   ``quality.metrics`` of two event sets
* ``log``       ``log_brightness`` of a clip
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2303_02608_amd import autograd, quality, synth
from paper_2303_02608_amd import binding as B
from paper_2303_02608_amd.simulator import BatchSimulator, Simulator

TAUS = (5e-4, 2e-3, 5e-3, 1e-2)
HS = (0.5, 0.75, 1.0, 1.5, 2.0)
EPS = 1e-3


def listed():
    return [
        # the smallest clip of the repository (64x64x16, r = 5, one frame per window), converted eagerly:
        # every frame is a few launches over 4096 pixels
        dict(name="convert_small", kind="convert", mode="thresholded", W=64, H=64, T=16, F=7, spp=4, discs=3,
             r=5, tr=0, C=0.2, f16=False, threshold=0, multi=False, f32c=False, graph=False),
        # the DVS-scale clip (640x480, r = 7, three frames per window), converted by graph replays
        dict(name="convert_dvs", kind="convert", mode="thresholded", W=640, H=480, T=24, F=7, spp=8, discs=30,
             r=7, tr=1, C=0.15, f16=False, threshold=0, multi=False, f32c=False, graph=True),
        # WLR+ESIM, every pixel of every frame, at an odd size
        dict(name="convert_exhaustive", kind="convert", mode="exhaustive", W=501, H=403, T=6, F=7, spp=8,
             discs=24, r=7, tr=1, C=0.15, f16=False, threshold=0, multi=False, f32c=False, graph=False),
        # plain ESIM with every level crossing at a larger sensor: no regression, bound by memory and launches
        dict(name="convert_raw", kind="convert", mode="raw", W=1280, H=720, T=16, F=3, spp=4, discs=8, r=3, tr=0,
             C=0.3, f16=False, threshold=0, multi=True, f32c=False, graph=False),
        # clips of uneven sizes, lengths and window radii in one plan
        dict(name="convert_batch", kind="batch", clips=6, W=520, H=360, T=8, pick=11),
        # one work-list regression of scattered pixels with every output, at an odd size
        dict(name="regress_list", kind="regress", W=641, H=479, F=7, spp=8, discs=30, r=7, tr=1, share=0.06,
             f16=False, f32c=False),
        # the precision workload's window (r = 10, five frames, ten half-precision features), every pixel
        dict(name="regress_dense_f16", kind="regress", W=960, H=540, F=10, spp=4, discs=20, r=10, tr=2, share=1.0,
             f16=True, f32c=False),
        # its compensated single-precision Gram, on the flagged pixels of a 1920x1080 frame
        dict(name="regress_list_f32c", kind="regress", W=1920, H=1080, F=10, spp=4, discs=20, r=10, tr=2, share=0.04,
             f16=True, f32c=True),
        # bandwidth selection among five candidates, every pixel of a frame
        dict(name="bandwidth_dense", kind="bandwidth", W=480, H=360, F=7, spp=8, discs=20, r=7, tr=1, share=1.0,
             f16=False),
        # the differentiation loss: every pixel of frame 0 and scattered later regressions, forward and backward
        dict(name="adjoint_dvs", kind="adjoint", W=640, H=480, T=10, F=7, spp=8, discs=30, r=7, tr=1, share=0.06,
             f16=False),
        # the event-set comparison of a conversion against its reference
        dict(name="compare_dvs", kind="compare", W=640, H=480, T=120, n=1500000, extra=1.3),
        # log brightness of the whole DVS-scale clip
        dict(name="log_clip", kind="log", n=640 * 480 * 120),
    ]


def _spread(rng, lo, hi):
    """An integer of [lo, hi], spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("convert", "convert", "convert", "batch", "regress", "regress", "bandwidth", "adjoint",
                       "compare", "log"))
    top = max(_cost(c) for c in listed())
    while True:
        W, H = _spread(rng, 48, 1280), _spread(rng, 40, 720)
        F = rng.choice((3, 5, 7, 7, 7, 8, 10))
        spp = rng.choice((2, 4, 8))
        if kind == "convert":
            mode = rng.choice(("thresholded", "thresholded", "thresholded", "exhaustive", "raw"))
            c = dict(kind=kind, mode=mode, W=W, H=H, T=_spread(rng, 4, 40), F=F, spp=spp,
                     discs=rng.randint(2, 30), r=rng.randint(3, 10), tr=rng.randint(0, 2),
                     C=round(rng.uniform(0.12, 0.4), 3), f16=rng.random() < 0.3,
                     threshold=rng.choice((0, 0, 0, 1, 2)) if mode == "thresholded" else 0,
                     multi=mode != "thresholded" and rng.random() < 0.5,
                     f32c=F in (7, 10) and mode == "thresholded" and rng.random() < 0.15,
                     graph=rng.random() < 0.5)
        elif kind == "batch":
            c = dict(kind=kind, clips=rng.randint(2, 8), W=max(64, W // 2), H=max(64, H // 2), T=_spread(rng, 4, 16),
                     pick=rng.randint(0, 9999))
        elif kind == "regress":
            f32c = F in (7, 10) and rng.random() < 0.2
            c = dict(kind=kind, W=W, H=H, F=F, spp=spp, discs=rng.randint(2, 30), r=rng.randint(3, 12),
                     tr=rng.randint(0, 2), share=1.0 if rng.random() < 0.4 else round(rng.uniform(0.005, 0.4), 4),
                     f16=rng.random() < 0.5, f32c=f32c)
        elif kind == "bandwidth":
            c = dict(kind=kind, W=W, H=H, F=F, spp=spp, discs=rng.randint(2, 30), r=rng.randint(3, 9),
                     tr=rng.randint(0, 1), share=1.0 if rng.random() < 0.5 else round(rng.uniform(0.01, 0.3), 4),
                     f16=rng.random() < 0.3)
        elif kind == "adjoint":
            c = dict(kind=kind, W=W, H=H, T=_spread(rng, 3, 20), F=F, spp=spp, discs=rng.randint(2, 30),
                     r=rng.randint(3, 10), tr=rng.randint(0, 1), share=round(rng.uniform(0.01, 0.15), 4),
                     f16=rng.random() < 0.2)
        elif kind == "compare":
            c = dict(kind=kind, W=W, H=H, T=_spread(rng, 8, 120), n=_spread(rng, 2000, 1500000),
                     extra=round(rng.uniform(0.5, 1.5), 2))
        else:
            c = dict(kind=kind, n=_spread(rng, 4001, 640 * 480 * 120) | 1)
        if _cost(c) <= top and (kind in ("compare", "log") or _pixels(c) <= 8.5e6):
            return c


# ---- what a pass cannot do without ------------------------------------------

def _omega(c):
    return (2 * c["tr"] + 1) * (2 * c["r"] + 1) ** 2


def _fit_flops(c):
    """One regression: the normal equations over its window and their solve."""
    P, D = c["F"] + 3, c["F"] + 2
    return _omega(c) * (P * P + 4 * P + 4 * D) + P ** 3 / 3 + 2 * P * P


def _pixels(c):
    """Pixel-frames that the case holds."""
    if c["kind"] == "batch":
        return sum(W * H * T for W, H, T, _, _ in _batch_shapes(c))
    return c["W"] * c["H"] * c.get("T", 2 * c.get("tr", 0) + 1)


def work(case):
    c = case
    if c["kind"] == "log":
        return {"bytes": 8.0 * c["n"], "flops": 10.0 * c["n"]}
    if c["kind"] == "compare":
        nq = c["n"] + int(c["n"] * c["extra"])
        return {"bytes": 2 * 13.0 * nq + 8.0 * nq, "flops": 50.0 * nq}
    if c["kind"] == "batch":
        out = {"bytes": 0.0, "flops": 0.0}
        for W, H, T, r, _ in _batch_shapes(c):
            one = work(dict(kind="convert", mode="thresholded", W=W, H=H, T=T, F=7, r=r, tr=1, f16=False))
            out = {k: out[k] + one[k] for k in out}
        return out
    hw = c["W"] * c["H"]
    sample = 4 + c["F"] * (2 if c.get("f16") else 4)
    model = 4.0 * (2 * c["F"] + 2)
    if c["kind"] == "convert":
        T = c["T"]
        if c["mode"] == "raw":
            return {"bytes": (4.0 + 8.0) * hw * T, "flops": 4.0 * hw * T}
        fits = hw * (1 + 0.06 * (T - 1)) if c["mode"] == "thresholded" else float(hw * T)
        return {"bytes": hw * T * (sample + 4.0) + fits * model, "flops": fits * _fit_flops(c)}
    n = int(hw * c["share"]) if c["kind"] != "adjoint" else int(hw * (1 + c["share"] * (c["T"] - 1)))
    if c["kind"] == "adjoint":
        return {"bytes": c["T"] * hw * (sample + 4.0) + n * 16.0, "flops": n * (2 * _fit_flops(c) + 40.0 * _omega(c))}
    k = len(HS) if c["kind"] == "bandwidth" else 1
    return {"bytes": (2 * c["tr"] + 1) * hw * sample + n * 4.0 * (c["F"] + 5), "flops": k * n * _fit_flops(c)}


def _cost(c):
    w = work(c)
    return w["flops"] / 2e13 + w["bytes"] / 1e12 + (3e-9 * c["n"] if c["kind"] == "compare" else 0.0)


# ---- inputs ------------------------------------------------------------------

def _spec(c, seed, T):
    return synth.ClipSpec(W=c["W"], H=c["H"], T=T, spp=c["spp"], F=c["F"], n_discs=c["discs"], speed=(0.05, 0.4),
                          rim_speed=(0.05, 0.4), radius=(0.1, 0.25), disc_cell=2.5, motion_scale=10.0,
                          feat_dtype="f16" if c.get("f16") else "f32", seed=(seed * 7919 + 101) % 1000003)


def _clip(c, seed, T, variance=False):
    d = synth.make_clip(_spec(c, seed, T), device="cuda")
    y = B.log_brightness(d["E"], EPS)
    if variance:
        return y, d["feat"], B.log_variance(d["E"], d["var"], c["spp"], EPS)
    return y, d["feat"]


def _list(c, seed, hw):
    """A share of the pixels in ascending order, half of them in patches as flagged edges are."""
    g = np.random.default_rng(seed + 17)
    n = max(1, int(hw * c["share"]))
    if n >= hw:
        return None
    patch = (g.integers(0, hw, max(1, n // 16))[:, None] + np.arange(8)[None, :]).reshape(-1) % hw
    rest = g.choice(hw, n, replace=False)
    got = np.unique(np.concatenate([patch[:n // 2], rest]))
    return np.sort(g.permutation(got)[:n]).astype(np.int64)


def _batch_shapes(c):
    """(W, H, T, r, seed) of each clip: uneven, odd, radii on both sides of a 16-column window."""
    g = np.random.default_rng(c["pick"])
    return [(max(48, int(c["W"] * g.uniform(0.3, 1.0))), max(40, int(c["H"] * g.uniform(0.3, 1.0))),
             max(2, int(c["T"] * g.uniform(0.5, 1.0))), int(g.integers(5, 10)), k) for k in range(c["clips"])]


def _cleared(ev):
    """The event buffers with zeros past the last event, so that they can be compared whole."""
    for t in (ev.x, ev.y, ev.t, ev.p, ev.clip, ev.ts):
        if t is not None:
            t.zero_()
    return ev


def prepare(case, seed):
    c, s = case, dict(case=case)
    kind = c["kind"]
    if kind == "convert":
        s["y"], s["feat"] = _clip(c, seed, c["T"])
        p = B.Params(r=c["r"], tr=c["tr"], C=c["C"], precision=B.GRAM_F32C if c["f32c"] else B.GRAM_F64,
                     multi_crossing=c["multi"], threshold=c["threshold"], dt=1e-3)
        frac = {"thresholded": 0.25, "exhaustive": 0.3, "raw": 3.0 if c["multi"] else 1.0}[c["mode"]]
        s["sim"] = Simulator(s["y"], s["feat"], p, capacity=int(c["W"] * c["H"] * c["T"] * frac) + 1024)
        _cleared(s["sim"].ev)
        if c["graph"]:
            s["sim"].capture(c["mode"])
    elif kind == "batch":
        ys, feats, params = [], [], []
        for W, H, T, r, k in _batch_shapes(c):
            d = dict(W=W, H=H, F=7, spp=2 + k % 4, discs=6 + 3 * k)
            y, f = _clip(d, seed * 64 + k, T)
            ys.append(y)
            feats.append(f)
            params.append(B.Params(r=r, tr=1, C=0.15, dt=1e-3))
        total = sum(int(y.numel()) for y in ys)
        s["sim"] = BatchSimulator(ys, feats, params, capacity=total // 3 + 1024)
        _cleared(s["sim"].ev)
        s["clips"] = (ys, feats)
    elif kind in ("regress", "bandwidth"):
        T = 2 * c["tr"] + 1
        if kind == "bandwidth":
            s["y"], s["feat"], s["vy"] = _clip(c, seed, T, variance=True)
        else:
            s["y"], s["feat"] = _clip(c, seed, T)
        p = B.Params(r=c["r"], tr=c["tr"], C=0.15, precision=B.GRAM_F32C if c.get("f32c") else B.GRAM_F64)
        s["plan"] = B.Plan([s["y"]], [s["feat"]], [p])
        hw = c["W"] * c["H"]
        pix = _list(c, seed, hw)
        n = hw if pix is None else len(pix)
        s["pix"] = np.arange(hw, dtype=np.int64) if pix is None else pix
        s["items"] = None if pix is None else torch.from_numpy(pix).cuda()
        s["count"] = None if pix is None else torch.tensor([n, n], dtype=torch.int32, device="cuda")
        s["n"] = n
        s["alpha"] = torch.zeros(n, device="cuda")
        s["beta"] = torch.zeros((c["F"] + 2, n), device="cuda")
        s["a"] = torch.zeros(n, device="cuda")
        s["b"] = torch.zeros(n, device="cuda") if kind == "bandwidth" else None
    elif kind == "adjoint":
        s["y"], s["feat"] = _clip(c, seed, c["T"])
        hw = c["W"] * c["H"]
        t, pix = [np.zeros(hw, np.int64)], [np.arange(hw, dtype=np.int64)]
        for k in range(1, c["T"]):
            p = _list(c, seed * 131 + k, hw)
            t.append(np.full(len(p), k, np.int64))
            pix.append(p)
        s["t"], s["pix"] = np.concatenate(t), np.concatenate(pix)
        s["items"] = autograd.frame_items(torch.from_numpy(s["t"]), torch.from_numpy(s["pix"])).cuda()
        g = torch.Generator().manual_seed(seed + 5)
        s["g"] = torch.randn(len(s["pix"]), generator=g).cuda()
        s["y"].requires_grad_()
        s["bw"] = torch.ones(c["F"] + 2, dtype=torch.float64, device="cuda", requires_grad=True)
    elif kind == "compare":
        s["gen"], s["ref"] = _event_sets(c, seed)
    else:
        g = torch.Generator(device="cuda").manual_seed(seed)
        s["E"] = torch.empty(c["n"], device="cuda").exponential_(1.0, generator=g)
        s["out"] = torch.empty_like(s["E"])
    return s


def _event_sets(c, seed):
    """Events on the rims of moving discs: a reference, and a generated set displaced by up to a pixel and a frame."""
    g = torch.Generator(device="cuda").manual_seed(seed + 23)
    W, H, T = c["W"], c["H"], c["T"]
    cx, cy = (torch.rand(16, generator=g, device="cuda") * v for v in (W, H))
    R = (0.1 + 0.15 * torch.rand(16, generator=g, device="cuda")) * min(W, H)
    vx, vy = ((torch.rand(16, generator=g, device="cuda") - 0.5) * 0.8 for _ in range(2))

    def one(n, shift):
        k = torch.randint(0, 16, (n,), generator=g, device="cuda")
        t = torch.randint(0, T, (n,), generator=g, device="cuda")
        a = torch.rand(n, generator=g, device="cuda") * (2 * math.pi)
        rr = R[k] * (1.0 - 0.3 * torch.rand(n, generator=g, device="cuda") ** 3)
        x = cx[k] + vx[k] * t + rr * torch.cos(a) + shift * torch.randn(n, generator=g, device="cuda")
        y = cy[k] + vy[k] * t + rr * torch.sin(a) + shift * torch.randn(n, generator=g, device="cuda")
        x, y = x.to(torch.int64) % W, y.to(torch.int64) % H
        p = torch.where(torch.cos(a) * vx[k] + torch.sin(a) * vy[k] > 0, 1, -1)
        key, at = torch.sort((t * H + y) * W + x, stable=True)      # in the order a conversion emits them
        return {"x": (key % W).to(torch.int32), "y": (key // W % H).to(torch.int32),
                "t": (key // (W * H)).to(torch.int32), "p": p[at].to(torch.int8)}

    return one(int(c["n"] * c["extra"]), 0.7), one(c["n"], 0.0)


# ---- one pass ------------------------------------------------------------------

def run(state):
    s, c = state, state["case"]
    kind = c["kind"]
    if kind in ("convert", "batch"):
        sim = s["sim"]
        if kind == "batch":
            sim.enqueue()
        elif c["graph"]:
            sim.replay()
        else:
            sim.enqueue(c["mode"])
        ev = sim.ev
        out = {"count": ev.count, "x": ev.x, "y": ev.y, "t": ev.t, "p": ev.p, "dl": sim.dl}
        if ev.ts is not None:
            out["ts"] = ev.ts
        if ev.clip is not None:
            out["clip"] = ev.clip
        if kind == "batch" or c["mode"] == "thresholded":
            out["state"] = [[st.alpha, st.beta, st.xref, st.tref] for st in sim.plan.states]
        else:
            out["state"] = [st.alpha for st in sim.plan.states]
        return out
    if kind == "regress":
        B.regress(s["plan"], c["tr"], s["items"], s["count"], s["n"], s["alpha"], s["beta"], s["a"])
        return {"alpha": s["alpha"], "beta": s["beta"], "resid": s["a"]}
    if kind == "bandwidth":
        B.regress_bandwidth(s["plan"], c["tr"], s["items"], s["count"], s["n"], s["vy"], HS, s["alpha"], s["beta"],
                            s["a"], s["b"])
        return {"alpha": s["alpha"], "beta": s["beta"], "h": s["a"], "sure": s["b"]}
    if kind == "adjoint":
        alpha = autograd.wlr_alpha(s["y"], s["bw"], s["feat"], s["items"], c["r"], c["tr"])
        g_y, g_b = torch.autograd.grad(alpha, (s["y"], s["bw"]), s["g"])
        return {"alpha": alpha.detach(), "g_y": g_y, "g_b": g_b}
    if kind == "compare":
        return quality.metrics(s["gen"], s["ref"], c["W"], c["H"], c["T"], TAUS, 0.05, keep=True)
    return B.log_brightness(s["E"], EPS, out=s["out"])


# ---- the same in 64 bits, in plain torch -----------------------------------------

def _solve(A, R):
    """A x = R over a batch (A symmetric positive definite [n, P, P], R [n, P, m]) by elimination."""
    P = A.shape[1]
    M = torch.cat([A, R], dim=2)
    for k in range(P):
        row = M[:, k, :] / M[:, k, k, None]
        M = M - M[:, :, k, None] * row[:, None, :]
        M[:, k, :] = row
    return M[:, :, P:]


def _window(y, feat, t, pix, r, tr, h):
    """Regressors z [n, P, K], weights [n, K], y [n, K] and sample indices [n, K] of the regressions at (t, pix)."""
    T, F, H, W = feat.shape
    dev = y.device
    o = torch.arange(-r, r + 1, device=dev)
    dt = torch.arange(-tr, tr + 1, device=dev)
    k = len(dt) * len(o) ** 2
    dts = dt[:, None, None].expand(len(dt), len(o), len(o)).reshape(k)
    dys = o[None, :, None].expand(len(dt), len(o), len(o)).reshape(k)
    dxs = o[None, None, :].expand(len(dt), len(o), len(o)).reshape(k)
    st, sy, sx = t[:, None] + dts, (pix // W)[:, None] + dys, (pix % W)[:, None] + dxs
    ok = (st >= 0) & (st < T) & (sy >= 0) & (sy < H) & (sx >= 0) & (sx < W)
    st, sp = st.clamp(0, T - 1), sy.clamp(0, H - 1) * W + sx.clamp(0, W - 1)
    n = len(t)
    z = torch.empty((n, F + 3, k), dtype=torch.float64, device=dev)
    z[:, 0] = 1.0
    z[:, 1] = dxs.double() / r
    z[:, 2] = dys.double() / r
    flat = feat.reshape(T, F, H * W)
    for f in range(F):
        z[:, 3 + f] = flat[st, f, sp].double() - flat[t, f, pix].double()[:, None]
    w = torch.exp(-0.5 * (z[:, 1:] ** 2).sum(1) / (h * h)) * ok
    return z, w, y.reshape(T, H * W)[st, sp].double(), st * (H * W) + sp


def _fit(y, feat, t, pix, r, tr, h=1.0, ridge=1e-6):
    z, w, ys, at = _window(y, feat, t, pix, r, tr, h)
    P = z.shape[1]
    iw = 1.0 / w.sum(1)
    wz = z * (w * iw[:, None])[:, None, :]
    A = torch.bmm(wz, z.transpose(1, 2).contiguous())
    A[:, range(1, P), range(1, P)] += ridge
    rhs = torch.stack([(wz * ys[:, None, :]).sum(2), torch.zeros_like(A[:, 0])], dim=2)
    rhs[:, 0, 1] = 1.0
    x = _solve(A, rhs)
    return z, w, ys, at, iw, x[:, :, 0], x[:, :, 1]


def _chunks(c, n):
    m = max(1, int(3e7 / (_omega(c) * (c["F"] + 3))))
    return [(a, min(n, a + m)) for a in range(0, n, m)]


def exact(case, seed):
    c = case
    if c["kind"] in ("convert", "batch"):
        return None
    with torch.no_grad():
        if c["kind"] == "log":
            return torch.log(prepare(c, seed)["E"].double() + EPS)
        if c["kind"] == "compare":
            return _exact_compare(c, seed)
        s = prepare(c, seed)
        y, feat = s["y"].detach(), s["feat"]
        pix = torch.from_numpy(s["pix"]).cuda()
        n = len(pix)
        if c["kind"] == "adjoint":
            t = torch.from_numpy(s["t"]).cuda()
            alpha = torch.empty(n, dtype=torch.float64, device="cuda")
            g_y = torch.zeros(y.numel(), dtype=torch.float64, device="cuda")
            g_b = torch.zeros(c["F"] + 2, dtype=torch.float64, device="cuda")
            for a, b in _chunks(c, n):
                z, w, ys, at, iw, th, v = _fit(y, feat, t[a:b], pix[a:b], c["r"], c["tr"])
                alpha[a:b] = th[:, 0]
                gw = w * (s["g"][a:b].double() * iw)[:, None]
                cs = (v[:, :, None] * z).sum(1)
                res = ys - (th[:, :, None] * z).sum(1)
                g_y.index_add_(0, at.reshape(-1), (gw * cs).reshape(-1))
                vlt = 1e-6 * (v[:, 1:] * th[:, 1:]).sum(1)
                g_b += ((gw * (cs * res - vlt[:, None]))[:, None, :] * z[:, 1:] ** 2).sum((0, 2))
            return {"alpha": alpha, "g_y": g_y.reshape(y.shape), "g_b": g_b}
        t = torch.full((n,), c["tr"], dtype=torch.int64, device="cuda")
        D = c["F"] + 2
        alpha, extra, sure = (torch.empty(n, dtype=torch.float64, device="cuda") for _ in range(3))
        beta = torch.empty((D, n), dtype=torch.float64, device="cuda")
        for a, b in _chunks(c, n):
            if c["kind"] == "regress":
                z, w, ys, _, iw, th, _ = _fit(y, feat, t[a:b], pix[a:b], c["r"], c["tr"])
                res = ys - (th[:, :, None] * z).sum(1)
                extra[a:b] = (w * res * res).sum(1) * iw
            else:
                yc, vc = (q.reshape(q.shape[0], -1)[c["tr"], pix[a:b]].double() for q in (y, s["vy"]))
                best = torch.full((b - a,), math.inf, dtype=torch.float64, device="cuda")
                th, hsel = torch.zeros((b - a, D + 1), dtype=torch.float64, device="cuda"), torch.zeros_like(best)
                for h in HS:
                    *_, iw, x, v = _fit(y, feat, t[a:b], pix[a:b], c["r"], c["tr"], h)
                    risk = (x[:, 0] - yc) ** 2 + 2 * vc * v[:, 0] * iw - vc
                    take = risk < best
                    best = torch.where(take, risk, best)
                    th, hsel = torch.where(take[:, None], x, th), torch.where(take, torch.full_like(hsel, h), hsel)
                extra[a:b], sure[a:b] = hsel, best
            alpha[a:b], beta[:, a:b] = th[:, 0], th[:, 1:].T
        if c["kind"] == "regress":
            return {"alpha": alpha, "beta": beta, "resid": extra}
        return {"alpha": alpha, "beta": beta, "h": extra, "sure": sure}


def _exact_compare(c, seed):
    s = prepare(c, seed)
    W, H, T, rmax = c["W"], c["H"], c["T"], 0.05

    def nearest(src, qry):
        rx, ry, rt = (int(rmax * v) for v in (W, H, T))
        full = torch.zeros((2, T + 2 * rt, H + 2 * ry, W + 2 * rx), dtype=torch.bool, device="cuda")
        pl = lambda e: (e["p"] < 0).long()
        full[pl(src), src["t"].long() + rt, src["y"].long() + ry, src["x"].long() + rx] = True
        best = torch.full((qry["x"].numel(),), math.inf, dtype=torch.float64, device="cuda")
        p, t, y, x = pl(qry), qry["t"].long(), qry["y"].long(), qry["x"].long()
        base = ((p * (T + 2 * rt) + t) * (H + 2 * ry) + y) * (W + 2 * rx) + x
        flat = full.reshape(-1)
        offs = sorted((((dt / T) ** 2 + (dy / H) ** 2 + (dx / W) ** 2), dt, dy, dx) for dt in range(-rt, rt + 1)
                      for dy in range(-ry, ry + 1) for dx in range(-rx, rx + 1))
        live = torch.arange(len(base), device="cuda")
        for i, (d2, dt, dy, dx) in enumerate(offs):
            if math.sqrt(d2) > rmax or not len(live):
                break
            at = base[live] + ((dt + rt) * (H + 2 * ry) + dy + ry) * (W + 2 * rx) + dx + rx
            hit = flat[at]
            best[live[hit]] = math.sqrt(d2)
            if i < 64 or i % 64 == 0:
                live = live[torch.isinf(best[live])]
            else:
                live = live[~hit]
        return best

    dg, dr = nearest(s["ref"], s["gen"]), nearest(s["gen"], s["ref"])
    out = {"P": [], "R": [], "F": []}
    for tau in TAUS:
        P, R = (float((d < tau).double().mean()) for d in (dg, dr))
        out["P"].append(P)
        out["R"].append(R)
        out["F"].append(2 * P * R / (P + R) if P + R > 0 else 0.0)
    out["CD"] = float((dg.clamp(max=rmax) ** 2).mean() + (dr.clamp(max=rmax) ** 2).mean())
    out["dg"], out["dr"] = dg, dr
    return out
