"""Schedule autotuner of the regression kernels.

A plan's schedule (esim_plan_set_schedule) is the number of lanes that share one
regression item, in dense and in work-list launches, and the persistent blocks per
CU.  Until one is set, each clip takes what suits its size: one lane per pixel, or
16 where the frame would not fill the device.  16 lanes per item make short wave
tasks, for small frames and the sparse per-frame work lists of the thresholded path;
one lane per pixel shares the solve between 64 items and needs no sums over lanes.

The tuner replays a short prefix of the real conversion (frame 0 dense, then a few
thresholded frames) once per candidate and times only the regression launches with
HIP events on the launch stream.  The candidates run on a plan of their own; the
plan itself keeps its automatic schedule where no candidate is faster.  Blocks per
CU reach only the instances of one and two lanes that read their windows from
memory (FP64 Gram), up to the blocks that fit: other values are not tried again.
Results are cached per clip shape and parameters for the life of the process.
"""
from __future__ import annotations

from typing import Dict, Iterable, Optional, Tuple

import torch

from . import binding as B

# None: the automatic schedule
_cache: Dict[tuple, Optional[Tuple[int, int, int]]] = {}


def _key(plan: B.Plan, frames: int):
    parts = []
    for y, f, p in zip(plan.ys, plan.feats, plan.params):
        parts.append((tuple(f.shape), str(f.dtype), p.r, p.tr, p.C, p.precision))
    return (tuple(parts), frames, plan.schedule_set)


def _time_prefix(plan: B.Plan, frames: int, bufs) -> Tuple[float, float]:
    """Runs frame 0 (dense) and frames 1..frames-1 (thresholded) of every clip
    of the plan; returns (dense regress ms, summed work-list regress ms)."""
    dl, wl, cnt, a, b, ev = bufs
    n_out = a.numel()
    stream = torch.cuda.current_stream()
    ev.count.zero_()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record(stream)
    B.regress(plan, 0, None, None, n_out, a, b)
    e1.record(stream)
    B.events(plan, 0, B.INIT, None, alpha=a, beta=b, n_out=n_out)
    marks = []
    for t in range(1, frames):
        B.threshold(plan, t, dl, wl, cnt)
        s0, s1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        s0.record(stream)
        B.regress(plan, t, wl, cnt, n_out, a, b)
        s1.record(stream)
        marks.append((s0, s1))
        B.events(plan, t, B.THRESHOLDED, ev, worklist=wl, count=cnt, dl=dl, alpha=a, beta=b,
                 n_out=n_out)
    torch.cuda.synchronize()
    dense = e0.elapsed_time(e1)
    # the first frames flag few pixels; weigh the later ones
    lst = sum(x.elapsed_time(y) for x, y in marks[len(marks) // 2:])
    return dense, lst


def _trial(plan: B.Plan) -> B.Plan:
    """A plan over the same clips and states, for the candidates."""
    return B.Plan(plan.ys, plan.feats, plan.params, plan.states)


def _blocks(plan: B.Plan, blocks_per_cu: Iterable[int]) -> list:
    """The blocks per CU that make a difference: up to the resident ones."""
    resident = 2 if plan.F <= 8 and plan.params[0].precision == B.GRAM_F64 else 1
    return list({min(b, resident): b for b in reversed(list(blocks_per_cu))}.values())[::-1]


def tune(plan: B.Plan, frames: int = 12, lanes_dense: Iterable[int] = (1, 2, 4, 16),
         lanes_list: Iterable[int] = (4, 8, 16), blocks_per_cu: Iterable[int] = (1, 2, 4, 8),
         reps: int = 2, verbose: bool = False) -> Tuple[int, int, int]:
    """Pick (lanes_dense, lanes_list, blocks_per_cu) for the plan and apply it; returns
    ``plan.schedule`` where the plan keeps its automatic schedule.

    The plan's states are overwritten (the prefix is a real conversion)."""
    key = _key(plan, frames)
    if key in _cache:
        if _cache[key] is None:
            return plan.schedule
        plan.set_schedule(*_cache[key])
        return _cache[key]
    dev = plan.feats[0].device
    n_out = max(plan.npix, plan.wl_capacity)
    bufs = (torch.empty(plan.npix, dtype=torch.float32, device=dev),
            torch.empty(plan.wl_capacity, dtype=torch.int64, device=dev),
            torch.zeros(2, dtype=torch.int32, device=dev),
            torch.empty(n_out, dtype=torch.float32, device=dev),
            torch.empty((plan.D, n_out), dtype=torch.float32, device=dev),
            B.Events(1 << 16, dev))
    frames = max(2, min(frames, min(f.shape[0] for f in plan.feats)))
    # the later lists' mean time counts for every frame of the clip
    weight = (min(f.shape[0] for f in plan.feats) - 1) / max(1, (frames - 1) - (frames - 1) // 2)
    blocks = _blocks(plan, blocks_per_cu)
    lanes_dense, lanes_list = list(lanes_dense), list(lanes_list)
    trial = _trial(plan)

    def measure(what: str) -> Tuple[float, float]:
        _time_prefix(trial, frames, bufs)           # warm-up
        best = (float("inf"), float("inf"))
        for _ in range(reps):
            best = tuple(min(v) for v in zip(best, _time_prefix(trial, frames, bufs)))
        if verbose:
            print(f"[autotune] {what}: dense {best[0]:.3f} ms, list {best[1]:.3f} ms", flush=True)
        return best

    own = None if plan.schedule_set else measure("automatic")
    # along the lines through (., 16, .) and (1, ., first blocks) only
    runs = [(ld, 16, b) for ld in lanes_dense for b in (blocks if ld <= 2 else blocks[:1])]
    runs += [(lanes_dense[0], ll, b) for ll in lanes_list if ll != 16 for b in (blocks if ll <= 2 else blocks[:1])]
    dense: Dict[Tuple[int, int], float] = {}
    lists: Dict[Tuple[int, int], float] = {}
    for ld, ll, b in runs:
        try:
            trial.set_schedule(ld, ll, b)
        except B.EsimError:
            continue          # no kernel instance for this combination
        d, l = measure(f"dense L={ld} list L={ll} blocks={b}")
        for table, lanes, v in ((dense, ld, d), (lists, ll, l)):
            for at in ([b] if lanes <= 2 else blocks):          # what the blocks do not reach holds for all
                table[(lanes, at)] = min(table.get((lanes, at), float("inf")), v)
    best = None
    for b in blocks:
        ds = [(v, L) for (L, at), v in dense.items() if at == b]
        ls = [(v, L) for (L, at), v in lists.items() if at == b and L in lanes_list]
        if ds and ls:
            total = min(ds)[0] + min(ls)[0] * weight
            if best is None or total < best[0]:
                best = (total, (min(ds)[1], min(ls)[1], b))
    # (a candidate that repeats the automatic choice differs by noise)
    if own is not None and (best is None or own[0] + own[1] * weight <= 1.02 * best[0]):
        _cache[key] = None
        return plan.schedule
    _cache[key] = best[1]
    plan.set_schedule(*best[1])
    return best[1]
