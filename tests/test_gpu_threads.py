"""Dense launches of plans with different amounts of LDS from several threads at
once, each on a stream of its own: every launch gets the LDS of its own plan."""
import threading

import pytest
import torch

from paper_2303_02608_amd import binding as B
from paper_2303_02608_amd import synth
from parity_util import say, to_dev

pytestmark = pytest.mark.gpu


def test_tiles_of_different_lds_from_several_threads():
    say("tiles from three threads")
    plans = []
    for r, tr in ((10, 1), (3, 1), (7, 1)):              # 129, 79 and 108 KB a block
        d = synth.random_features_clip(130, 40, 3, 7, 30 + r)
        y, f = to_dev(d["E"].numpy(), d["feat"].numpy())
        p = B.Plan([y], [f], [B.Params(r=r, tr=tr, C=0.2)])
        p.set_schedule(1, 16, 2)
        plans.append(p)

    def run(p, stream, n, out):
        with torch.cuda.stream(stream):
            for _ in range(n):
                a = torch.empty(p.npix, device="cuda")
                b = torch.empty((p.D, p.npix), device="cuda")
                B.regress(p, 1, None, None, p.npix, a, b)
                out.append((a, b))
        stream.synchronize()

    want = []
    for p in plans:
        one = []
        run(p, torch.cuda.current_stream(), 1, one)
        want.append(one[0])
    outs = [[] for _ in plans]
    threads = [threading.Thread(target=run, args=(p, torch.cuda.Stream(), 40, o)) for p, o in zip(plans, outs)]
    torch.cuda.synchronize()
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for w, o in zip(want, outs):
        assert len(o) == 40
        for a, b in o:
            assert torch.equal(a, w[0]) and torch.equal(b, w[1])
