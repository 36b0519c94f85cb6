"""Whole runs of several contexts at once, on streams of their own and from threads of their own:
every field is what one context alone computes, for plans that fill the chip and plans that fit
beside each other, with and without a graph, with a capture of the caller's in between, and after a
context has gone."""
import threading

import numpy as np
import pytest

from paper_2301_05518_amd import synth
from tests.gpu_common import log, to_dev

pytestmark = pytest.mark.gpu

CASES = [((32, 32, 24, 1), "f32"), ((16, 12, 8, 1), "f32"), ((32, 24, 20, 1), "f64"), ((24, 24, 24, 2), "bf16")]


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


class Worker:
    def __init__(self, torch, k, flags):
        import paper_2301_05518_amd as tl
        L, prec = CASES[k % len(CASES)]
        ts = [t for t in range(L[3]) for _ in range(3)]
        U = synth.gauge_field(L, "haar", 9970 + k)
        self.torch, self.stream, self.runs = torch, torch.cuda.Stream(), 12
        with torch.cuda.stream(self.stream):
            self.c = tl.Context(0, self.stream)
            self.src = to_dev(synth.random_field(np.random.default_rng([9970, k]), (len(ts), L[2], L[1], L[0], 3)))
            self.job = tl.Job(L, self.c.build_twolinks(L, to_dev(U), prec), ts, self.src.clone())
            self.plan = self.c.plan([self.job], 20, 2.0, prec, flags)
            assert self.plan.info()["variant"] == 9
            self.c.sync()

    def go(self):
        """`runs` runs in a row from the sources, without waiting in between; the smeared fields."""
        with self.torch.cuda.stream(self.stream):
            self.job.psi.copy_(self.src)
            self.plan.load()
            for _ in range(self.runs):
                self.plan.run()
            self.plan.store()
            self.out = self.job.psi.clone()

    def close(self):
        self.plan.close()
        self.c.close()


@pytest.mark.parametrize("threads", [False, True])
@pytest.mark.parametrize("graph", [False, True])
def test_contexts_at_once(torch, graph, threads):
    import paper_2301_05518_amd as tl
    workers = [Worker(torch, k, tl.TL_GRAPH if graph else 0) for k in range(4)]
    want = []
    for w in workers:         # one after the other
        w.go()
        torch.cuda.synchronize()
        want.append(w.out)
    for rep in range(4):
        log(f"contexts at once: graph {graph} threads {threads} rep {rep}, {len(workers)} contexts")
        if threads:
            ts = [threading.Thread(target=w.go) for w in workers]
            for t in ts:
                t.start()
            for t in ts:
                t.join()
        else:
            for w in workers:
                w.go()
        for w in workers:
            w.c.sync()
        for w, x in zip(workers, want):
            assert torch.equal(w.out, x), rep
        if rep == 2:          # the others go on
            workers.pop(0).close()
            want.pop(0)
    for w in workers:
        w.close()


def test_capture_beside_another_context(torch):
    a, b = Worker(torch, 0, 0), Worker(torch, 2, 0)
    for w in (a, b):
        w.go()
    torch.cuda.synchronize()
    want = a.out.clone(), b.out.clone()
    g = torch.cuda.CUDAGraph()
    b.go()                    # in flight while a's stream is captured
    with torch.cuda.graph(g, stream=a.stream):
        a.go()
    for rep in range(3):
        b.go()
        g.replay()
        b.go()
        a.stream.synchronize()
        b.stream.synchronize()
        assert torch.equal(a.out, want[0]) and torch.equal(b.out, want[1]), rep
        a.go()
        a.c.sync()
        assert torch.equal(a.job.psi, want[0]), rep
        a.out = want[0] if rep else a.out
    a.close()
    b.close()
