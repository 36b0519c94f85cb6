"""Whole runs end in the resident buffer in which n one-step launches end: replays of a captured
tl_plan_run of an even number of steps advance the field each time, for every way the whole-run
kernel cuts the lattice (one-tile cells, cut ones, threads per RHS, a team too small for its cell),
and give the one-step launches' bits.  An odd number of steps ends in the other buffer; its captured
run is replayed once (one-step launches leave step n - 1 in the buffer that it reads)."""
import numpy as np
import pytest

from paper_2301_05518_amd import synth
from tests.gpu_common import log, to_dev

pytestmark = pytest.mark.gpu

DIRECT = "0,64,1,0"
TILES = [None, "9,512,32,0,0,0", "9,256,64,0,0,1", "9,512,64,8,0,0"]


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


def replays(torch, monkeypatch, tile, prec, n, count):
    """The fields after `count` replays of one captured run, and after one more eager run."""
    import paper_2301_05518_amd as tl
    if tile:
        monkeypatch.setenv("TL_TILE", tile)
    else:
        monkeypatch.delenv("TL_TILE", raising=False)
    side = torch.cuda.Stream()
    c = tl.Context(0, side)
    jobs = []
    with torch.cuda.stream(side):
        for L, ts in (((4, 6, 4, 2), [0, 1, 1]), ((32, 24, 20, 1), [0, 0, 0]), ((14, 9, 16, 1), [0, 0])):
            U = synth.gauge_field(L, "haar", 9300)
            psi = synth.random_field(np.random.default_rng([9300, *L]), (len(ts), L[2], L[1], L[0], 3))
            jobs.append(tl.Job(L, c.build_twolinks(L, to_dev(U), prec), ts, to_dev(psi)))
        plan = c.plan(jobs, n, 0.4 * n, prec)
        plan.load()
        plan.run()
        plan.run()          # an even number of runs: the field is in the first buffer again
        side.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            plan.run()
        for _ in range(count):
            g.replay()
        plan.store()
        side.synchronize()
        out = [j.psi.clone() for j in jobs]
        plan.run()
        plan.store()
        side.synchronize()
        out += [j.psi.clone() for j in jobs]
        variant = plan.info()["variant"]
    plan.close()
    c.close()
    return variant, out


@pytest.mark.parametrize("prec,n", [("f32", 6), ("f64", 4), ("bf16", 6), ("f16s", 4), ("f32", 5)])
def test_replays_advance_the_field(torch, monkeypatch, prec, n):
    count = 1 if n % 2 else 3
    _, one = replays(torch, monkeypatch, DIRECT, prec, n, 1)
    _, want = replays(torch, monkeypatch, DIRECT, prec, n, count)
    assert torch.equal(one[1], want[1]) == (count == 1)     # the field moves on with each replay
    for tile in TILES:
        variant, got = replays(torch, monkeypatch, tile, prec, n, count)
        log(f"{prec} n={n} tile {tile}: variant {variant}")
        assert variant == 9
        for a, b in zip(got, want):
            assert torch.equal(a, b), tile
