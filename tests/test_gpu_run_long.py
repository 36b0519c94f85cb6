"""Runs of more steps than a whole-run launch takes (32768 per unit of a team's share): several
launches, bit for bit the one-step launches' result, with a remainder, with several units per
share, and with members that have no tile of the smaller lattice's units."""
import numpy as np
import pytest

from paper_2301_05518_amd import synth
from tests.gpu_common import log, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_long_runs(torch, monkeypatch, prec):
    import paper_2301_05518_amd as tl
    n = 32768 + 3
    c = tl.Context(0)
    lats = []
    for L, ts in (((12, 16, 8, 1), [0, 0]), ((4, 6, 4, 2), [0, 1])):
        U = synth.gauge_field(L, "haar", 9500)
        src = to_dev(synth.random_field(np.random.default_rng([9500, *L]), (len(ts), L[2], L[1], L[0], 3)))
        lats.append((L, c.build_twolinks(L, to_dev(U), prec), ts, src))
    outs = {}
    for tile in ("0,64,4,0", "9,512,8,0,0,1", "9,64,4,8,0,0"):     # the last: two teams, 12 units a share
        monkeypatch.setenv("TL_TILE", tile)
        jobs = [tl.Job(L, W, ts, src.clone()) for L, W, ts, src in lats]
        log(f"{prec} {n} steps: tile {tile}")
        plan = c.plan(jobs, n, 8.0, prec)     # converged enough to stay far from underflow
        plan.load()
        plan.run()
        plan.store()
        c.sync()
        assert plan.info()["variant"] == int(tile[0])
        plan.close()
        outs[tile] = [j.psi for j in jobs]
    c.close()
    want = outs.pop("0,64,4,0")
    assert all(w.abs().max() > 1e-6 for w in want)
    for tile, got in outs.items():
        for a, b in zip(got, want):
            assert torch.equal(a, b), tile
