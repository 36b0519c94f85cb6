"""Whole-run launches with incomplete teams (TL_FAULT=team: each runs with the workgroups that were
there when its first one looked, however many) and with teams that spread over two, four and eight
XCDs in parts that do not divide evenly: the direct kernel's bits, run after run."""
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


def bits(torch, monkeypatch, fault, tile, lats, prec, n, runs):
    import paper_2301_05518_amd as tl
    monkeypatch.setenv("TL_TILE", tile)
    monkeypatch.setenv("TL_FAULT", fault)
    c = tl.Context(0)
    jobs, srcs = [], []
    for L, ts in lats:
        U = synth.gauge_field(L, "haar", 9950)
        srcs.append(to_dev(synth.random_field(np.random.default_rng([9950, *L]), (len(ts), L[2], L[1], L[0], 3))))
        links = c.pack_links if prec.endswith("-onelink") else c.build_twolinks
        jobs.append(tl.Job(L, links(L, to_dev(U), prec), ts, srcs[-1].clone()))
    plan = c.plan(jobs, n, 0.1 * n, prec)
    outs = []
    for _ in range(runs):
        for j, s in zip(jobs, srcs):
            j.psi.copy_(s)
        plan.load()
        plan.run()
        plan.store()
        c.sync()
        outs.append([j.psi.clone() for j in jobs])
    log(f"{prec} tile {tile} {fault or 'whole teams'}: variant {plan.info()['variant']}, {plan.info()['n_tiles']} tiles")
    assert plan.info()["variant"] == int(tile[0])
    plan.close()
    c.close()
    return outs


BATCH = [((32, 24, 20, 2), [0, 1, 1, 1]), ((16, 12, 20, 3), [0, 1, 2, 2]), ((26, 11, 24, 1), [0, 0, 0])]


# RHS per thread: four, two (the incomplete team's half-groups), one; teams of two to all members
@pytest.mark.parametrize("prec", ["f64", "f32", "f16s", "bf16", "f32-w12", "f64-onelink"])
def test_incomplete_teams(torch, monkeypatch, prec):
    lats = BATCH if prec != "f64" else [(L, ts[:1]) for L, ts in BATCH] + [((32, 24, 20, 1), [0] * 3)]
    (want,) = bits(torch, monkeypatch, "", "0,64,1,0", lats, prec, 5, 1)
    for tile in ("9,512,4,0,0,0", "9,512,32,0,0,0", "9,512,64,0,1,0", "9,256,64,0,0,1", "9,512,128,0,0,0"):
        try:
            outs = bits(torch, monkeypatch, "team", tile, lats, prec, 5, 4)
        except Exception as e:
            # FP64 cells that do not fit so few or so narrow workgroups
            assert prec.startswith("f64") and "TL_ERR_UNSUPPORTED" in str(e), (prec, tile)
            continue
        for out in outs:
            for a, b in zip(out, want):
                assert torch.equal(a, b), tile


@pytest.mark.parametrize("fault", ["", "team"])
@pytest.mark.parametrize("L", [(40, 36, 20, 1), (44, 36, 28, 1), (64, 44, 36, 1)])
def test_teams_over_several_xcds(torch, monkeypatch, L, fault):
    (want,) = bits(torch, monkeypatch, "", "0,64,1,0", [(L, [0, 0])], "f32", 6, 1)
    for out in bits(torch, monkeypatch, fault, "9,64,256,0,0,0", [(L, [0, 0])], "f32", 6, 4):
        assert torch.equal(out[0], want[0])
