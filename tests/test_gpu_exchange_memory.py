"""Memory of whole-run launches that cannot be had or cleared (TL_FAULT=exchange): nothing uncleared
is ever taken for cleared."""
import numpy as np
import pytest

from paper_2301_05518_amd import synth
from tests.gpu_common import log, to_dev

pytestmark = pytest.mark.gpu

DIRECT = "0,64,1,0"


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


@pytest.fixture
def ctx(torch, monkeypatch):
    import paper_2301_05518_amd as tl
    monkeypatch.setenv("TL_FAULT", "exchange")
    c = tl.Context(0)
    monkeypatch.delenv("TL_FAULT")
    yield c
    c.close()


@pytest.fixture
def work(ctx, torch, monkeypatch):
    """A job on a lattice of cut cells, its sources, and the direct kernel's result of 20 steps."""
    import paper_2301_05518_amd as tl
    L = (32, 24, 20, 1)
    U = synth.gauge_field(L, "haar", 9800)
    src = to_dev(synth.random_field(np.random.default_rng([9800]), (3, L[2], L[1], L[0], 3)))
    job = tl.Job(L, ctx.build_twolinks(L, to_dev(U), "f32"), [0, 0, 0], src.clone())
    monkeypatch.setenv("TL_TILE", DIRECT)
    plan = ctx.plan([job], 20, 2.0, "f32", tl.TL_ONE_STEP)
    run(plan)
    want = job.psi.clone()
    plan.close()
    monkeypatch.delenv("TL_TILE")
    job.psi.copy_(src)
    return job, src, want


def run(plan):
    plan.load()
    plan.run()
    plan.store()


def test_forced_whole_run_is_refused_each_time(ctx, torch, work, monkeypatch):
    import paper_2301_05518_amd as tl
    job, src, want = work
    plan = ctx.plan([job], 20, 2.0, "f32", tl.TL_ONE_STEP)
    monkeypatch.setenv("TL_TILE", "9,512,32,0,0,0")
    for k in range(3):       # a second try does not find the first one's memory
        log(f"try {k}")
        with pytest.raises(tl.TwolinkError, match="TL_ERR_NOMEM"):
            plan.run()
    monkeypatch.delenv("TL_TILE")
    run(plan)
    ctx.sync()
    assert plan.info()["variant"] == 0
    assert torch.equal(job.psi, want)
    plan.close()


@pytest.mark.parametrize("how", ["plan", "graph", "tuned", "smear"])
def test_step_launches_where_there_is_none(ctx, torch, work, how):
    import paper_2301_05518_amd as tl
    job, src, want = work
    for rep in range(2):
        job.psi.copy_(src)
        if how == "smear":
            ctx.smear([job], 20, 2.0, "f32")
        else:
            plan = ctx.plan([job], 20, 2.0, "f32", {"plan": 0, "graph": tl.TL_GRAPH, "tuned": tl.TL_AUTOTUNE}[how])
            run(plan)
            log(f"{how}: variant {plan.info()['variant']}")
            assert plan.info()["variant"] != 9
            plan.close()
        ctx.sync()
        assert torch.equal(job.psi, want), rep


def test_cached_whole_run(torch, work, monkeypatch, tmp_path):
    """A tuning-cache entry that names a whole run: its one-step companion runs."""
    import json

    import paper_2301_05518_amd as tl
    job, src, want = work
    cache = tmp_path / "tune.json"
    monkeypatch.setenv("TL_TUNE_CACHE", str(cache))
    for fault, variant in (("", 9), ("exchange", 0)):
        monkeypatch.setenv("TL_FAULT", fault)
        c = tl.Context(0)
        for _ in range(2):
            plan = c.plan([job], 20, 2.0, "f32", tl.TL_AUTOTUNE)
            job.psi.copy_(src)
            run(plan)
            c.sync()
            assert torch.equal(job.psi, want)
            if fault:
                assert plan.info()["variant"] == variant and c.stats()["tune_sweeps"] == 0
            plan.close()
        c.close()
        cache.write_text(json.dumps({k: "9,512,32,0,0,0;0,64,1,0,0,0" for k in json.loads(cache.read_text())}))
