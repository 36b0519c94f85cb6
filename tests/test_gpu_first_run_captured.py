"""A plan's first run inside the caller's own graph: an untuned plan is ready when it is created, so
eager runs before any replay, and replays, give the eager result; what would have to prepare
something under the capture (a new plan, tl_smear, the tuned or forced first run) is refused and
leaves the plan usable."""
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


def setup(torch, c, L, ts, seed):
    import paper_2301_05518_amd as tl
    U = synth.gauge_field(L, "haar", 9100 + seed)
    src = to_dev(synth.random_field(np.random.default_rng([9100, seed]), (len(ts), L[2], L[1], L[0], 3)))
    job = tl.Job(L, c.build_twolinks(L, to_dev(U), "f32"), ts, src.clone())
    return src, job


def passes(plan, job, src):
    job.psi.copy_(src)
    plan.load()
    plan.run()
    plan.store()


# one-step launches and whole runs; a units table and a step table that travel in a launch's
# arguments (3 groups) and that do not (64 slices: more than 3072 bytes of each)
@pytest.mark.parametrize("n", [2, 3, 6, 7])
@pytest.mark.parametrize("slices", [3, 64])
def test_first_run_captured(torch, monkeypatch, n, slices):
    import paper_2301_05518_amd as tl
    side = torch.cuda.Stream()
    c = tl.Context(0, side)
    with torch.cuda.stream(side):
        src, job = setup(torch, c, (8, 6, 4, slices), list(range(slices)) * 2, slices)
        monkeypatch.setenv("TL_TILE", DIRECT)
        ref = c.plan([job], n, 0.3 * n, "f32")
        passes(ref, job, src)
        side.synchronize()
        want = job.psi.clone()
        ref.close()
        monkeypatch.delenv("TL_TILE")
        plan = c.plan([job], n, 0.3 * n, "f32")
        log(f"n={n}, {slices} slices: variant {plan.info()['variant']}")
        side.synchronize()
        graphs = []
        for _ in range(2):     # one graph per buffer parity; neither has been replayed yet
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=side):
                passes(plan, job, src)
            graphs.append(g)
        job.psi.zero_()
        passes(plan, job, src)
        side.synchronize()
        assert torch.equal(job.psi, want), "eager after the capture"
        for rep in range(3):
            for k in (1, 0):
                job.psi.zero_()
                graphs[k].replay()
                side.synchronize()
                assert torch.equal(job.psi, want), (rep, k)
            passes(plan, job, src)
            side.synchronize()
            assert torch.equal(job.psi, want), rep
    plan.close()
    c.close()


@pytest.mark.parametrize("how", ["create", "smear", "smear-graph", "autotune", "tile"])
def test_refused_under_capture(torch, monkeypatch, how):
    import paper_2301_05518_amd as tl
    side = torch.cuda.Stream()
    c = tl.Context(0, side)
    n = 5
    with torch.cuda.stream(side):
        src, job = setup(torch, c, (8, 6, 4, 2), [0, 1, 1], 7)
        ref = c.plan([job], n, 1.5, "f32")
        passes(ref, job, src)
        side.synchronize()
        want = job.psi.clone()
        ref.close()
        plan = None
        flags = tl.TL_AUTOTUNE if how == "autotune" else tl.TL_GRAPH if how == "smear-graph" else 0
        if how in ("autotune", "tile"):
            plan = c.plan([job], n, 1.5, "f32", flags)
        if how == "smear-graph":       # a kept plan: the second call would replay it
            c.smear([job], n, 1.5, "f32", flags)
        if how == "tile":
            monkeypatch.setenv("TL_TILE", "9,512,8,0,0,0")
        side.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            job.psi.copy_(src)
            with pytest.raises(tl.TwolinkError, match="TL_ERR_HIP.*captured"):
                if how == "create":
                    c.plan([job], n, 1.5, "f32")
                elif how.startswith("smear"):
                    c.smear([job], n, 1.5, "f32", flags)
                else:
                    plan.run()
        g.replay()
        side.synchronize()
        assert torch.equal(job.psi, src)
        if plan is None:
            plan = c.plan([job], n, 1.5, "f32")
        passes(plan, job, src)
        side.synchronize()
        assert torch.equal(job.psi, want)
    plan.close()
    c.close()
