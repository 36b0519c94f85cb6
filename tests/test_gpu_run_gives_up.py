"""A whole-run launch whose waits run out (TL_FAULT=wait: a halo word that is not there at the first
look) ends, leaves NaNs, and is reported once by every entry point that can know of it; other plans
and contexts are not concerned, the plan works on, and the tuner takes no such candidate."""
import numpy as np
import pytest

from paper_2301_05518_amd import synth
from tests.gpu_common import log, to_dev

pytestmark = pytest.mark.gpu

GAVE_UP = "TL_ERR_HIP.*gave up waiting"
CUT = (32, 24, 20, 1)      # cells of 16x12x10, cut into tiles
WHOLE = (8, 6, 8, 1)       # cells of 4x3x4: one tile, nothing to wait for


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


@pytest.fixture
def ctx(torch, monkeypatch):
    import paper_2301_05518_amd as tl
    monkeypatch.setenv("TL_FAULT", "wait")
    c = tl.Context(0)
    monkeypatch.delenv("TL_FAULT")
    yield c
    c.close()


def make_job(c, L, prec):
    import paper_2301_05518_amd as tl
    U = synth.gauge_field(L, "haar", 9700)
    psi = synth.random_field(np.random.default_rng([9700, *L]), (3, L[2], L[1], L[0], 3))
    return tl.Job(L, c.build_twolinks(L, to_dev(U), prec), [0, 0, 0], to_dev(psi))


@pytest.mark.parametrize("tile", [None, "9,512,64,8,0,0"])      # whole teams; a team too small for its cell
@pytest.mark.parametrize("prec", ["f64", "f32", "f16s", "bf16"])
def test_reported_with_nans(ctx, torch, monkeypatch, prec, tile):
    import paper_2301_05518_amd as tl
    if tile:
        monkeypatch.setenv("TL_TILE", tile)
    job = make_job(ctx, CUT, prec)
    plan = ctx.plan([job], 40, 4.0, prec)
    plan.load()
    plan.run()
    plan.store()
    log(f"gives up: {prec} tile {tile}")
    torch.cuda.synchronize()
    assert plan.info()["variant"] == 9
    assert torch.isnan(torch.view_as_real(job.psi)).any()
    with pytest.raises(tl.TwolinkError, match=GAVE_UP):
        ctx.sync()
    ctx.sync()          # reported once
    plan.close()


@pytest.mark.parametrize("how", ["run", "store", "reduce", "time", "destroy", "smear"])
def test_reported_by(ctx, torch, how):
    import paper_2301_05518_amd as tl
    job, other = make_job(ctx, CUT, "f32"), make_job(ctx, WHOLE, "f32")
    plan, sound = ctx.plan([job], 40, 4.0, "f32"), ctx.plan([other], 40, 4.0, "f32")
    if how != "smear":
        plan.load()
        plan.run()
        torch.cuda.synchronize()
    for call in (sound.load, sound.run, sound.store):      # another plan is not concerned
        call()
    log(f"gives up: reported by {how}")
    call = {"run": plan.run, "store": plan.store, "reduce": lambda: plan.reduce("norm2"), "time": lambda: plan.time(2),
            "destroy": plan.close, "smear": lambda: ctx.smear([job], 40, 4.0, "f32")}[how]
    with pytest.raises(tl.TwolinkError, match=GAVE_UP):
        call()
    torch.cuda.synchronize()
    if how != "time":       # whose own runs gave up again
        ctx.sync()
    assert not torch.isnan(torch.view_as_real(other.psi)).any()
    try:
        plan.close()
    except tl.TwolinkError:
        assert how == "time"
    sound.close()


def test_tuner_takes_no_launch_that_gives_up(ctx, torch, monkeypatch):
    import paper_2301_05518_amd as tl
    job = make_job(ctx, CUT, "f32")
    src = job.psi.clone()
    monkeypatch.setenv("TL_TILE", "0,64,1,0")
    ctx.smear([job], 40, 4.0, "f32")
    want = job.psi.clone()
    monkeypatch.delenv("TL_TILE")
    job.psi.copy_(src)
    plan = ctx.plan([job], 40, 4.0, "f32", tl.TL_AUTOTUNE)
    plan.load()
    plan.run()
    plan.store()
    ctx.sync()
    log(f"tuned with waits that run out: variant {plan.info()['variant']}")
    assert torch.equal(job.psi, want)
    plan.close()
