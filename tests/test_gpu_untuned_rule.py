"""What a plan that is neither tuned nor forced runs: all steps in one launch from four steps on
where the cells fit, step launches for few steps, flags that ask for them, lattices that do not fit
and many rounds of few steps; the direct kernel's bits each time."""
import pytest

from tests.gpu_common import log

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


@pytest.fixture(scope="module")
def ctx(torch):
    import paper_2301_05518_amd as tl
    c = tl.Context(0)
    yield c
    c.close()


def job(torch, ctx, L, per, prec):
    import paper_2301_05518_amd as tl
    g = torch.Generator(device="cuda").manual_seed(41)
    V = (L[3], L[2], L[1], L[0])
    U = torch.view_as_complex(0.3 * torch.randn(*V, 4, 3, 3, 2, dtype=torch.float64, device="cuda", generator=g))
    ts = [t for t in range(L[3]) for _ in range(per)]
    psi = torch.view_as_complex(torch.randn(len(ts), *V[1:], 3, 2, dtype=torch.float64, device="cuda", generator=g))
    return tl.Job(L, (ctx.pack_links if prec.endswith("-onelink") else ctx.build_twolinks)(L, U, prec), ts, psi)


CASES = [
    ((8, 8, 8, 1), 1, "f64", 4, 0, 9),                 # one-tile cells
    ((16, 16, 16, 1), 3, "f32", 4, 0, 9),              # cut cells, one round
    ((16, 16, 16, 2), 4, "f16s", 20, 0, 9),
    ((32, 32, 32, 1), 3, "f64", 8, 0, 9),
    ((7, 9, 5, 3), 2, "bf16", 5, 0, 9),                # odd extents
    ((24, 24, 24, 2), 3, "f32-w12-onelink", 12, 0, 9),
    ((33, 33, 17, 24), 1, "bf16", 60, 0, 9),           # six rounds of many steps
    ((33, 33, 17, 24), 1, "bf16", 4, 0, 0),            # six rounds of few steps
    ((16, 16, 16, 1), 3, "f32", 3, 0, 0),              # fewer than four steps
    ((16, 16, 16, 1), 3, "f32", 8, "TL_PLAIN", 0),
    ((16, 16, 16, 1), 3, "f32", 8, "TL_ONE_STEP", 0),
    ((16, 16, 16, 1), 3, "f32", 8, "TL_GRAPH", 9),
    ((65, 65, 33, 1), 1, "f32", 8, 0, 0),              # a cell that no team holds
]


@pytest.mark.parametrize("L,per,prec,n,flags,variant", CASES)
def test_rule(torch, ctx, monkeypatch, L, per, prec, n, flags, variant):
    j = job(torch, ctx, L, per, prec)
    src = j.psi.clone()
    check(ctx, torch, monkeypatch, [j], [src], prec, n, flags, variant)


def test_batch_of_one_round(torch, ctx, monkeypatch):
    """Units of several lattices, each on a team of its own: one round, four steps suffice."""
    jobs = [job(torch, ctx, L, 2, "f16s") for L in ((32, 24, 20, 1), (14, 9, 16, 1), (4, 6, 4, 2))]
    check(ctx, torch, monkeypatch, jobs, [j.psi.clone() for j in jobs], "f16s", 4, 0, 9)


def check(ctx, torch, monkeypatch, jobs, srcs, prec, n, flags, variant):
    import paper_2301_05518_amd as tl
    outs = []
    for tile in (None, "0,64,1,0"):
        if tile:
            monkeypatch.setenv("TL_TILE", tile)
        for j, src in zip(jobs, srcs):
            j.psi.copy_(src)
        plan = ctx.plan(jobs, n, 0.1 * n, prec, getattr(tl, flags) if flags else 0)
        if not tile:
            log(f"{[j.L for j in jobs]} {prec} n={n} {flags}: variant {plan.info()['variant']}")
            assert plan.info()["variant"] == variant       # ready when created
        plan.load()
        plan.run()
        plan.store()
        ctx.sync()
        assert plan.info()["variant"] == (0 if tile else variant)
        plan.close()
        outs.append([j.psi.clone() for j in jobs])
    assert all(torch.equal(a, b) for a, b in zip(*outs))
