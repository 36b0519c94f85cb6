"""All steps of a run in one launch (step variant 9) against one-step launches of the direct
kernel, bit for bit: every storage form; cells that are one tile, that are cut in one, two and
three directions with ragged last tiles, and that a short grid cuts into more tiles than a team
has workgroups; cells of one and two sites per direction; odd extents (one chain per direction)
and even ones (two); RHS sharing a thread and on threads of their own; several units per team;
then repeated runs of one plan, its autotuner entry and the refusals."""
import numpy as np
import pytest

from paper_2301_05518_amd import synth
from tests.gpu_common import errors, log, to_dev, tol

pytestmark = pytest.mark.gpu

DIRECT = "0,64,1,0"

# (lattice, RHS slices): cells of 4x3x5, 2x2x1 (one tile each), 7x9x5 (odd extents: one cell),
# 16x12x10 and 13x11x12 (cut into tiles), 32x4x3 (long rows)
CASES = [((8, 6, 10, 3), [0, 2, 0, 0]), ((4, 4, 2, 1), [0, 0]), ((7, 9, 5, 2), [1, 0]),
         ((32, 24, 20, 2), [0, 1, 1]), ((26, 11, 24, 1), [0, 0, 0, 0]), ((64, 8, 6, 1), [0, 0])]

# "9,threads per workgroup,workgroups per team,grid,two thread sets per group,one per RHS"; teams
# of more than 32 workgroups of a full grid span several XCDs
TILES = ["9,512,32,0,0,0", "9,256,64,0,0,1", "9,512,8,64,0,1", "9,512,256,0,0,0", "9,512,64,8,0,0",
         "9,512,32,0,1,0", "9,256,128,0,1,0"]


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


def lattices(seed0, cases=CASES):
    out = []
    for k, (L, ts) in enumerate(cases):
        U = synth.gauge_field(L, "haar", 5400 + seed0 + k)
        psi = synth.random_field(np.random.default_rng([5400, seed0, k]), (len(ts), L[2], L[1], L[0], 3))
        out.append((L, U, ts, psi))
    return out


def smear(ctx, torch, lats, n, sigma, prec, flags=0, runs=1):
    """Smear through a plan `runs` times from the same sources; the plan's variant and the results."""
    import paper_2301_05518_amd as tl
    jobs = []
    for L, U, ts, psi in lats:
        links = ctx.pack_links if prec.endswith("-onelink") else ctx.build_twolinks
        jobs.append(tl.Job(tuple(L), links(L, to_dev(U), prec), list(ts), to_dev(psi)))
    plan = ctx.plan(jobs, n, sigma, prec, flags)
    outs = []
    try:
        for _ in range(runs):
            for j, (_, _, _, psi) in zip(jobs, lats):
                j.psi.copy_(to_dev(psi))
            plan.load()
            plan.run()
            plan.store()
            ctx.sync()
            outs.append([j.psi.cpu().numpy() for j in jobs])
        info = plan.info()
    finally:
        plan.close()
    return info, outs


@pytest.mark.parametrize("prec", ["f64", "f32", "f16s", "bf16", "f32-w12", "f64-w12", "f16s-w12", "bf16-w12",
                                  "f32-onelink", "f64-onelink", "bf16-w12-onelink"])
def test_whole_run_bit_identical(ctx, orc, torch, prec, monkeypatch):
    import paper_2301_05518_amd as tl
    lats = lattices(10)
    n, sigma = (5, 0.6) if prec.endswith("-onelink") else (5, 2.5)
    monkeypatch.setenv("TL_TILE", DIRECT)
    _, (ref,) = smear(ctx, torch, lats, n, sigma, prec)
    ran = 0
    for tile in TILES:
        for part in (lats, lats[:3], lats[3:4], lats[4:5]):   # the batch, and lattices on their own
            monkeypatch.setenv("TL_TILE", tile)
            log(f"whole run {prec}: tile {tile}, {[p[0] for p in part]}")
            try:
                info, (out,) = smear(ctx, torch, part, n, sigma, prec)
            except tl.TwolinkError as e:   # FP64 threads take one RHS
                assert "TL_ERR_UNSUPPORTED" in str(e)
                log("  not applicable")
                continue
            ran += 1
            assert info["variant"] == 9 and info["steps_per_launch"] == 1 and info["tile_width"] == 1
            for (L, _, _, psi), a in zip(part, out):
                b = next(r for q, r in zip(lats, ref) if q[0] == L)
                assert np.array_equal(a, b), (tile, L)
    assert ran >= 8
    base = prec.replace("-onelink", "")
    for (L, U, ts, psi), o in zip(lats, ref):
        if prec.endswith("-onelink"):
            r = orc.smear_onelink_batch(U, ts, n, sigma, psi)
        else:
            r = orc.smear_batch(orc.build_twolinks(U), ts, n, sigma, psi)
        mr, l2 = errors(o, r)
        assert mr < tol(base, n) and l2 < tol(base, n), L


@pytest.mark.parametrize("n", [1, 4, 7])
def test_runs_of_one_plan(ctx, torch, n, monkeypatch):
    """Repeated runs of one plan (other tags each run, the resident buffer flips once per run),
    with and without TL_GRAPH."""
    import paper_2301_05518_amd as tl
    lats = lattices(30, [((24, 20, 18, 2), [0, 1, 0, 0])])
    monkeypatch.setenv("TL_TILE", DIRECT)
    _, (ref,) = smear(ctx, torch, lats, n, 0.3 * n, "f32")
    for tile in ("9,512,16,0,0,0", "9,256,32,0,0,1"):
        monkeypatch.setenv("TL_TILE", tile)
        for flags in (tl.TL_GRAPH, 0):
            log(f"repeated runs n={n}: tile {tile} flags {flags}")
            _, outs = smear(ctx, torch, lats, n, 0.3 * n, "f32", flags, runs=5)
            for out in outs:
                assert np.array_equal(out[0], ref[0])


def test_captured_by_the_caller(ctx, torch, monkeypatch):
    """tl_plan_run inside the caller's own graph: several replays, each against the eager result."""
    import paper_2301_05518_amd as tl
    (L, U, ts, psi), = lattices(40, [((20, 18, 16, 1), [0, 0, 0])])
    monkeypatch.setenv("TL_TILE", DIRECT)
    _, (ref,) = smear(ctx, torch, [(L, U, ts, psi)], 6, 2.0, "f32")
    monkeypatch.setenv("TL_TILE", "9,256,32,0,0,0")
    side = torch.cuda.Stream()
    c = tl.Context(0, side)
    src = to_dev(psi)
    with torch.cuda.stream(side):
        job = tl.Job(L, c.build_twolinks(L, to_dev(U), "f32"), ts, src.clone())
        plan = c.plan([job], 6, 2.0, "f32")
        for _ in range(2):   # an even number of runs: the capture starts on the first buffer
            job.psi.copy_(src)
            plan.load()
            plan.run()
            plan.store()
        side.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            for _ in range(2):
                job.psi.copy_(src)
                plan.load()
                plan.run()
                plan.store()
        for rep in range(4):
            job.psi.zero_()
            g.replay()
            side.synchronize()
            log(f"replay {rep}")
            assert np.array_equal(job.psi.cpu().numpy(), ref[0]), rep
    c.sync()
    plan.close()
    c.close()


def test_autotuned(ctx, torch, monkeypatch):
    """The autotuner's pick gives the direct kernel's bits, also when a plan of fewer steps takes
    the same entry of the tuning cache."""
    import paper_2301_05518_amd as tl
    lats = lattices(50, [((20, 16, 12, 2), [0, 1, 1])])
    for n in (9, 4, 2, 1):
        monkeypatch.setenv("TL_TILE", DIRECT)
        _, (ref,) = smear(ctx, torch, lats, n, 0.2 * n, "f16s")
        monkeypatch.delenv("TL_TILE")
        info, outs = smear(ctx, torch, lats, n, 0.2 * n, "f16s", tl.TL_GRAPH | tl.TL_AUTOTUNE, runs=3)
        log(f"autotuned n={n}: variant {info['variant']}")
        for out in outs:
            assert np.array_equal(out[0], ref[0]), n
        assert n >= 4 or info["variant"] != 9


def test_refusals(ctx, torch, monkeypatch):
    import paper_2301_05518_amd as tl
    lats = lattices(60, [((12, 8, 10, 1), [0, 0])])
    for tile, prec, flags in (("9,512,32,0", "f32", tl.TL_PLAIN), ("9,64,32,0,0,1", "f32", 0), ("9,64,1,0", "f32", 0)):
        monkeypatch.setenv("TL_TILE", tile)
        with pytest.raises(tl.TwolinkError, match="TL_ERR_UNSUPPORTED"):
            smear(ctx, torch, lats, 4, 2.0, prec, flags)
    # a slice whose one cell (odd extents) exceeds every team
    lats = lattices(61, [((65, 65, 33, 1), [0])])
    monkeypatch.setenv("TL_TILE", "9,512,256,0")
    with pytest.raises(tl.TwolinkError, match="TL_ERR_UNSUPPORTED"):
        smear(ctx, torch, lats, 4, 1.0, "f32")


@pytest.mark.parametrize("n", [4, 5])
@pytest.mark.parametrize("tile", ["9,512,32,0,0,0", "9,512,32,0,0,1", "9,512,32,64,0,0", "9,512,64,8,0,0"])
def test_smaller_units_share_a_team(ctx, torch, tile, n, monkeypatch):
    """Units of the smaller lattices of a batch run several at once in one team: even and uneven
    numbers of them per team (3, 2 and 5 slices), one-tile cells, odd and even step counts (the
    two scratch planes), a short grid, and a team too small for its place (run one by one)."""
    import paper_2301_05518_amd as tl
    lats = lattices(90, [((32, 24, 32, 1), [0]), ((16, 12, 20, 3), [0, 1, 2]), ((12, 7, 16, 2), [0, 1, 1]),
                         ((4, 6, 4, 5), [0, 1, 2, 3, 4])])
    monkeypatch.setenv("TL_TILE", DIRECT)
    _, (want,) = smear(ctx, torch, lats, n, 0.1 * n, "f32")
    monkeypatch.setenv("TL_TILE", tile)
    info, outs = smear(ctx, torch, lats, n, 0.1 * n, "f32", tl.TL_GRAPH, runs=3)
    assert info["variant"] == 9
    for got in outs:
        for w, g in zip(want, got):
            np.testing.assert_array_equal(g, w)
