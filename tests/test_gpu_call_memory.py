"""Memory that tl_smear keeps for later calls, and exchange memory that changes its layout under one
control block: calls of changing sizes, formats, RHS counts and step counts on one context, in an
order that reuses, replaces, grows and displaces blocks, with the context's stream changed in
between and created plans in use meanwhile; every result is a fresh context's, bit for bit."""
import numpy as np
import pytest

from paper_2301_05518_amd import synth
from tests.gpu_common import log, to_dev

pytestmark = pytest.mark.gpu

# (lattice, RHS, format, steps): one-tile and cut cells, odd extents, one and several rounds
CALLS = [((16, 16, 16, 1), 3, "f32", 20), ((8, 8, 8, 2), 4, "f64", 7), ((30, 27, 22, 1), 2, "bf16", 9),
         ((32, 24, 20, 1), 4, "f32", 12), ((6, 4, 8, 3), 1, "f16s", 4), ((32, 32, 32, 1), 1, "f64", 6),
         ((24, 24, 24, 2), 3, "f32-w12", 8), ((16, 16, 16, 1), 3, "f32", 2), ((40, 36, 20, 1), 2, "f16s", 5),
         ((12, 10, 8, 1), 3, "bf16-w12-onelink", 10), ((48, 16, 16, 2), 2, "f32-onelink", 11), ((9, 7, 5, 1), 2, "f64", 5),
         ((20, 20, 20, 1), 4, "bf16", 16), ((48, 48, 24, 1), 3, "f32", 6)]


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


@pytest.fixture(scope="module")
def work(torch):
    """Jobs, sources and a fresh context's result for every call."""
    import paper_2301_05518_amd as tl
    out = []
    for k, (L, per, prec, n) in enumerate(CALLS):
        c = tl.Context(0)
        U = synth.gauge_field(L, "haar", 9800 + k)
        ts = [t for t in range(L[3]) for _ in range(per)]
        src = to_dev(synth.random_field(np.random.default_rng([9801, k]), (len(ts), L[2], L[1], L[0], 3)))
        links = c.pack_links if prec.endswith("-onelink") else c.build_twolinks
        job = tl.Job(L, links(L, to_dev(U), prec), ts, src.clone())
        c.smear([job], n, 0.1 * n, prec)
        out.append((job, src, job.psi.clone()))
        c.close()
    return out


def one(torch, c, work, k, flags=0):
    L, per, prec, n = CALLS[k]
    job, src, want = work[k]
    job.psi.copy_(src)
    torch.cuda.synchronize()
    c.smear([job], n, 0.1 * n, prec, flags)
    if flags:      # a kept call does not wait
        c.sync()
    assert torch.equal(job.psi, want), CALLS[k]


def test_calls_in_changing_order(torch, work):
    import paper_2301_05518_amd as tl
    c = tl.Context(0)
    rng = np.random.default_rng(9802)
    order = list(range(len(CALLS))) + [k for k in range(len(CALLS)) for _ in range(2)] + list(rng.integers(0, len(CALLS), 60))
    log(f"{len(order)} calls on one context")
    for k in order:
        one(torch, c, work, int(k))
    c.close()


def test_streams_and_plans_in_between(torch, work):
    import paper_2301_05518_amd as tl
    streams = [torch.cuda.default_stream(), torch.cuda.Stream(), torch.cuda.Stream()]
    c = tl.Context(0, streams[0])
    rng = np.random.default_rng(9803)
    plans = {}
    for rep in range(60):
        s = streams[int(rng.integers(0, 3))]
        c.set_stream(s)
        k = int(rng.integers(0, len(CALLS)))
        L, per, prec, n = CALLS[k]
        job, src, want = work[k]
        if rep % 3 == 0:          # a created plan, kept over several calls
            old = plans.pop(k, None)
            if old:
                old.close()
            plans[k] = c.plan([job], n, 0.1 * n, prec, tl.TL_GRAPH if rep % 2 else 0)
        if k in plans:
            job.psi.copy_(src)
            torch.cuda.synchronize()
            plans[k].load()
            plans[k].run()
            plans[k].store()
            c.sync()
            assert torch.equal(job.psi, want), (rep, CALLS[k])
        one(torch, c, work, k, tl.TL_GRAPH if rep % 5 == 4 else 0)
    for p in plans.values():
        p.close()
    c.close()


def test_more_than_is_kept(torch):
    """Calls whose memory exceeds what is kept (256 MB): the same bits, and the device gets the memory back."""
    import paper_2301_05518_amd as tl
    L, ts, n = (64, 64, 64, 1), [0] * 8, 4
    g = torch.Generator(device="cuda").manual_seed(9804)
    U = torch.view_as_complex(0.3 * torch.randn(1, 64, 64, 64, 4, 3, 3, 2, dtype=torch.float64, device="cuda", generator=g))
    src = torch.view_as_complex(torch.randn(8, 64, 64, 64, 3, 2, dtype=torch.float64, device="cuda", generator=g))
    c = tl.Context(0)
    W = {p: c.build_twolinks(L, U, p) for p in ("f64", "f32")}
    job = {p: tl.Job(L, W[p], ts, src.clone()) for p in W}
    want = {}
    torch.cuda.synchronize()
    free = []
    for rep in range(6):
        for p in W:
            job[p].psi.copy_(src)
            torch.cuda.synchronize()
            c.smear([job[p]], n, 0.4, p)
            if p in want:
                assert torch.equal(job[p].psi, want[p]), (rep, p)
            want.setdefault(p, job[p].psi.clone())
        free.append(torch.cuda.mem_get_info()[0])
    c.close()
    after = torch.cuda.mem_get_info()[0]
    log(f"free after each round {free}, after the context {after}")
    assert min(free[2:]) >= free[1] - (1 << 20) * 16          # nothing grows from call to call
    assert after - free[-1] <= (512 + 64) * (1 << 20)         # at most 512 MB were kept
