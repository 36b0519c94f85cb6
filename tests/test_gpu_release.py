"""tl_plan_destroy, and tl_smear without TL_GRAPH, return when the smearing is done, on every stream:
the caller may then reuse W and psi on a stream that the context's does not order."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


@pytest.mark.parametrize("stream", ["null", "side"])
@pytest.mark.parametrize("how", ["destroy", "smear"])
def test_returns_when_done(torch, how, stream):
    import paper_2301_05518_amd as tl
    s = torch.cuda.Stream() if stream == "side" else torch.cuda.default_stream()
    L, ts, n = (64, 64, 64, 1), [0, 0, 0], 400     # several ms of device time
    with torch.cuda.stream(s):
        g = torch.Generator(device="cuda").manual_seed(77)
        U = torch.view_as_complex(torch.randn(1, 64, 64, 64, 4, 3, 3, 2, dtype=torch.float64, device="cuda", generator=g))
        psi = torch.view_as_complex(torch.randn(3, 64, 64, 64, 3, 2, dtype=torch.float64, device="cuda", generator=g))
        c = tl.Context(0, s)
        job = tl.Job(L, c.build_twolinks(L, U, "f32"), ts, psi)
        for rep in range(3):       # the later calls reuse the first one's memory
            if how == "destroy":
                plan = c.plan([job], n, 1.0, "f32")
                plan.load()
                plan.run()
                plan.store()
                assert not s.query()       # queued, not done
                plan.close()
            else:
                c.smear([job], n, 1.0, "f32")
            assert s.query(), rep
        c.close()


def test_destroy_waits_for_replays_elsewhere(torch):
    """Replays of a captured run on a stream that the context does not know are done when
    tl_plan_destroy returns, and the next plan's memory is its own."""
    import paper_2301_05518_amd as tl
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    L, ts, n = (32, 32, 32, 1), [0, 0, 0], 400
    c = tl.Context(0, side)
    with torch.cuda.stream(side):
        g = torch.Generator(device="cuda").manual_seed(78)
        U = torch.view_as_complex(0.3 * torch.randn(1, 32, 32, 32, 4, 3, 3, 2, dtype=torch.float64, device="cuda", generator=g))
        src = torch.view_as_complex(torch.randn(3, 32, 32, 32, 3, 2, dtype=torch.float64, device="cuda", generator=g))
        W = c.build_twolinks(L, U, "f32")
        jobs = [tl.Job(L, W, ts, src.clone()) for _ in range(2)]
        want = None
        for rep in range(4):
            plan = c.plan([jobs[0]], n, 1.0, "f32")
            plan.load()
            side.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side):
                plan.run()
            # several ms of replays on the other stream, then a new plan in the destroyed one's memory
            with torch.cuda.stream(other):
                for _ in range(10):
                    graph.replay()
            assert not other.query()
            plan.close()
            assert other.query(), rep
            jobs[1].psi.copy_(src)
            again = c.plan([jobs[1]], 20, 1.0, "f32")
            again.load()
            again.run()
            again.store()
            c.sync()
            want = jobs[1].psi.clone() if want is None else want
            assert torch.equal(jobs[1].psi, want), rep
            again.close()
            del graph
    c.close()
