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
