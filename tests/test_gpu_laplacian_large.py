"""The Laplacian of large slices of 16-bit vectors (pack, step and unpack) against the one-launch
kernel: a small slice repeated periodically has the small slice's Laplacian, bit for bit, on both
sides of the limit; two calls of different sizes share the scratch memory; refused under capture."""
import pytest

from tests.gpu_common import log

pytestmark = pytest.mark.gpu

BASE = (32, 25, 24)      # 19200 sites; repeated 4 x 4 x 4 times: 1228800, 4 x 4 x 3 times: 921600


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


@pytest.mark.parametrize("prec", ["f16s", "bf16", "f16s-w12", "bf16-onelink", "f32", "f64"])
def test_repeated_slice(torch, prec):
    import paper_2301_05518_amd as tl
    c = tl.Context(0)
    g = torch.Generator(device="cuda").manual_seed(61)
    x, y, z = BASE
    U = torch.view_as_complex(0.3 * torch.randn(1, z, y, x, 4, 3, 3, 2, dtype=torch.float64, device="cuda", generator=g))
    psi = torch.view_as_complex(torch.randn(z, y, x, 3, 2, dtype=torch.float64, device="cuda", generator=g))
    links = c.pack_links if prec.endswith("-onelink") else c.build_twolinks
    L = (*BASE, 1)
    want = c.laplacian(L, links(L, U, prec), prec, 0, psi)
    for rz in (4, 3, 4):
        big = (4 * x, 4 * y, rz * z, 1)
        W = links(big, U.repeat(1, rz, 4, 4, 1, 1, 1).contiguous(), prec)
        got = c.laplacian(big, W, prec, 0, psi.repeat(rz, 4, 4, 1).contiguous())
        log(f"{prec}: {big[0] * big[1] * big[2]} sites")
        assert torch.equal(got, want.repeat(rz, 4, 4, 1))
    c.close()


def test_capture(torch):
    import paper_2301_05518_amd as tl
    side = torch.cuda.Stream()
    c = tl.Context(0, side)
    with torch.cuda.stream(side):
        for L, ok in (((32, 25, 24, 1), True), ((128, 100, 96, 1), False)):
            V = (L[2], L[1], L[0])
            U = torch.view_as_complex(torch.randn(1, *V, 4, 3, 3, 2, dtype=torch.float64, device="cuda"))
            psi = torch.view_as_complex(torch.randn(*V, 3, 2, dtype=torch.float64, device="cuda"))
            out = torch.empty_like(psi)
            W = c.build_twolinks(L, U, "bf16")
            want = c.laplacian(L, W, "bf16", 0, psi).clone()
            side.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side):
                if ok:
                    c.laplacian(L, W, "bf16", 0, psi, out)
                else:
                    with pytest.raises(tl.TwolinkError, match="TL_ERR_HIP.*captured"):
                        c.laplacian(L, W, "bf16", 0, psi, out)
            if ok:
                for _ in range(3):
                    out.zero_()
                    graph.replay()
                    side.synchronize()
                    assert torch.equal(out, want)
            else:
                c.laplacian(L, W, "bf16", 0, psi, out)
                side.synchronize()
                assert torch.equal(out, want)
    c.close()
