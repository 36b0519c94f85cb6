"""The Laplacian as one launch on natural fields, and the FP64 reductions at the sizes where the
number of blocks per field changes."""
import numpy as np
import pytest

from oracle import checks
from paper_2301_05518_amd import synth
from tests.gpu_common import log, to_dev, tol_lap

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


@pytest.mark.parametrize("L", [(1, 1, 1), (2, 3, 1), (4, 4, 4), (7, 9, 5), (64, 2, 3), (21, 13, 17)])
@pytest.mark.parametrize("prec", ["f64", "f32", "f16s", "bf16", "f32-w12", "f16s-w12", "f32-onelink", "bf16-w12-onelink"])
def test_laplacian(ctx, orc, torch, prec, L):
    """Against the oracle; and rounding the input to storage beforehand (a plan's load and store)
    changes no bit of the result, so the kernel rounds what it reads as the packing does."""
    import paper_2301_05518_amd as tl
    L = L + (2,)
    U = synth.gauge_field(L, "haar", 7700)
    psi = synth.random_field(np.random.default_rng([7700, *L]), (L[2], L[1], L[0], 3))
    one = prec.endswith("-onelink")
    base = prec.replace("-onelink", "")
    W = (ctx.pack_links if one else ctx.build_twolinks)(L, to_dev(U), prec)
    out = ctx.laplacian(L, W, prec, 1, to_dev(psi))
    ref = orc.laplacian_onelink(U, 1, psi) if one else orc.laplacian(orc.build_twolinks(U), 1, psi)
    mr = checks.max_rel(out.cpu().numpy(), ref)
    log(f"laplacian {prec} {L}: max-rel {mr:.3e}")
    # one-link rows 1 and 2 with the same neighbour twice can cancel against 6 psi; the bound of a
    # Laplacian is relative to its own size, which for a single site of Haar two-links is of order 1
    assert mr < 4 * max(tol_lap(base), 1e-14)
    rounded = to_dev(psi[None])
    job = tl.Job(L, W, [1], rounded)
    plan = ctx.plan([job], 0, 0.0, prec)
    plan.load()
    plan.store()
    again = ctx.laplacian(L, W, prec, 1, rounded[0])
    torch.cuda.synchronize()
    plan.close()
    if not prec.startswith("f16s"):     # an F16S scale may change when a rounded site is rounded again
        assert torch.equal(again, out)


# 2048 blocks of 4096 down to 512 sites: block counts on both sides of every halving
@pytest.mark.parametrize("n_rhs,n_sites", [(1, 1), (3, 511), (2, 513), (5, 4095), (7, 4097), (1, 100003),
                                           (12, 110592), (31, 66 * 4096), (33, 62 * 4096 + 1)])
def test_reductions(ctx, torch, n_rhs, n_sites):
    g = torch.Generator(device="cuda").manual_seed(7710 + n_rhs)
    psi = torch.randn((n_rhs, n_sites, 3), dtype=torch.complex128, device="cuda", generator=g)
    phi = torch.randn((n_rhs, n_sites, 3), dtype=torch.complex128, device="cuda", generator=g)
    norm, dot, site = ctx.reduce("norm2", psi), ctx.reduce("dot", psi, phi), ctx.reduce("site_norm", psi)
    sq = psi.real ** 2 + psi.imag ** 2
    want_n, want_d = sq.sum((1, 2)), (phi.conj() * psi).sum((1, 2))
    # rounding of a sum of N terms in any tree or chain order: below N u times the sum of their sizes;
    # u = 2^-53, and both sides carry it
    u = 2.0 ** -53
    assert ((norm - want_n).abs() <= 2 * 6 * n_sites * u * want_n).all()
    size = (phi.abs() * psi.abs()).sum((1, 2))
    assert ((dot - want_d).abs() <= 2 * 12 * n_sites * u * size).all()
    assert torch.allclose(site, sq.sum(-1).sqrt(), rtol=8 * u, atol=0)
    for kind, a, b in (("norm2", norm, None), ("dot", dot, phi)):    # the same bits every time, and without allocation
        assert torch.equal(ctx.reduce(kind, psi, b), a)
        assert torch.equal(ctx.reduce_noalloc(kind, psi, b), a)
