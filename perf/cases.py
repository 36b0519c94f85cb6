"""The work that users of the library have it do, as cases that can be timed and compared.

Every case goes through the public Python entry points.  Five kinds of work:

* ``smear``  a resident plan, as a production program keeps it for one gauge field: new sources are put
             into the caller's buffer, then load, run (n smearing steps), store.  With ``build`` the
             two-links are built anew first and the FP64 norms are taken last (a whole pass over a new
             configuration).
* ``call``   one ``Context.smear`` call with its default flags (no plan kept, nothing tuned).
* ``lap``    one application of the Laplacian (an eigen-solver's or a test's call).
* ``build``  the two-link field of all slices of a configuration.
* ``reduce`` FP64 inner products, norms and per-site norms of natural fields (two-point functions).

``listed()`` holds the sizes of the repository's own workloads and a few general ones, ``draw()`` more of
the same ranges.
"""
import functools
import math

import torch

import paper_2301_05518_amd as tl

PRECS = ("f64", "f32", "f16s", "bf16")
MAX_UPDATES = 24 * 64 ** 3 * 60     # RHS-site-updates of the largest listed case
KEEP = tl.TL_GRAPH | tl.TL_AUTOTUNE


# ------------------------------------------------------------------ the cases

def _smear(name, shape, per_slice, prec, n, sigma, source, slices=1, links="haar", build=False):
    return {"name": name, "kind": "smear", "shape": shape, "slices": slices, "per_slice": per_slice, "prec": prec,
            "n": n, "sigma": sigma, "source": source, "links": links, "build": build}


def listed():
    return [
        # the smallest plan: one point source on a test-sized lattice, all launch latency
        _smear("plan_8_f64_point", "8x8x8", 1, "f64", 20, 2.0, "point", links="exp"),
        # one propagator's three colour point sources on one slice, double precision
        _smear("plan_32_f64_points", "32x32x32", 3, "f64", 40, 4.0, "point"),
        # the same on a 48^3 slice in the two storage formats production runs use there
        _smear("plan_48_f32_points", "48x48x48", 3, "f32", 40, 5.0, "point"),
        _smear("plan_48_f16s_points", "48x48x48", 3, "f16s", 40, 5.0, "point"),
        # several ensembles at once: uneven lattices with 1, 2 and 4 slices of three Z2 sources each
        _smear("plan_uneven_bf16_z2", "24x24x24+32x32x32+48x48x48", 3, "bf16", 40, 4.0, "z2", slices="1+2+4"),
        # a whole pass of the largest workload: eight 64^3 slices, three colour walls each, new two-links
        _smear("pass_64_f32_walls", "64x64x64", 3, "f32", 60, 6.0, "wall", slices=8, build=True),
        # one-link smearing on a mid-sized lattice with twelve-real links, sources already smooth
        _smear("plan_24_onelink_f32w12", "24x24x24", 3, "f32-w12-onelink", 30, 3.0, "normal", slices=2),
        # ragged extents, four sources on each of two slices, an odd number of steps
        _smear("plan_ragged_f32", "30x27x22", 4, "f32", 25, 4.0, "normal", slices=2),
        # a single call on a small lattice by a program that keeps nothing
        {"name": "call_16_f32", "kind": "call", "shape": "16x16x16", "slices": 1, "per_slice": 3, "prec": "f32",
         "n": 20, "sigma": 2.0, "source": "point", "links": "haar", "build": False},
        # one Laplacian of a 32^3 slice in double precision
        {"name": "lap_32_f64", "kind": "lap", "shape": "32x32x32", "prec": "f64", "source": "normal", "links": "haar"},
        # the two-link field of a dozen slices of a 48^3 configuration
        {"name": "build_48_f32", "kind": "build", "shape": "48x48x48", "slices": 12, "prec": "f32", "links": "haar"},
        # correlators of 12 smeared vectors of a 48^3 slice: inner products and norms
        {"name": "reduce_48x12", "kind": "reduce", "shape": "48x48x48", "per_slice": 12},
    ]


def _extent(rng, lo=6, hi=64):
    e = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return e if rng.random() < 0.3 else max(lo, e & ~1)      # lattices are mostly even; odd ones are valid


def _shape(rng, lo=6, hi=64):
    a = _extent(rng, lo, hi)
    if rng.random() < 0.5:
        return (a, a, a)
    return (a, _extent(rng, max(lo, a // 2), min(hi, 2 * a)), _extent(rng, max(lo, a // 2), min(hi, 2 * a)))


def _text(shapes):
    return "+".join("x".join(str(v) for v in s) for s in shapes)


def draw(rng):
    kind = rng.choices(("smear", "call", "lap", "build", "reduce"), (10, 2, 2, 2, 2))[0]
    shape = _shape(rng)
    v3 = shape[0] * shape[1] * shape[2]
    if kind == "reduce":
        most = max(1, min(96, 20_000_000 // v3))
        return {"kind": kind, "shape": _text([shape]), "per_slice": int(round(math.exp(rng.uniform(0, math.log(most)))))}
    prec = rng.choice(PRECS) + ("-w12" if rng.random() < 0.2 else "")
    if kind == "build":
        most = max(1, min(24, 2_000_000 // v3))
        return {"kind": kind, "shape": _text([shape]), "slices": rng.randint(1, most), "prec": prec, "links": "haar"}
    if rng.random() < 0.2:
        prec += "-onelink"
    if kind == "lap":
        return {"kind": kind, "shape": _text([shape]), "prec": prec, "source": "normal", "links": "haar"}
    shapes = [shape]
    if kind == "smear" and rng.random() < 0.2:
        shapes.append(_shape(rng, hi=48))
    per_slice = rng.choice((1, 3, 3, 3, 4, 6))
    slices = [rng.choice((1, 1, 2, 4, 8)) for _ in shapes]
    n = rng.randint(8, 60)

    def updates():
        return n * per_slice * sum(k * s[0] * s[1] * s[2] for k, s in zip(slices, shapes))

    while updates() > MAX_UPDATES // (4 if kind == "call" else 1):
        slices = [max(1, k // 2) for k in slices]
        per_slice = min(per_slice, 3)
        n = max(8, n // 2)
    step = rng.uniform(0.02, 0.15)       # sigma / n
    return {"kind": kind, "shape": _text(shapes), "slices": "+".join(map(str, slices)), "per_slice": per_slice,
            "prec": prec, "n": n, "sigma": round(step * n, 3), "source": rng.choice(("point", "wall", "z2", "normal")),
            "links": rng.choice(("haar", "exp")), "build": kind == "smear" and rng.random() < 0.2}


# ------------------------------------------------------------------ inputs

def _shapes(case):
    return [tuple(int(v) for v in s.split("x")) for s in case["shape"].split("+")]


def _slices(case):
    return [int(v) for v in str(case.get("slices", 1)).split("+")]


def _gen(seed, key):
    g = torch.Generator(device="cuda")
    g.manual_seed((seed * 1000003 + key * 7919 + 12345) & 0x7FFFFFFFFFFF)
    return g


def _gauss(shape, g):
    return torch.view_as_complex(torch.randn(*shape, 2, dtype=torch.float64, device="cuda", generator=g))


def _su3(r1, r2):
    u1 = r1 / torch.linalg.vector_norm(r1, dim=-1, keepdim=True)
    r2 = r2 - (u1.conj() * r2).sum(-1, keepdim=True) * u1
    u2 = r2 / torch.linalg.vector_norm(r2, dim=-1, keepdim=True)
    return torch.stack([u1, u2, torch.linalg.cross(u1, u2, dim=-1).conj()], dim=-2)


def _links(shape, n_slices, recipe, seed, key):
    """Gauge field [t][z][y][x][mu][a][b]: Haar SU(3), or links scattered about 1 ("exp")."""
    lx, ly, lz = shape
    out = torch.empty(n_slices, lz, ly, lx, 4, 3, 3, dtype=torch.complex128, device="cuda")
    for t in range(n_slices):
        g = _gen(seed, 100 * key + t)
        r = _gauss((lz * ly * lx * 4, 2, 3), g)
        if recipe == "exp":
            r = 0.4 * r
            r[:, 0, 0] += 1.0
            r[:, 1, 1] += 1.0
        out[t] = _su3(r[:, 0], r[:, 1]).view(lz, ly, lx, 4, 3, 3)
    return out


def _sources(shape, n_rhs, per_slice, kind, seed, key):
    lx, ly, lz = shape
    g = _gen(seed, 50000 + key)
    psi = torch.zeros(n_rhs, lz, ly, lx, 3, dtype=torch.complex128, device="cuda")
    if kind == "normal":
        return psi.copy_(_gauss(tuple(psi.shape), g))
    for r in range(n_rhs):
        c = (r % per_slice) % 3
        if kind == "wall":
            psi[r, ..., c] = 1.0
        elif kind == "z2":
            psi[r, ..., c] = (torch.randint(0, 2, (lz, ly, lx), device="cuda", generator=g) * 2 - 1).to(torch.complex128)
        else:
            x0 = torch.randint(0, 1 << 30, (3,), device="cuda", generator=g).tolist()
            psi[r, x0[0] % lz, x0[1] % ly, x0[2] % lx, c] = 1.0
    return psi


@functools.cache
def _context():
    return tl.Context(0)


def _field(ctx, prec, L, U, W=None):
    if prec.endswith("-onelink"):
        return ctx.pack_links(L, U, prec, W=W)
    return ctx.build_twolinks(L, U, prec, W=W)


def prepare(case, seed):
    ctx = _context()
    kind = case["kind"]
    if kind == "reduce":
        (shape,) = _shapes(case)
        n = case["per_slice"]
        psi = _sources(shape, n, 3, "normal", seed, 0)
        phi = _sources(shape, n, 3, "normal", seed, 1)
        return {"case": case, "ctx": ctx, "psi": psi, "phi": phi}
    if kind == "lap":
        (shape,) = _shapes(case)
        U = _links(shape, 1, case["links"], seed, 0)
        L = shape + (1,)
        return {"case": case, "ctx": ctx, "L": L, "W": _field(ctx, case["prec"], L, U),
                "psi": _sources(shape, 1, 1, case["source"], seed, 0)[0]}
    if kind == "build":
        (shape,) = _shapes(case)
        L = shape + (case["slices"],)
        W = torch.zeros(tl.twolinks_bytes(L, case["prec"]), dtype=torch.uint8, device="cuda")
        return {"case": case, "ctx": ctx, "L": L, "U": _links(shape, case["slices"], case["links"], seed, 0), "W": W}
    jobs, sources, links = [], [], []
    for k, (shape, n_slices) in enumerate(zip(_shapes(case), _slices(case))):
        U = _links(shape, n_slices, case["links"], seed, k)
        L = shape + (n_slices,)
        ts = [t for t in range(n_slices) for _ in range(case["per_slice"])]
        src = _sources(shape, len(ts), case["per_slice"], case["source"], seed, k)
        jobs.append(tl.Job(L, _field(ctx, case["prec"], L, U), ts, torch.empty_like(src)))
        sources.append(src)
        links.append(U if case["build"] else None)
    state = {"case": case, "ctx": ctx, "jobs": jobs, "sources": sources, "links": links}
    if kind == "smear":
        state["plan"] = ctx.plan(jobs, case["n"], case["sigma"], case["prec"], KEEP)
    return state


# ------------------------------------------------------------------ one pass

def run(state):
    case, ctx = state["case"], state["ctx"]
    kind = case["kind"]
    if kind == "reduce":
        return [ctx.reduce("dot", state["psi"], state["phi"]), ctx.reduce("norm2", state["psi"]),
                ctx.reduce("site_norm", state["psi"])]
    if kind == "lap":
        return ctx.laplacian(state["L"], state["W"], case["prec"], 0, state["psi"])
    if kind == "build":
        return ctx.build_twolinks(state["L"], state["U"], case["prec"], W=state["W"])
    jobs = state["jobs"]
    for job, src in zip(jobs, state["sources"]):      # new sources for this pass
        job.psi.copy_(src)
    if kind == "call":
        ctx.smear(jobs, case["n"], case["sigma"], case["prec"])
        return [job.psi for job in jobs]
    for job, U in zip(jobs, state["links"]):
        if U is not None:
            _field(ctx, case["prec"], job.L, U, W=job.W)
    plan = state["plan"]
    plan.load()
    plan.run()
    norms = [plan.reduce("norm2")] if case["build"] else []
    plan.store()
    return [job.psi for job in jobs] + norms


# ------------------------------------------------------------------ work and exact results

def _reals(prec, what):
    """Stored bytes per site of a link (per direction) or a colour vector."""
    base = prec.split("-")[0]
    if what == "psi":
        return {"f64": 48, "f32": 24, "f16s": 16, "bf16": 12}[base]
    if "-w12" in prec:
        return {"f64": 96, "f32": 48, "f16s": 24, "bf16": 24}[base]
    return {"f64": 144, "f32": 72, "f16s": 40, "bf16": 36}[base]


def work(case):
    kind = case["kind"]
    shapes = _shapes(case)
    vols = [s[0] * s[1] * s[2] for s in shapes]
    if kind == "reduce":
        n = case["per_slice"] * vols[0]
        return {"bytes": (2 * 48 + 8) * n, "flops": (24 + 12) * n}
    w = 3 * _reals(case["prec"], "w")
    if kind == "lap":
        return {"bytes": vols[0] * (w + 96), "flops": 444 * vols[0]}
    if kind == "build":
        n = case["slices"] * vols[0]
        return {"bytes": n * (432 + w), "flops": 594 * n}
    sites = [v * k for v, k in zip(vols, _slices(case))]
    rhs = [s * case["per_slice"] for s in sites]
    per_site = w + (432 + w if case["build"] else 0)
    return {"bytes": sum(sites) * per_site + sum(rhs) * 96,
            "flops": 444 * case["n"] * sum(rhs) + (594 * sum(sites) + 12 * sum(rhs) if case["build"] else 0)}


def _hops(W, psi, dist):
    """sum_mu W_mu(x) psi(x + dist mu) + W_mu^dag(x - dist mu) psi(x - dist mu); psi [r][z][y][x][3], W [z][y][x][3][a][b]."""
    out = torch.zeros_like(psi)
    for mu in range(3):
        axis = 3 - mu
        m = W[..., mu, :, :]
        out += (m * torch.roll(psi, -dist, axis)[..., None, :]).sum(-1)
        out += torch.roll((m.conj().transpose(-1, -2) * psi[..., None, :]).sum(-1), dist, axis)
    return out


def _two_links(U):
    """W_mu(x) = U_mu(x) U_mu(x + mu) of one slice [z][y][x][mu][a][b]."""
    out = []
    for mu in range(3):
        a = U[..., mu, :, :]
        b = torch.roll(a, -1, 2 - mu)
        out.append((a[..., :, :, None] * b[..., None, :, :]).sum(-2))
    return torch.stack(out, dim=-3)


def exact(case, seed):
    kind = case["kind"]
    if kind == "build":
        return None                  # a packed field: compared byte by byte
    if kind == "reduce":
        (shape,) = _shapes(case)
        n = case["per_slice"]
        psi = _sources(shape, n, 3, "normal", seed, 0).view(n, -1)
        phi = _sources(shape, n, 3, "normal", seed, 1).view(n, -1)
        squares = psi.real ** 2 + psi.imag ** 2
        lx, ly, lz = shape
        return [(phi.conj() * psi).sum(-1), squares.sum(-1), squares.view(n, lz, ly, lx, 3).sum(-1).sqrt()]
    one = case["prec"].endswith("-onelink")
    dist, quarter = (1, 1.0) if one else (2, 0.25)
    if kind == "lap":
        (shape,) = _shapes(case)
        U = _links(shape, 1, case["links"], seed, 0)[0]
        psi = _sources(shape, 1, 1, case["source"], seed, 0)
        W = U[..., :3, :, :] if one else _two_links(U)
        return (quarter * (_hops(W, psi, dist) - 6.0 * psi))[0]
    outs, norms = [], []
    for k, (shape, n_slices) in enumerate(zip(_shapes(case), _slices(case))):
        U = _links(shape, n_slices, case["links"], seed, k)
        per = case["per_slice"]
        psi = _sources(shape, n_slices * per, per, case["source"], seed, k)
        for t in range(n_slices):
            W = U[t, ..., :3, :, :].contiguous() if one else _two_links(U[t])
            v = psi[t * per:(t + 1) * per]
            for _ in range(case["n"]):
                v = v + (case["sigma"] / case["n"] * quarter) * (_hops(W, v, dist) - 6.0 * v)
            psi[t * per:(t + 1) * per] = v
        outs.append(psi)
        norms.append((psi.real ** 2 + psi.imag ** 2).sum((1, 2, 3, 4)))
    return outs + ([torch.cat(norms)] if case["build"] else [])
