"""Tuned tilings by step count: a short plan's entry, or one of a cache file from before whole-run
launches, does not decide for a long plan; step counts of one power of two share an entry."""
import json

import numpy as np
import pytest

from paper_2301_05518_amd import synth
from tests.gpu_common import log, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


def tuned(c, n, flags=0):
    """The variant and (sweeps, hits) of a tuned plan of n steps on 8^3 (a launch costs 5 us there, a step of a
    whole run 1 to 2 us)."""
    import paper_2301_05518_amd as tl
    L = (8, 8, 8, 1)
    U = synth.gauge_field(L, "haar", 9900)
    psi = to_dev(synth.random_field(np.random.default_rng([9900]), (3, 8, 8, 8, 3)))
    plan = c.plan([tl.Job(L, c.build_twolinks(L, to_dev(U), "f32"), [0, 0, 0], psi)], n, 0.1 * n, "f32", tl.TL_AUTOTUNE | flags)
    plan.load()
    plan.run()
    c.sync()
    variant = plan.info()["variant"]
    plan.close()
    st = c.stats()
    log(f"n={n} flags {flags}: variant {variant}, {st['tune_sweeps']} sweeps, {st['tune_hits']} hits")
    return variant, (st["tune_sweeps"], st["tune_hits"])


def test_short_plan_first(torch):
    import paper_2301_05518_amd as tl
    c = tl.Context(0)
    assert tuned(c, 2)[1] == (1, 0)
    assert tuned(c, 20) == (9, (2, 0))
    assert tuned(c, 31) == (9, (2, 1))
    assert tuned(c, 3)[1] == (2, 2)
    assert tuned(c, 60) == (9, (3, 2))
    assert tuned(c, 1000) == (9, (3, 3))
    # one step per launch: the step count decides nothing
    assert tuned(c, 2, tl.TL_ONE_STEP)[1] == (4, 3)
    assert tuned(c, 60, tl.TL_ONE_STEP)[1] == (4, 4)
    c.close()


def test_older_cache_file(torch, monkeypatch, tmp_path):
    import paper_2301_05518_amd as tl
    cache = tmp_path / "tune.json"
    monkeypatch.setenv("TL_TUNE_CACHE", str(cache))
    c = tl.Context(0)
    tuned(c, 20)
    c.close()
    (key,) = json.loads(cache.read_text())
    assert "|c2" in key and "|n16" in key
    old = key.replace("|c2", "").replace("|n16", "")
    cache.write_text(json.dumps({old: "0,256,4,0,0,0"}))
    c = tl.Context(0)
    assert tuned(c, 20) == (9, (1, 0))
    c.close()
    assert json.loads(cache.read_text())[key].startswith("9,")


def test_tuning_time_does_not_grow_with_the_steps(torch):
    import time

    import paper_2301_05518_amd as tl
    took = {}
    for n in (64, 20001):      # 200 launches of 20001 steps would take more than 4 s
        c = tl.Context(0)
        c.sync()
        t0 = time.perf_counter()
        assert tuned(c, n) == (9, (1, 0))
        took[n] = time.perf_counter() - t0
        c.close()
    log(f"tuning took {took}")
    assert took[20001] < 3 * took[64] + 0.5
