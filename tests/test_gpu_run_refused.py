"""Which whole-run tilings apply to which lattices: exactly the expected ones are refused, so that a
comparison that skips refused tilings does not lose any unnoticed."""
import pytest

from tests.gpu_common import log
from tests.test_gpu_run import TILES, lattices, smear

pytestmark = pytest.mark.gpu

PARTS = {"all": slice(None), "small": slice(0, 3), "32x24x20": slice(3, 4), "26x11x24": slice(4, 5)}

# tile -> parts whose cells do not fit.  Two-link cells of 32x24x20 and 26x11x24 have 1920 and 1716
# sites, one-link ones 15360 and 6864 and one chain each; four RHS on threads of their own leave 128
# of 512 threads for the sites of each, three 128 as well, two sets 256.  FP64 holds 27 link words a
# site in LDS, which bounds its tiles further.
SETS_OF_4 = "9,512,8,64,0,1"
TWO = {SETS_OF_4: {"all", "26x11x24"}}
TWO_F64 = {SETS_OF_4: {"all", "32x24x20", "26x11x24"}}
CUT = {"all", "32x24x20", "26x11x24"}
ONE = {SETS_OF_4: CUT, "9,256,64,0,0,1": CUT, "9,512,32,0,1,0": {"all", "32x24x20"}}
ONE_F64 = {SETS_OF_4: CUT, "9,256,64,0,0,1": CUT, "9,512,32,0,1,0": CUT, "9,512,32,0,0,0": CUT,
           "9,512,64,8,0,0": {"all", "32x24x20"}}
EXPECTED = {"f64": TWO_F64, "f32": TWO, "f16s": TWO, "bf16": TWO, "f32-w12": TWO, "f64-w12": TWO_F64,
            "f32-onelink": ONE, "f64-onelink": ONE_F64, "bf16-w12-onelink": ONE}


@pytest.mark.parametrize("prec", list(EXPECTED))
def test_refused_tilings(monkeypatch, prec):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2301_05518_amd as tl
    ctx = tl.Context(0)
    lats = lattices(10)
    refused = {}
    for tile in TILES:
        monkeypatch.setenv("TL_TILE", tile)
        for name, part in PARTS.items():
            try:
                info, _ = smear(ctx, torch, lats[part], 5, 0.5, prec)
                assert info["variant"] == 9
            except tl.TwolinkError as e:
                assert "TL_ERR_UNSUPPORTED" in str(e) and "does not fit" in str(e)
                refused.setdefault(tile, set()).add(name)
    log(f"{prec}: refused {refused}")
    assert refused == EXPECTED[prec]
    ctx.close()
