"""The staged 3D column passes at the ends of their lengths.  z convolution: 4 and
8 points (2 to 4 layers with more rows than the one-pass y/z form takes), where
a plane of a tile has more 16-byte chunks than the workgroup has threads, and a
single column per kx (one row of cells).  y transforms: 1, 4, 8, 16, 32 and 64
points, where columns are shorter than a wave, and 1024 and 2048.

Against the oracle with the tolerance of test_gpu_columns.py; an ensemble's
member, which takes the per-component form, must equal the single grid bit for
bit."""
import pytest

from paper_1406_7635_amd import mm, synth
from tests.gpu_helpers import log, make_pair, rel_inf, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", [(40, 600, 2), (70, 600, 2), (40, 600, 3), (140, 300, 4), (600, 1, 150),
                                  (1000, 2, 70), (1000, 3, 70), (900, 7, 40), (600, 10, 30), (300, 20, 40)])
def test_field_matches_oracle(gpu, grid):
    import numpy as np

    case = synth.random_problem(grid, (2e-9, 3e-9, 2.5e-9), seed=6, nregions=3, vacuum=True)
    ctx, prob, m = make_pair(case)
    b, bd = ctx.beff(m, want_demag=True)
    e = rel_inf(to_np(b), prob.beff(case["m0"].astype(np.float64)))
    ed = rel_inf(to_np(bd), prob.demag_field(case["m0"].astype(np.float64)))
    log("short columns %s: B_eff %.1e B_demag %.1e" % (grid, e, ed))
    assert e < 1e-5 and ed < 1e-5
    ctx.close()


def test_members_equal_single_grids(gpu):
    import torch

    grids = [(140, 300, 4), (150, 300, 3), (200, 512, 4)]
    cases = [synth.random_problem(g, (3e-9, 3e-9, 3e-9), seed=17 + i) for i, g in enumerate(grids)]
    b = mm.Batch(cases)
    got = b.beff(b.pack([c["m0"] for c in cases]))
    for i, c in enumerate(cases):
        ctx = mm.Context(c["grid"], c["cell"], c["region"], c["params"])
        one = ctx.beff(torch.from_numpy(c["m0"]).to("cuda:0"))
        assert torch.equal(one.reshape(-1), b.member(got, i).reshape(-1)), c["grid"]
        ctx.close()
    b.close()
