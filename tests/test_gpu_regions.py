"""Whether a grid lies in one region is found chunk by chunk (32768 cells) when the
context is created; and the DMI forms of the x passes with and without the
one-region epilogue, which six-wave workgroups (1024 points) do not have.

Tolerances of test_gpu_x_quads.py."""
import numpy as np
import pytest

from paper_1406_7635_amd import synth
from tests.gpu_helpers import log, make_pair, rel_inf, to_np
from tests.test_gpu_x_quads import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("odd_cell", [None, 0, 32767, 32768, -1])
def test_odd_cell_in_any_chunk(gpu, odd_cell):
    grid = (200, 328, 1)  # 65600 cells: two whole chunks and 64 cells
    case = synth.random_problem(grid, (2e-9, 2.5e-9, 3e-9), seed=3, nregions=4)
    case["region"][:] = 2
    if odd_cell is not None:
        case["region"].reshape(-1)[odd_cell] = 3
    ctx, prob, m = make_pair(case)
    e = rel_inf(to_np(ctx.beff(m)), prob.beff(case["m0"].astype(np.float64)))
    log("odd cell", odd_cell, "B_eff %.1e" % e)
    assert e < 1e-5
    ctx.close()


@pytest.mark.parametrize("nregions", [1, 3])
@pytest.mark.parametrize("grid,pbc", [((512, 6, 1), (0, 0, 0)), ((1024, 4, 1), (1, 0, 0)), ((256, 8, 2), (0, 0, 0)),
                                      ((512, 10, 1), (1, 1, 0))])
def test_dmi_forms(gpu, grid, pbc, nregions):
    check(grid, pbc, nregions, True)
