"""The x passes that take four cells per access, on both sides of their rule
(nx a multiple of four, ny even, a narrow workgroup) and with one region, where
regions and pair coefficients are not read, against several.

B_eff within 1e-5 of its largest value of the oracle's (FP32 transforms: at most
2 x 12 radix-2 levels with one rounding of 6e-8 each stay below 1.5e-6), and m
after three Dormand-Prince attempts at a fixed step within 2e-6 (unit vectors
in FP32; the fused pass runs in every attempt)."""
import numpy as np
import pytest

from oracle import fields as ofields
from oracle import integrate as ointegrate
from paper_1406_7635_amd import mm, synth
from tests.gpu_helpers import log, rel_inf, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nregions", [1, 3])
@pytest.mark.parametrize("pbc", [(0, 0, 0), (1, 1, 0)])
@pytest.mark.parametrize("grid", [(4, 2, 1), (4, 3, 1), (8, 2, 2), (12, 6, 1), (16, 10, 3), (60, 34, 1), (62, 34, 1),
                                  (64, 35, 1), (128, 64, 1), (260, 20, 2), (1024, 4, 1), (1028, 6, 1)])
def test_field_and_steps_match_oracle(gpu, grid, pbc, nregions):
    check(grid, pbc, nregions, False)


@pytest.mark.parametrize("nregions", [1, 3])
@pytest.mark.parametrize("grid,pbc", [((12, 6, 1), (0, 0, 0)), ((16, 10, 3), (1, 0, 0)), ((60, 34, 1), (0, 1, 0)),
                                      ((62, 34, 1), (0, 0, 0)), ((64, 64, 1), (1, 1, 0)), ((1028, 6, 1), (0, 0, 0))])
def test_field_and_steps_with_dmi(gpu, grid, pbc, nregions):
    check(grid, pbc, nregions, True)


def check(grid, pbc, nregions, dmi):
    import torch

    case = synth.random_problem(grid, (2e-9, 2.5e-9, 3e-9), seed=sum(grid) + nregions, nregions=nregions,
                                vacuum=nregions > 1)
    if dmi:
        case["params"]["dind"] = np.zeros(256)
        case["params"]["dind"][:nregions] = [2e-3, -1e-3, 3e-3][:nregions]
    log("x quads", grid, pbc, nregions, dmi)
    ctx = mm.Context(case["grid"], case["cell"], case["region"], case["params"], pbc=pbc)
    prob = ofields.Problem(case["grid"], case["cell"], case["region"], case["params"], pbc=pbc)
    m = torch.from_numpy(np.ascontiguousarray(case["m0"])).to("cuda:0")
    m_ref = case["m0"].astype(np.float64)
    e = rel_inf(to_np(ctx.beff(m)), prob.beff(m_ref))
    assert e < 1e-5
    f = prob.torque
    k1 = f(m_ref)
    t, dt = 0.0, 2e-14
    opts = mm.solver_opts(max_err=1.0)
    for _ in range(3):
        acc, t, _, _ = ctx.rk45_step(m, t, dt, opts)
        assert acc
        ms, k1, _ = ointegrate.embedded_step(f, m_ref, k1, dt, ointegrate.DP45)
        m_ref = ointegrate.normalize(ms)
    d = float(np.max(np.abs(to_np(m) - m_ref)))
    log("  B_eff %.1e, |dm| %.2e" % (e, d))
    assert d < 2e-6
    ctx.close()
