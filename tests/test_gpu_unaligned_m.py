"""The four-cell loads of the x passes take m at any float address: a tensor that
starts 4, 8 or 12 bytes past a 16-byte boundary gives the same field and the
same step, bit for bit."""
import pytest

from paper_1406_7635_amd import synth
from tests.gpu_helpers import make_ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", [(64, 64, 1), (512, 512, 1), (32, 32, 4), (40, 30, 7)])
def test_offset_tensors(gpu, grid):
    import torch

    ctx, m = make_ctx(synth.random_problem(grid, (3e-9, 3e-9, 3e-9), seed=3))
    field = ctx.beff(m)
    step = m.clone()
    ctx.reset_solver()
    ctx.rk45_step(step, 0.0, 1e-14)
    n = m.numel()
    for off in (1, 2, 3):
        v = torch.zeros(n + 8, device="cuda:0")[off:off + n].view(m.shape)
        v.copy_(m)
        assert v.data_ptr() % 16 == 4 * off
        assert torch.equal(ctx.beff(v), field)
        ctx.reset_solver()
        ctx.rk45_step(v, 0.0, 1e-14)
        assert torch.equal(v, step)
    ctx.close()
