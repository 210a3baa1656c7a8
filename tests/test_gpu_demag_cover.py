"""Every entry of the demagnetising tensor is written by one of its two kernels,
also where the distance is exactly the one at which they meet (12 cell
diagonals): cubic cells hold displacements (12, 12, 12) and (20, 4, 4) there,
cells of 3 x 4 x 12 (diagonal 13) the ones with |d| = 156, such as (52, 0, 0).

The output is filled with NaN before the call.  Entries at that distance against
the dipole tensor under the triangular density, with the tolerance of
test_gpu_demag_orders.py."""
import numpy as np
import pytest

from paper_1406_7635_amd import mm, synth
from tests.gpu_helpers import log, to_np
from tests.test_gpu_demag_orders import reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,cell", [((23, 22, 21), (2.0, 2.0, 2.0)), ((23, 22, 21), (0.7, 0.7, 0.7)),
                                       ((60, 42, 15), (3.0, 4.0, 12.0)), ((21, 13, 13), (1.1, 1.1, 1.1))])
def test_every_entry_is_written(gpu, grid, cell):
    import torch

    nx, ny, nz = grid
    ctx = mm.Context(grid, tuple(c * 1e-9 for c in cell), np.zeros((nz, ny, nx), np.uint8), synth.material(8e5, 1e-11),
                     demag=False)
    out = torch.full((6, nz, ny, nx), float("nan"), dtype=torch.float64, device="cuda:0")
    mm._check(mm.load().mm_demag_tensor_dump(ctx._h, mm._ptr(out)), "mm_demag_tensor_dump")
    torch.cuda.synchronize()
    got = to_np(out)
    ctx.close()
    assert np.isfinite(got).all()
    k, j, i = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    r = np.stack([i * cell[0], j * cell[1], k * cell[2]])
    rho = np.sqrt((r * r).sum(0)) / np.sqrt(sum(c * c for c in cell))
    edge = np.argwhere(np.abs(rho - 12) < 1e-9)
    assert len(edge) >= 2
    for p in map(tuple, edge):
        ref = reference([r[a][p] for a in range(3)], cell)
        err = np.max(np.abs(got[(slice(None),) + p] - ref)) / np.max(np.abs(ref))
        log("tensor at 12 diagonals", grid, p, "%.1e" % err)
        assert err < 1.2e-11
