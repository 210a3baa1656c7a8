"""The far entries of the demagnetising tensor across the bands of its
quadrature order (edges at 2.5, 4, 6, 12, 24 and 80 cell diagonals).

Reference: the dipole tensor under the triangular density with 12
Gauss-Legendre points on each half axis, in extended precision (below 5e-15
from 2.5 diagonals on).  The rules stay within 6e-12 of a cell's largest
component at the near edge of their bands; FP64 sums of at most 1331 terms add
some 1e-13, so 1.2e-11."""
import numpy as np
import pytest

from paper_1406_7635_amd import mm, synth
from tests.gpu_helpers import log, to_np

pytestmark = pytest.mark.gpu


def reference(r, cell):
    x, w = np.polynomial.legendre.leggauss(12)
    s = (0.5 * (1 + x)).astype(np.longdouble)
    d = 0.5 * w * (1 - s)
    s, d = np.concatenate([s, -s]), np.concatenate([d, d])
    u = [r[a] + s * np.longdouble(cell[a]) for a in range(3)]
    ux, uy, uz = u[0][:, None, None], u[1][None, :, None], u[2][None, None, :]
    r2 = ux * ux + uy * uy + uz * uz
    f = d[:, None, None] * d[None, :, None] * d[None, None, :] / (r2 * r2 * np.sqrt(r2))
    xx, yy, zz = (f * ux * ux).sum(), (f * uy * uy).sum(), (f * uz * uz).sum()
    off = [3 * (f * a * b).sum() for a, b in ((ux, uy), (ux, uz), (uy, uz))]
    pre = -np.longdouble(cell[0]) * cell[1] * cell[2] / (4 * np.pi)
    return np.array([pre * v for v in [2 * xx - yy - zz, 2 * yy - xx - zz, 2 * zz - xx - yy] + off], dtype=float)


@pytest.mark.parametrize("grid,cell", [((200, 3, 2), (2.0, 2.0, 2.0)), ((24, 30, 12), (3.0, 2.0, 2.5)),
                                       ((2, 260, 3), (4.0, 1.0, 0.5)), ((3, 4, 300), (1.0, 8.0, 5.0)),
                                       ((60, 2, 9), (20.0, 1.0, 1.0))])
def test_far_entries(gpu, grid, cell):
    nx, ny, nz = grid
    ctx = mm.Context(grid, tuple(c * 1e-9 for c in cell), np.zeros((nz, ny, nx), np.uint8), synth.material(8e5, 1e-11),
                     demag=False)
    got = to_np(ctx.tensor_dump())
    k, j, i = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    r = np.stack([i * cell[0], j * cell[1], k * cell[2]])
    rho = np.sqrt((r * r).sum(0)) / np.sqrt(sum(c * c for c in cell))
    rng = np.random.default_rng(sum(grid))
    pick = []
    for edge in (2.5, 4, 6, 12, 24, 80):  # the entries just past each edge, and some further out
        far = np.argwhere(rho >= edge * (1 + 1e-9))
        order = np.argsort(rho[tuple(far.T)])
        pick += [tuple(far[o]) for o in order[:6]] + [tuple(far[o]) for o in rng.permutation(order)[:6]]
    worst = 0.0
    for p in pick:
        ref = reference([r[a][p] for a in range(3)], cell)
        worst = max(worst, np.max(np.abs(got[(slice(None),) + p] - ref)) / np.max(np.abs(ref)))
    log("demag orders", grid, cell, "entries", len(pick), "worst %.1e" % worst)
    assert len(pick) >= 36 and worst < 1.2e-11
    ctx.close()
