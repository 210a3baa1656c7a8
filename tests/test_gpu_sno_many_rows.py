"""The training kernels on more rows than one round of workgroups takes: a
workgroup of the row passes then carries its weight sums from one group of
rows to the next, and nothing may be lost or counted twice between them.

Gradients of random samples against reverse-mode differentiation of the
network in FP64, on grids with more than 512 row groups that do not divide
evenly (one row per group, and four).  The forward values are within 1e-5 of
their largest (test_gpu_sno_rows.py), the backward pass has as many sums
again, and FP32 chains of at most 512 pixels add 3.1e-5: 5e-5 of the largest
component of a parameter group.  A row left out would show as its share of a
component, some 1e-3."""
import numpy as np
import pytest

from oracle import sno as osno
from paper_1406_7635_amd import mm, synth
from tests.gpu_helpers import log
from tests.test_gpu_sno_train import groups

pytestmark = pytest.mark.gpu


def fp64_gradient(w, m, t):
    """Gradient of the mean relative L2 error by reverse-mode differentiation in FP64."""
    import torch

    flat = torch.tensor(w, dtype=torch.float64, requires_grad=True)
    c, kx, ky = osno.C, osno.KX, osno.KY
    m, t = torch.tensor(m, dtype=torch.float64), torch.tensor(t, dtype=torch.float64)
    nx, ny = m.shape[3], m.shape[2]
    px = torch.arange(kx, dtype=torch.float64)[:, None] * torch.arange(nx, dtype=torch.float64) * (2 * np.pi / nx)
    py = torch.arange(-ky // 2, ky // 2, dtype=torch.float64)[:, None] * torch.arange(ny, dtype=torch.float64) \
        * (2 * np.pi / ny)
    ex, ey = torch.polar(torch.ones_like(px), -px), torch.polar(torch.ones_like(py), -py)  # [k][x], [j][y]
    wk = torch.full((kx,), 2.0 / (nx * ny), dtype=torch.float64)
    wk[0] *= 0.5
    o = 0

    def take(*shape):
        nonlocal o
        n = int(np.prod(shape))
        o += n
        return flat[o - n:o].reshape(shape)

    h = torch.tensordot(take(c, 3), m, ([1], [1])).movedim(0, 1) + take(c)[:, None, None]
    for _ in range(osno.NLAYER):
        r = torch.view_as_complex(take(ky, kx, c, c, 2).contiguous())
        wl, b = take(c, c), take(c)
        hh = ey @ (h.to(torch.complex128) @ ex.T.contiguous())                  # [b][c][j][k]
        hh = hh.permute(2, 3, 1, 0).contiguous()                                # [j][k][c][b]
        gh = (r @ hh).permute(3, 2, 0, 1).contiguous()                          # [b][o][j][k]
        g = (ey.conj().T.contiguous() @ (gh * wk) @ ex.conj().contiguous()).real
        z = g + torch.tensordot(wl, h, ([1], [1])).movedim(0, 1) + b[:, None, None]
        h = torch.nn.functional.gelu(z)
    y = torch.tensordot(take(3, c), h, ([1], [1])).movedim(0, 1) + take(3)[:, None, None]
    d, n = (y - t).flatten(1), t.flatten(1)
    loss = (torch.linalg.norm(d, dim=1) / torch.linalg.norm(n, dim=1)).mean()
    loss.backward()
    return float(loss.detach()), flat.grad.numpy()


@pytest.mark.parametrize("nx,ny,batch", [(257, 130, 5), (33, 131, 17)])
def test_gradient_many_row_groups(gpu, nx, ny, batch):
    import torch

    w = synth.sno_random_weights(51, scale=0.7)
    rng = np.random.Generator(np.random.PCG64(52))
    m = synth.film_textures(batch, seed=53, grid=(nx, ny), cell=4e-9)[:, :, 0].astype(np.float32)
    t = (0.3 * rng.standard_normal((batch, 3, ny, nx))).astype(np.float32)
    tr = mm.SurrogateTrainer(nx, ny, batch, w)
    loss, g = tr.grad(torch.from_numpy(m).cuda(), torch.from_numpy(t).cuda())
    g = g.cpu().numpy().astype(np.float64)
    tr.close()
    loss_ref, ref = fp64_gradient(w.astype(np.float64), m, t)
    assert loss == pytest.approx(loss_ref, rel=2e-6)
    for name, lo, hi in groups():
        err = np.max(np.abs(g[lo:hi] - ref[lo:hi])) / np.max(np.abs(ref[lo:hi]))
        log("grad %dx%dx%d %-3s rel %.1e" % (nx, ny, batch, name, err))
        assert err < 5e-5, name
