"""The surrogate's row passes at the sizes where their tiling can go wrong:
rows shorter than, equal to and just past a 32-pixel tile, tile counts that are
no power of two, the largest rows, odd numbers of rows and samples, against the
FP64 oracle of the network (forward) and central differences of its loss
(gradient).

Tolerances: a value passes four layers of sums of at most 32 + 33 + nx + ny
FP32 terms; with one rounding of 6e-8 per term, growing like the square root
of their number, that is 4 x 6e-8 x sqrt(1100) < 1e-5 of the largest value.
Gradients: the 2e-3 of the difference quotient, as in test_gpu_sno_train.py."""
import numpy as np
import pytest

from oracle import sno
from paper_1406_7635_amd import mm, synth
from tests.gpu_helpers import log, rel_inf, to_np
from tests.test_gpu_sno import bf16_round
from tests.test_gpu_sno_train import groups, oracle_loss

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", [(32, 16), (33, 17), (64, 31), (65, 128), (160, 33), (257, 19), (512, 512)])
def test_forward_at_tile_edges(gpu, grid):
    import torch

    nx, ny = grid
    w = bf16_round(synth.sno_random_weights(31))
    m = synth.random_sphere((nx, ny, 1), 32)
    s = mm.Surrogate(nx, ny, w, out_scale=1.5)
    got = to_np(s(torch.from_numpy(m).to("cuda:0")))[:, 0]
    err = rel_inf(got, 1.5 * sno.forward(w.astype(np.float64), m))
    log("surrogate rows %dx%d: rel %.2e" % (nx, ny, err))
    assert err < 1e-5
    s.close()


@pytest.mark.parametrize("nx,ny,batch", [(33, 17, 3), (95, 16, 1), (288, 18, 2)])
def test_gradient_at_tile_edges(gpu, nx, ny, batch):
    import torch

    w = synth.sno_random_weights(41, scale=0.7).astype(np.float64)
    rng = np.random.Generator(np.random.PCG64(42))
    m = synth.film_textures(batch, seed=43, grid=(nx, ny), cell=4e-9)[:, :, 0].astype(np.float32)
    t = (0.3 * rng.standard_normal((batch, 3, ny, nx))).astype(np.float32)
    tr = mm.SurrogateTrainer(nx, ny, batch, w)
    loss, g = tr.grad(torch.from_numpy(m).cuda(), torch.from_numpy(t).cuda())
    g = g.cpu().numpy().astype(np.float64)
    m, t = m.astype(np.float64), t.astype(np.float64)
    assert loss == pytest.approx(oracle_loss(w, m, t), rel=2e-6)
    for name, lo, hi in groups():
        v = np.zeros_like(w)
        v[lo:hi] = rng.standard_normal(hi - lo)
        eps = 1e-4 / max(1.0, np.linalg.norm(v[lo:hi]) / np.sqrt(hi - lo))
        fd = (oracle_loss(w + eps * v, m, t) - oracle_loss(w - eps * v, m, t)) / (2 * eps)
        got = float(np.dot(g, v))
        scale = max(abs(fd), np.linalg.norm(g[lo:hi]) * np.linalg.norm(v[lo:hi]) / np.sqrt(hi - lo))
        log("grad %dx%d %-3s <g,v> %.6e finite difference %.6e" % (nx, ny, name, got, fd))
        assert abs(got - fd) <= 2e-3 * scale, name
    tr.close()
