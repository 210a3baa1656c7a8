"""The training kernels' sums over pixels where a workgroup of the row passes
takes many rows: their rounding must not grow with the batch.

Constant samples (m, t and every activation the same at all pixels, no
spectral weights) make each term of a weight gradient equal, the worst case of
an FP32 sum: its rounding errors all have one sign.  With the gradient of a
pixel in FP64 as reference: an FP32 chain of at most 512 pixels, finished in
FP64, is off by less than 512 x 2^-24 = 3.1e-5; a term itself went through four
layers of 65-term sums forward and 33-term sums back, each within 2^-24 per
term, 4 x 98 x 6e-8 = 2.3e-5: together 5.4e-5."""
import numpy as np
import pytest

from oracle import sno as osno
from paper_1406_7635_amd import mm
from tests.gpu_helpers import log

pytestmark = pytest.mark.gpu


def pixel_gradient(w, m, t):
    """FP64 gradient of the loss for constant samples m, t (3 values each) without spectral weights."""
    import torch

    p = {k: [torch.tensor(x.real, requires_grad=True) for x in v] if isinstance(v, list)
         else torch.tensor(v, requires_grad=True) for k, v in w.items()}
    h = p["P"] @ torch.tensor(m) + p["p"]
    for wl, b in zip(p["W"], p["b"]):
        h = torch.nn.functional.gelu(wl @ h + b)
    y = p["Q"] @ h + p["q"]
    loss = torch.linalg.norm(y - torch.tensor(t)) / torch.linalg.norm(torch.tensor(t))
    loss.backward()
    return float(loss.detach()), {k: [x.grad for x in v] if isinstance(v, list) else v.grad for k, v in p.items()}


def test_long_sums(gpu):
    import torch

    nx = ny = 512
    batch = 128  # 128 rows of 512 pixels per workgroup: 8192 pixels per wave
    rng = np.random.Generator(np.random.PCG64(3))
    w = osno.unpack(np.zeros(osno.weight_count()))
    w = {k: ([x.copy() for x in v] if isinstance(v, list) else v.copy()) for k, v in w.items()}
    f32 = lambda a: a.astype(np.float32).astype(np.float64)
    w["P"], w["p"] = f32(rng.standard_normal((32, 3))), f32(rng.standard_normal(32))
    w["W"] = [f32(rng.standard_normal((32, 32)) / 6) for _ in range(osno.NLAYER)]
    w["b"] = [f32(0.5 + 0.3 * rng.standard_normal(32)) for _ in range(osno.NLAYER)]
    w["Q"], w["q"] = f32(rng.standard_normal((3, 32)) / 6), f32(rng.standard_normal(3))
    mv, tv = f32(np.array([0.36, -0.48, 0.8])), f32(np.array([0.7, 1.3, -0.4]))
    loss_ref, ref = pixel_gradient(w, mv, tv)
    const = lambda v: torch.tensor(v, dtype=torch.float32, device="cuda:0").reshape(1, 3, 1, 1).expand(
        batch, 3, ny, nx).contiguous()
    tr = mm.SurrogateTrainer(nx, ny, batch, osno.pack(w).astype(np.float32))
    loss, g = tr.grad(const(mv), const(tv))
    got = osno.unpack(g.cpu().numpy())
    tr.close()
    assert loss == pytest.approx(loss_ref, rel=2e-6)
    for name in ("P", "p", "W", "b", "Q", "q"):
        pairs = list(zip(got[name], ref[name])) if name in "Wb" else [(got[name], ref[name])]
        for l, (a, b) in enumerate(pairs):
            b = b.numpy()
            # every component is one product: relative to the component itself
            # where it is not tiny (a product of factors near zero keeps their
            # absolute errors)
            big = np.abs(b) > 1e-2 * np.abs(b).max()
            err = np.max(np.abs(a - b)[big] / np.abs(b)[big])
            log("long sums %s%d: rel %.1e over %d components" % (name, l, err, big.sum()))
            assert err < 5.4e-5, (name, l)
