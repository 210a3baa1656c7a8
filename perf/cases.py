"""Measured workloads of the library, called through its public entry points.

Each listed case stands for something a simulation does in earnest:

  film64_run            the throughput workload at a small size: Dormand-Prince attempts on 64 x 64 x 1,
                        where the latency of an attempt counts, not its bytes
  film1024_run          the benchmark film: Dormand-Prince attempts on the 1024 x 1024 x 1 vortex
  film_regions_observe  what a script evaluates at an output time on an odd-sized film of several
                        regions (uniaxial and cubic anisotropy, a vacuum region): torque, energies,
                        maximum torque
  thin4_rk4             fixed-step RK4 on 32 x 32 x 4, the smallest three-dimensional calls
  grains_run            Dormand-Prince attempts on 256 x 256 x 64 grains of 256 materials
  box_field             B_eff and B_demag of an odd-sized 3D box (150 x 90 x 37)
  film_periodic_run     Bogacki-Shampine attempts on a film periodic in x and y with interfacial DMI
  ensemble_run          a parameter sweep: 96 independent grids advanced together
  thermal_run           the thermal-switching workload: 512 x 512 uncoupled cells, Heun at a fixed step
  surrogate_eval        one prediction of the spectral neural operator, 256 x 256
  surrogate_grad        loss and gradient of a training batch of 16 textures, 256 x 256
  new_simulation        a new context with its demagnetising kernel, 256 x 256 x 16

The matrix-core precisions of the convolution are left out: FP32 is faster at every size and is the
default.  relax() is left out because its length depends on the last bits of the energies; its parts
(RK23 attempts, energy, maximum torque) are in other cases.

`exact` evaluates the same things in 64 bits with torch alone: Newell's closed form and Gauss-Legendre
quadrature of the dipole tensor for the demagnetising kernel, FFT convolution, the local terms, the
embedded Runge-Kutta pairs, Philox and Box-Muller for the thermal field, the network with autograd.
"""
import math

import numpy as np
import torch

from paper_1406_7635_amd import mm

MU0 = 4e-7 * math.pi
GAMMA = 1.7595e11
KB = 1.380649e-23
NREG = 256

_RUN = {"kind": "run", "pbc": 0, "dmi": 0.0, "material": "film", "init": "vortex", "dt": 1e-14}  # dt: the first step and dt_max


def listed():
    return [
        dict(_RUN, name="film64_run", nx=64, ny=64, nz=1, cell=4.0, solver=45, attempts=10),
        dict(_RUN, name="film1024_run", nx=1024, ny=1024, nz=1, cell=2.0, solver=45, attempts=4),
        {"name": "film_regions_observe", "kind": "observe", "nx": 300, "ny": 171, "nz": 1, "cell": 3.0,
         "material": "regions", "init": "random", "pbc": 0, "dmi": 0.0},
        {"name": "thin4_rk4", "kind": "rk4", "nx": 32, "ny": 32, "nz": 4, "cell": 4.0, "material": "film",
         "init": "random", "pbc": 0, "dmi": 0.0, "dt": 1e-13, "steps": 5},
        dict(_RUN, name="grains_run", nx=256, ny=256, nz=64, cell=3.0, solver=45, attempts=2, material="grains",
             init="random", dt=1e-15),
        {"name": "box_field", "kind": "field", "nx": 150, "ny": 90, "nz": 37, "cell": 3.0, "material": "regions",
         "init": "random", "pbc": 0, "dmi": 0.0},
        dict(_RUN, name="film_periodic_run", nx=512, ny=512, nz=1, cell=3.0, solver=23, attempts=4, pbc=3,
             dmi=3e-3),
        {"name": "ensemble_run", "kind": "ensemble", "members": 96, "attempts": 2, "dt": 2e-15},
        {"name": "thermal_run", "kind": "thermal", "nx": 512, "ny": 512, "nz": 1, "cell": 10.0, "coupled": False,
         "steps": 100, "dt": 1e-12},
        {"name": "surrogate_eval", "kind": "surrogate", "nx": 256, "ny": 256},
        {"name": "surrogate_grad", "kind": "train", "nx": 256, "ny": 256, "batch": 16},
        {"name": "new_simulation", "kind": "setup", "nx": 256, "ny": 256, "nz": 16, "cell": 4.0, "pbc": 0},
    ]


def _size(rng, lo, hi):
    """A length spread over the logarithm of [lo, hi]; a power of two now and then, else whatever falls, odd or not."""
    if rng.random() < 0.3:
        return 1 << rng.randint(math.ceil(math.log2(lo)), int(math.log2(hi)))
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["run", "run", "run3d", "observe", "field", "rk4", "ensemble", "thermal", "surrogate", "train",
                       "setup"])
    cell = rng.choice([2.0, 3.0, 4.0, 5.0])
    if kind == "run":
        return dict(_RUN, nx=_size(rng, 16, 1024), ny=_size(rng, 16, 1024), nz=rng.choice([1, 1, 1, 2, 3]), cell=cell,
                    solver=rng.choice([45, 45, 23]), attempts=rng.randint(2, 5), pbc=rng.choice([0, 0, 1, 3]),
                    dmi=rng.choice([0.0, 0.0, 2e-3]), material=rng.choice(["film", "regions"]))
    if kind == "run3d":
        return dict(_RUN, nx=_size(rng, 20, 256), ny=_size(rng, 20, 256), nz=_size(rng, 5, 64), cell=cell,
                    solver=rng.choice([45, 23]), attempts=2, material=rng.choice(["film", "grains"]), init="random",
                    dt=1e-15)
    if kind in ("observe", "field"):
        flat = rng.random() < 0.5
        return {"kind": kind, "nx": _size(rng, 16, 700 if flat else 200), "ny": _size(rng, 16, 700 if flat else 200),
                "nz": 1 if flat else _size(rng, 2, 48), "cell": cell, "material": rng.choice(["film", "regions"]),
                "init": "random", "pbc": rng.choice([0, 0, 1]), "dmi": 0.0}
    if kind == "rk4":
        return {"kind": "rk4", "nx": _size(rng, 16, 256), "ny": _size(rng, 16, 256), "nz": rng.randint(1, 8),
                "cell": cell, "material": "film", "init": "random", "pbc": 0, "dmi": 0.0, "dt": 5e-14,
                "steps": rng.randint(1, 5)}
    if kind == "ensemble":
        return {"kind": "ensemble", "members": _size(rng, 8, 96), "attempts": 2, "dt": 2e-15}
    if kind == "thermal":
        return {"kind": "thermal", "nx": _size(rng, 32, 512), "ny": _size(rng, 32, 512), "nz": 1, "cell": 10.0,
                "coupled": rng.random() < 0.5, "steps": rng.randint(10, 60), "dt": 5e-14}
    if kind == "surrogate":
        return {"kind": "surrogate", "nx": _size(rng, 32, 512), "ny": _size(rng, 32, 512)}
    if kind == "train":
        return {"kind": "train", "nx": _size(rng, 32, 256), "ny": _size(rng, 32, 256), "batch": rng.randint(1, 16)}
    return {"kind": "setup", "nx": _size(rng, 32, 256), "ny": _size(rng, 32, 256), "nz": _size(rng, 1, 16),
            "cell": cell, "pbc": 0}


# ---- inputs ---------------------------------------------------------------------------------------------------------


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _unit(v):
    return v / v.norm(dim=0, keepdim=True)


def _tables():
    return {"msat": np.zeros(NREG), "aex": np.zeros(NREG), "alpha": np.zeros(NREG), "ku1": np.zeros(NREG),
            "ku2": np.zeros(NREG), "anis_u": np.tile([1.0, 0.0, 0.0], (NREG, 1)), "bext": np.zeros((NREG, 3)),
            "exch_scale": np.ones(NREG * (NREG + 1) // 2), "gamma_ll": GAMMA}


def _grain_map(shape, size, g):
    """Voronoi grains about `size` cells wide: one seed in every block of the lattice, 256 colours."""
    dims = [(n + size - 1) // size + 2 for n in shape]
    pos = torch.rand((*dims, 3), generator=g, device="cuda")
    colour = torch.randint(0, NREG, dims, generator=g, device="cuda")
    at = torch.meshgrid(*(torch.arange(n, device="cuda") for n in shape), indexing="ij")
    best = torch.full(shape, math.inf, device="cuda")
    region = torch.zeros(shape, dtype=torch.uint8, device="cuda")
    for dz in (0, 1, 2):
        for dy in (0, 1, 2):
            for dx in (0, 1, 2):
                b = [at[i] // size + d for i, d in enumerate((dz, dy, dx))]
                p = pos[b[0], b[1], b[2]]
                d2 = sum((((b[i] - 1) + p[..., i]) * size - (at[i] + 0.5)) ** 2 for i in range(3))
                near = d2 < best
                best = torch.where(near, d2, best)
                region = torch.where(near, colour[b[0], b[1], b[2]].to(torch.uint8), region)
    return region


def _problem(case, seed):
    """Region map (uint8 [nz, ny, nx]), region tables and m (float32 [3, nz, ny, nx]), all on the GPU but the tables."""
    g = _gen(seed)
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    rng = np.random.default_rng(seed)
    p = _tables()
    kind = case.get("material", "film")
    if kind == "film":  # permalloy
        region = torch.zeros((nz, ny, nx), dtype=torch.uint8, device="cuda")
        p["msat"][0], p["aex"][0], p["alpha"][0], p["bext"][0] = 8e5, 1.3e-11, 0.01, (0.01, 0.0, 0.0)
    elif kind == "regions":  # patches of six materials, the last one vacuum
        n = 6
        region = _grain_map((nz, ny, nx), 12, g) % n
        p["msat"][:n] = rng.uniform(4e5, 1.2e6, n)
        p["msat"][n - 1] = 0.0
        p["aex"][:n] = rng.uniform(5e-12, 2e-11, n)
        p["alpha"][:n] = rng.uniform(0.01, 0.5, n)
        p["ku1"][:n] = rng.uniform(-5e5, 5e5, n)
        p["ku2"][:n] = rng.uniform(-2e5, 2e5, n)
        u = rng.standard_normal((n, 3))
        p["anis_u"][:n] = u / np.linalg.norm(u, axis=1, keepdims=True)
        p["bext"][:n] = rng.uniform(-0.1, 0.1, (n, 3))
        p["exch_scale"][:] = rng.uniform(0.5, 1.0, p["exch_scale"].shape)
        p["kc"] = np.zeros((NREG, 3))
        p["kc"][:n] = rng.uniform(-5e4, 5e4, (n, 3))
        p["anis_c1"] = np.tile([1.0, 0.0, 0.0], (NREG, 1))
        p["anis_c2"] = np.tile([0.0, 1.0, 0.0], (NREG, 1))
    else:  # grains of (20 nm)^3 and 256 materials
        region = _grain_map((nz, ny, nx), max(2, round(20 / case["cell"])), g)
        p["msat"][:] = rng.uniform(6e5, 1e6, NREG)
        p["aex"][:] = 1.5e-11
        p["alpha"][:] = 0.01
        p["ku1"][:] = rng.uniform(0.0, 5e5, NREG)
        u = rng.standard_normal((NREG, 3))
        p["anis_u"][:] = u / np.linalg.norm(u, axis=1, keepdims=True)
        p["exch_scale"][:] = 0.9
    if case.get("dmi", 0.0):
        p["dind"] = np.full(NREG, case["dmi"])
    m = torch.randn((3, nz, ny, nx), generator=g, device="cuda", dtype=torch.float64)
    if case.get("init", "random") == "vortex":
        x = (torch.arange(nx, device="cuda", dtype=torch.float64) - (nx - 1) / 2) * case["cell"]
        y = (torch.arange(ny, device="cuda", dtype=torch.float64) - (ny - 1) / 2) * case["cell"]
        r = torch.hypot(x[None, :], y[:, None])
        phi = torch.atan2(y[:, None], x[None, :])
        mz = torch.exp(-(r / 10.0) ** 2)
        s = torch.sqrt(1 - mz * mz)
        m = torch.stack([-torch.sin(phi) * s, torch.cos(phi) * s, mz])[:, None] + 0.01 * m
    return region.contiguous(), p, _unit(m).float().contiguous()


def _grid(case):
    c = case["cell"] * 1e-9
    return (case["nx"], case["ny"], case["nz"]), (c, c, c)


def _pbc(case):
    """One image per side along x (bit 0) and y (bit 1)."""
    return (case["pbc"] & 1, (case["pbc"] >> 1) & 1, 0)


def _members(case, seed):
    """Independent grids; their sizes follow from the number of members, materials and states from the seed."""
    sizes, rng = np.random.default_rng(case["members"]), np.random.default_rng(seed)
    g = _gen(seed)
    out = []
    for _ in range(case["members"]):
        nx, ny = (int(v) for v in sizes.choice([32, 64, 128, 256], 2))
        nz = int(sizes.choice([1, 2]))
        d = float(rng.uniform(2e-9, 5e-9))
        p = _tables()
        p["msat"][0], p["aex"][0] = rng.uniform(4e5, 1.2e6), rng.uniform(5e-12, 2e-11)
        p["alpha"][0] = rng.uniform(0.005, 0.5)
        m = _unit(torch.randn((3, nz, ny, nx), generator=g, device="cuda", dtype=torch.float64)).float()
        out.append({"grid": (nx, ny, nz), "cell": (d, d, d), "region": np.zeros((nz, ny, nx), np.uint8), "params": p,
                    "m": m})
    return out


def _thermal_problem(case, seed):
    """10 nm cubes with KV/kT = 8; uncoupled (no exchange, no demag), or a film with both."""
    p = _tables()
    p["msat"][0], p["alpha"][0], p["ku1"][0], p["anis_u"][0] = 1e6, 0.1, 1e4, (0.0, 0.0, 1.0)
    if case["coupled"]:
        p["aex"][0] = 1e-11
    n = (3, case["nz"], case["ny"], case["nx"])
    m = 0.1 * torch.randn(n, generator=_gen(seed), device="cuda", dtype=torch.float64)
    m[2] += 1.0
    region = torch.zeros(n[1:], dtype=torch.uint8, device="cuda")
    return region, p, _unit(m).float().contiguous(), 1e4 * (case["cell"] * 1e-9) ** 3 / (8 * KB)


_C, _KX, _KY, _LAYERS = 32, 16, 16, 4


def _weights(seed):
    g = _gen(seed)

    def n(*shape, s):
        return (torch.randn(shape, generator=g, device="cuda") * s).reshape(-1)

    parts = [n(_C, 3, s=3 ** -0.5), n(_C, s=0.1)]
    for _ in range(_LAYERS):
        parts += [n(_KY, _KX, _C, _C, 2, s=1.0 / _C), n(_C, _C, s=_C ** -0.5), n(_C, s=0.1)]
    parts += [n(3, _C, s=_C ** -0.5), n(3, s=0.01)]
    return torch.cat(parts).cpu().numpy()


def _textures(n, nx, ny, seed):
    """Smooth unit-vector textures with a little noise, float32 [n, 3, 1, ny, nx]: random fields cut off at wavelengths
    of about 20 to 100 cells."""
    g = _gen(seed)
    v = torch.randn((n, 3, ny, nx), generator=g, device="cuda")
    kx = torch.fft.rfftfreq(nx, device="cuda")
    ky = torch.fft.fftfreq(ny, device="cuda")
    cut = 0.01 + 0.04 * torch.rand((n, 1, 1, 1), generator=g, device="cuda")
    v = torch.fft.irfft2(torch.fft.rfft2(v) * torch.exp(-(kx[None, :] ** 2 + ky[:, None] ** 2) / cut ** 2), s=(ny, nx))
    v = v / v.norm(dim=1, keepdim=True)
    v = v + 0.05 * torch.randn(v.shape, generator=g, device="cuda")
    return (v / v.norm(dim=1, keepdim=True))[:, :, None].contiguous()


def _batch(case, seed):
    """A training batch: textures, and targets of the size of the reduced field (about -m_z z with smooth x and y)."""
    m = _textures(case["batch"], case["nx"], case["ny"], seed)
    t = _textures(case["batch"], case["nx"], case["ny"], seed + 1000003) * 0.3
    t[:, 2] -= 0.9 * m[:, 2]
    return m, t.contiguous()


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("run", "observe", "field", "rk4"):
        region, p, m0 = _problem(case, seed)
        ctx = mm.Context(*_grid(case), region, p, pbc=_pbc(case))
        return {"case": case, "ctx": ctx, "m0": m0, "m": m0.clone()}
    if kind == "ensemble":
        members = _members(case, seed)
        b = mm.Batch(members)
        m0 = torch.cat([x["m"].reshape(-1) for x in members])
        return {"case": case, "batch": b, "m0": m0, "m": m0.clone()}
    if kind == "thermal":
        region, p, m0, temp = _thermal_problem(case, seed)
        ctx = mm.Context(*_grid(case), region, p, demag=case["coupled"])
        return {"case": case, "ctx": ctx, "m0": m0, "m": m0.clone(), "temp": temp, "seed": seed}
    if kind == "surrogate":
        s = mm.Surrogate(case["nx"], case["ny"], _weights(seed), MU0 * 8e5)
        return {"case": case, "net": s, "m": _textures(1, case["nx"], case["ny"], seed)[0].contiguous()}
    if kind == "train":
        m, t = _batch(case, seed)
        return {"case": case, "net": mm.SurrogateTrainer(case["nx"], case["ny"], case["batch"], _weights(seed)),
                "m": m, "t": t}
    region, p, _ = _problem(case, seed)
    rng = np.random.default_rng(seed)
    grid, cell = _grid(case)
    cell = (cell[0], cell[1] * rng.uniform(0.8, 1.2), cell[2] * rng.uniform(0.5, 1.5))
    return {"case": case, "grid": grid, "cell": cell, "region": region, "params": p}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "run":
        ctx, m = state["ctx"], state["m"]
        m.copy_(state["m0"])
        ctx.reset_solver()
        t, dt, st = ctx.run(m, math.inf, dt=case["dt"], solver=case["solver"], max_attempts=case["attempts"],
                            opts=mm.solver_opts(dt_max=case["dt"]))
        return {"m": m, "t": t, "dt": dt, "steps": st["steps"]}
    if kind == "observe":
        ctx, m = state["ctx"], state["m"]
        tau = ctx.torque(m)
        # scalars of FP32 fields, in the precision of those
        return {"torque": tau, "energy": np.array(list(ctx.energy(m).values()), np.float32),
                "max_torque": np.float32(ctx.max_torque(m))}
    if kind == "field":
        b, bd = state["ctx"].beff(state["m"], want_demag=True)
        return {"beff": b, "bdemag": bd}
    if kind == "rk4":
        ctx, m = state["ctx"], state["m"]
        m.copy_(state["m0"])
        for _ in range(case["steps"]):
            ctx.rk4_step(m, case["dt"])
        return {"m": m}
    if kind == "ensemble":
        b, m = state["batch"], state["m"]
        m.copy_(state["m0"])
        b.start(45, 0.0, case["dt"])
        n, active = b.run(m, case["attempts"])
        return {"m": m, "attempts": n, "active": active}
    if kind == "thermal":
        ctx, m = state["ctx"], state["m"]
        m.copy_(state["m0"])
        ctx.set_temperature(state["temp"], state["seed"])
        t, dt, st = ctx.run(m, math.inf, dt=case["dt"], solver=12, max_attempts=case["steps"])
        return {"m": m, "t": t, "steps": st["steps"]}
    if kind == "surrogate":
        return {"bdemag": state["net"](state["m"])}
    if kind == "train":
        loss, grad = state["net"].grad(state["m"], state["t"])
        return {"loss": np.float32(loss), "grad": grad}
    ctx = mm.Context(state["grid"], state["cell"], state["region"], state["params"])
    k = ctx.kernel_dump()
    ctx.close()
    return {"kernel": k}


# ---- the least a pass has to move and compute -----------------------------------------------------------------------


def _pad(n, periodic=False):
    return 1 if n == 1 else (1 << (n - 1).bit_length() if periodic else 1 << (2 * n - 2).bit_length())


def _eval_flops(nx, ny, nz, pbc=0):
    """FFT convolution (three real components forth and back, the kernel product) and about 120 operations per cell."""
    px, py, pz = _pad(nx, pbc & 1), _pad(ny, pbc & 2), _pad(nz)
    p = px * py * pz
    return 2 * 3 * 2.5 * p * math.log2(max(p, 2)) + 15 * p + 120.0 * nx * ny * nz


def _kernel_bytes(nx, ny, nz, pbc=0):
    px, py, pz = _pad(nx, pbc & 1), _pad(ny, pbc & 2), _pad(nz)
    return 4.0 * (px // 2 + 1) * (py // 2 + 1) * (pz // 2 + 1) * (4 if nz == 1 else 6)


def work(case):
    kind = case["kind"]
    if kind == "ensemble":
        rng_cells = case["members"] * 120.0 * 120.0 * 1.5  # the mean of the drawn sizes
        return {"bytes": rng_cells * 25 + case["members"] * _kernel_bytes(120, 120, 2),
                "flops": case["members"] * (1 + 6 * case["attempts"]) * _eval_flops(120, 120, 2)}
    if kind in ("surrogate", "train"):
        n = case["nx"] * case["ny"] * case.get("batch", 1)
        layer = n * (2.0 * _C * _C + 4.0 * 2 * _C * _KX + 20 * _C) + case.get("batch", 1) * _KY * _KX * 8.0 * _C * _C
        fwd = _LAYERS * layer + n * 2.0 * 6 * _C
        if kind == "surrogate":
            return {"bytes": n * 24.0 + 2.0 * mm.SNO_NWEIGHTS, "flops": fwd}
        return {"bytes": n * 24.0 + 8.0 * mm.SNO_NWEIGHTS, "flops": 3 * fwd}
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    cells = float(nx * ny * nz)
    pbc = case.get("pbc", 0)
    kb, ef = _kernel_bytes(nx, ny, nz, pbc), _eval_flops(nx, ny, nz, pbc)
    if kind == "run":
        evals = 1 + (6 if case["solver"] == 45 else 3) * case["attempts"]
        return {"bytes": cells * 25 + kb, "flops": evals * ef}
    if kind == "observe":
        return {"bytes": cells * (3 * 13 + 12) + kb, "flops": 3 * ef}
    if kind == "field":
        return {"bytes": cells * 37 + kb, "flops": ef}
    if kind == "rk4":
        return {"bytes": cells * 25 + kb, "flops": 4 * case["steps"] * ef}
    if kind == "thermal":
        return {"bytes": cells * 25 + (kb if case["coupled"] else 0),
                "flops": case["steps"] * (2 * ef if case["coupled"] else 300.0 * cells)}
    p = _pad(nx) * _pad(ny) * _pad(nz)
    return {"bytes": 2 * kb + cells,
            "flops": cells * 216 * 30 + (4 if nz == 1 else 6) * 2.5 * (p / 8) * math.log2(max(p, 2))}


# ---- the same in 64 bits --------------------------------------------------------------------------------------------


def _ratio(a, b):
    return torch.where(b != 0, a / torch.where(b != 0, b, torch.ones_like(b)), torch.zeros_like(a))


def _newell_f(x, y, z):
    x2, y2, z2 = x * x, y * y, z * z
    r = torch.sqrt(x2 + y2 + z2)
    return ((2 * x2 - y2 - z2) * r / 6 + 0.5 * y * (z2 - x2) * torch.asinh(_ratio(y, torch.sqrt(x2 + z2)))
            + 0.5 * z * (y2 - x2) * torch.asinh(_ratio(z, torch.sqrt(x2 + y2)))
            - x * y * z * torch.atan(_ratio(y * z, x * r)))


def _newell_g(x, y, z):
    x2, y2, z2 = x * x, y * y, z * z
    r = torch.sqrt(x2 + y2 + z2)
    return (x * y * z * torch.asinh(_ratio(z, torch.sqrt(x2 + y2)))
            + y / 6 * (3 * z2 - y2) * torch.asinh(_ratio(x, torch.sqrt(y2 + z2)))
            + x / 6 * (3 * z2 - x2) * torch.asinh(_ratio(y, torch.sqrt(x2 + z2)))
            - z2 * z / 6 * torch.atan(_ratio(x * y, z * r)) - z * y2 / 2 * torch.atan(_ratio(x * z, y * r))
            - z * x2 / 2 * torch.atan(_ratio(y * z, x * r)) - x * y * r / 3)


def _tensor_octant(w, cell):
    """Demagnetising tensor [6][wz][wy][wx] of the displacements 0 <= d < w (order xx, yy, zz, xy, xz, yz)."""
    dx, dy, dz = cell
    f64 = {"device": "cuda", "dtype": torch.float64}
    k, j, i = torch.meshgrid(torch.arange(w[2], **f64) * dz, torch.arange(w[1], **f64) * dy,
                             torch.arange(w[0], **f64) * dx, indexing="ij")
    X, Y, Z = i.reshape(-1), j.reshape(-1), k.reshape(-1)
    out = torch.zeros((6, X.numel()), **f64)
    rho = torch.sqrt(X * X + Y * Y + Z * Z) / math.sqrt(dx * dx + dy * dy + dz * dz)
    near = torch.nonzero(rho < 2.5).reshape(-1)
    off = torch.tensor([(p, q, r) for p in (-1, 0, 1) for q in (-1, 0, 1) for r in (-1, 0, 1)], **f64)
    wgt = torch.where(off == 0, 2.0, -1.0).prod(dim=1)[:, None]

    def newell(f, a, b, c, da, db, dc):
        v = f(a[near][None] + off[:, :1] * da, b[near][None] + off[:, 1:2] * db, c[near][None] + off[:, 2:] * dc)
        return (wgt * v).sum(dim=0) / (4 * math.pi * da * db * dc)

    out[0, near] = newell(_newell_f, X, Y, Z, dx, dy, dz)
    out[1, near] = newell(_newell_f, Y, X, Z, dy, dx, dz)
    out[2, near] = newell(_newell_f, Z, Y, X, dz, dy, dx)
    out[3, near] = newell(_newell_g, X, Y, Z, dx, dy, dz)
    out[4, near] = newell(_newell_g, X, Z, Y, dx, dz, dy)
    out[5, near] = newell(_newell_g, Y, Z, X, dy, dz, dx)
    for lo, hi, n in ((2.5, 4, 9), (4, 7, 7), (7, 14, 5), (14, 60, 4), (60, math.inf, 3)):
        sel = torch.nonzero((rho >= lo) & (rho < hi)).reshape(-1)
        if sel.numel() == 0:
            continue
        xi, wi = np.polynomial.legendre.leggauss(n)
        s = np.concatenate([-(1 + xi[::-1]) / 2, (1 + xi) / 2])  # triangular density on [-1, 1]
        ws = np.concatenate([(wi * (1 - xi) / 4)[::-1], wi * (1 - xi) / 4])
        s, ws = torch.tensor(s, **f64), torch.tensor(ws, **f64)
        q = torch.cartesian_prod(s, s, s)
        qw = torch.cartesian_prod(ws, ws, ws).prod(dim=1)
        chunk = max(1, (1 << 24) // q.shape[0])
        for c in sel.split(chunk):
            ux, uy, uz = X[c][None] + q[:, :1] * dx, Y[c][None] + q[:, 1:2] * dy, Z[c][None] + q[:, 2:] * dz
            r2 = ux * ux + uy * uy + uz * uz
            g = qw[:, None] * r2 ** -2.5
            pre = -dx * dy * dz / (4 * math.pi)
            for e, v in enumerate((3 * ux * ux - r2, 3 * uy * uy - r2, 3 * uz * uz - r2, 3 * ux * uy, 3 * ux * uz,
                                   3 * uy * uz)):
                out[e, c] = pre * (g * v).sum(dim=0)
    return out.reshape(6, w[2], w[1], w[0])


_ODD = ((), (), (), (0, 1), (0, 2), (1, 2))  # axes (x, y, z) in which a component is odd


def _kernel(grid, cell, pbc, length):
    """rfftn of the six components on the lengths `length` (x, y, z); displacements of periodic axes fold."""
    w = [n * p if p else n for n, p in zip(grid, pbc)]
    octant = _tensor_octant(w, cell)
    out = []
    for c in range(6):
        v = octant[c]
        for ax in range(3):
            dim = 2 - ax
            if w[ax] > 1:
                neg = torch.flip(v.narrow(dim, 1, w[ax] - 1), (dim,))
                v = torch.cat([-neg if ax in _ODD[c] else neg, v], dim=dim)
            pos = torch.arange(1 - w[ax], w[ax], device="cuda") % length[ax]
            shape = list(v.shape)
            shape[dim] = length[ax]
            v = torch.zeros(shape, device="cuda", dtype=torch.float64).index_add_(dim, pos, v)
        out.append(torch.fft.rfftn(v).real)
    return out


class _Reference:
    """B_eff, torque and energies of one grid in 64 bits."""

    def __init__(self, grid, cell, pbc, region, p, demag=True):
        self.grid, self.cell, self.pbc = grid, cell, pbc
        self.r = region.long()
        t = {k: torch.tensor(np.asarray(v), device="cuda", dtype=torch.float64) for k, v in p.items()}
        ms = t["msat"]
        lam = torch.where(ms > 0, t["aex"] / torch.where(ms > 0, ms, torch.ones_like(ms)), torch.zeros_like(ms))
        i = torch.arange(NREG, device="cuda")
        hi, lo = torch.maximum(i[:, None], i[None]), torch.minimum(i[:, None], i[None])
        s = t["exch_scale"][hi * (hi + 1) // 2 + lo]
        s = torch.where(hi == lo, torch.ones_like(s), s)
        self.pair = 2 * s * _ratio(2 * lam[:, None] * lam[None], lam[:, None] + lam[None])
        self.pair = self.pair * ((ms[:, None] > 0) & (ms[None] > 0))
        self.ms = ms[self.r]
        self.mag = self.ms > 0
        inv = _ratio(torch.ones_like(self.ms), self.ms)
        self.alpha = t["alpha"][self.r]
        self.k1, self.k2 = 2 * t["ku1"][self.r] * inv, 4 * t["ku2"][self.r] * inv
        self.u = t["anis_u"][self.r].movedim(-1, 0)
        self.bext = t["bext"][self.r].movedim(-1, 0)
        self.kc = None
        if "kc" in t:
            kc = t["kc"][self.r]
            c1, c2 = (_unit(t[n].T).T for n in ("anis_c1", "anis_c2"))
            self.kc = (-2 * kc[..., 0] * inv, -2 * kc[..., 1] * inv, -4 * kc[..., 2] * inv)
            self.axes = [a[self.r].movedim(-1, 0) for a in (c1, c2, torch.linalg.cross(c1, c2))]
        self.dmi = None
        if "dind" in t:
            d, a = t["dind"][self.r], t["aex"][self.r]
            self.dmi = (2 * d * inv, _ratio(d, 2 * a))
        self.k = None
        if demag:
            self.length = [1 if n == 1 else (n if q else 2 * n) for n, q in zip(grid, pbc)]
            self.k = _kernel(grid, cell, pbc, self.length)

    def demag(self, m):
        if self.k is None:
            return torch.zeros_like(m)
        s = tuple(self.length[::-1])
        a = [torch.fft.rfftn(self.ms * m[c], s=s) for c in range(3)]
        k = self.k
        rows = ((0, 3, 4), (3, 1, 5), (4, 5, 2))
        nx, ny, nz = self.grid
        return torch.stack([torch.fft.irfftn(-MU0 * sum(k[j] * a[c] for c, j in enumerate(row)), s=s)[:nz, :ny, :nx]
                            for row in rows])

    def _side(self, v, ax, d):
        """The neighbour's value along x, y or z, and whether it lies in the grid (wrapped on periodic axes)."""
        dim = v.dim() - 1 - ax
        n = torch.roll(v, -d, dims=dim)
        inside = torch.ones(self.r.shape, dtype=torch.bool, device="cuda")
        if not self.pbc[ax]:
            edge = [slice(None)] * 3
            edge[2 - ax] = -1 if d > 0 else 0
            inside[tuple(edge)] = False
        return n, inside

    def exchange(self, m):
        b = torch.zeros_like(m)
        around = {}
        for ax in range(3):
            for d in (-1, 1):
                n, inside = self._side(m, ax, d)
                rn, _ = self._side(self.r, ax, d)
                b += torch.where(inside, self.pair[self.r, rn], 0.0) / self.cell[ax] ** 2 * (n - m)
                around[ax, d] = (n, inside & (self.ms > 0) & self._side(self.ms, ax, d)[0].gt(0))
        if self.dmi is not None:
            pre, xi = self.dmi
            zero = torch.zeros_like(xi)
            slope = (torch.stack([-xi * m[2], zero, xi * m[0]]), torch.stack([zero, -xi * m[2], xi * m[1]]))
            diff = []
            for ax in (0, 1):
                v = {}
                for d in (-1, 1):
                    n, real = around[ax, d]
                    ghost = m + d * self.cell[ax] * slope[ax]
                    v[d] = torch.where(real, n, ghost)
                    b += torch.where(real, 0.0, self.pair[self.r, self.r]) / self.cell[ax] ** 2 * (ghost - m)
                diff.append((v[1] - v[-1]) / (2 * self.cell[ax]))
            b += pre * torch.stack([diff[0][2], diff[1][2], -diff[0][0] - diff[1][1]])
        return b

    def anisotropy(self, m):
        """The field, and the sum of m.B weighted as the energy takes it (1/2, 1/4; 1/4, 1/6, 1/8 for the cubic terms)."""
        um = (self.u * m).sum(dim=0)
        b = (self.k1 * um + self.k2 * um ** 3) * self.u
        e = 0.5 * self.k1 * um ** 2 + 0.25 * self.k2 * um ** 4
        if self.kc is not None:
            a = [(c * m).sum(dim=0) for c in self.axes]
            for i in range(3):
                j, k = (i + 1) % 3, (i + 2) % 3
                f = (self.kc[0] * a[i] * (a[j] ** 2 + a[k] ** 2), self.kc[1] * a[i] * a[j] ** 2 * a[k] ** 2,
                     self.kc[2] * a[i] ** 3 * (a[j] ** 4 + a[k] ** 4))
                b = b + sum(f) * self.axes[i]
                e = e + a[i] * (f[0] / 4 + f[1] / 6 + f[2] / 8)
        return b, e

    def beff(self, m, extra=None):
        b = self.demag(m) + self.exchange(m) + self.anisotropy(m)[0] + self.bext
        return torch.where(self.mag, b if extra is None else b + extra, 0.0)

    def torque(self, m, extra=None):
        b = self.beff(m, extra)
        mxb = torch.linalg.cross(m, b, dim=0)
        return -GAMMA / (1 + self.alpha ** 2) * (mxb + self.alpha * torch.linalg.cross(m, mxb, dim=0))

    def energy(self, m):
        v = self.cell[0] * self.cell[1] * self.cell[2]
        e = [(-0.5 * self.ms * (m * self.demag(m)).sum(dim=0)).sum().item() * v,
             (-0.5 * self.ms * (m * self.exchange(m)).sum(dim=0)).sum().item() * v,
             (-self.ms * self.anisotropy(m)[1]).sum().item() * v, (-self.ms * (m * self.bext).sum(dim=0)).sum().item() * v]
        return e + [sum(e)]


_PAIRS = {
    45: (4, [[], [1 / 5], [3 / 40, 9 / 40], [44 / 45, -56 / 15, 32 / 9],
             [19372 / 6561, -25360 / 2187, 64448 / 6561, -212 / 729],
             [9017 / 3168, -355 / 33, 46732 / 5247, 49 / 176, -5103 / 18656],
             [35 / 384, 0, 500 / 1113, 125 / 192, -2187 / 6784, 11 / 84]],
         [35 / 384 - 5179 / 57600, 0, 500 / 1113 - 7571 / 16695, 125 / 192 - 393 / 640, -2187 / 6784 + 92097 / 339200,
          11 / 84 - 187 / 2100, -1 / 40]),
    23: (2, [[], [1 / 2], [0, 3 / 4], [2 / 9, 1 / 3, 4 / 9]], [2 / 9 - 7 / 24, 1 / 3 - 1 / 4, 4 / 9 - 1 / 3, -1 / 8]),
}


def _embedded(ref, m, solver, dt, attempts, dt_max=math.inf, max_err=1e-5):
    order, a, e = _PAIRS[solver]
    t, steps, k1 = 0.0, 0, ref.torque(m)
    for _ in range(attempts):
        k = [k1]
        for row in a[1:]:
            ms = m + dt * sum(c * q for c, q in zip(row, k))
            k.append(ref.torque(ms))
        err = dt * sum(c * q for c, q in zip(e, k)).norm(dim=0).max().item()
        grow = 2.0 if err == 0 else min(2.0, max(0.1, 0.8 * (max_err / err) ** (1 / (order + 1))))
        if err <= max_err:
            t, steps, k1 = t + dt, steps + 1, k[-1]
            n = ms.norm(dim=0, keepdim=True)
            m = torch.where(n > 0, ms / n, 0.0)
        dt = min(dt * grow, dt_max)
    return m, t, dt, steps


def _philox(cells, step, seed):
    """Philox4x32-10 at counter (cell, step, 0, 0) and key (seed, 0), 32-bit words in int64."""
    mask = 0xFFFFFFFF
    c = [cells, torch.full_like(cells, step), torch.zeros_like(cells), torch.zeros_like(cells)]
    k = [seed & mask, (seed >> 32) & mask]
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57  # the low 64 bits, whatever the sign
        c = [((p1 >> 32) & mask) ^ c[1] ^ k[0], p1 & mask, ((p0 >> 32) & mask) ^ c[3] ^ k[1], p0 & mask]
        k = [(k[0] + 0x9E3779B9) & mask, (k[1] + 0xBB67AE85) & mask]
    return c


def _thermal(case, seed):
    region, p, m, temp = _thermal_problem(case, seed)
    grid, cell = _grid(case)
    ref = _Reference(grid, cell, (0, 0, 0), region, p, demag=case["coupled"])
    m, dt = m.double(), case["dt"]
    sigma = math.sqrt(2 * 0.1 * KB * temp / (1e6 * GAMMA * cell[0] * cell[1] * cell[2] * dt))
    cells = torch.arange(region.numel(), device="cuda")
    for s in range(case["steps"]):
        u = [((x >> 8).double() + 0.5) * 2.0 ** -24 for x in _philox(cells, s, seed)]
        r0, r2 = torch.sqrt(-2 * torch.log(u[0])), torch.sqrt(-2 * torch.log(u[2]))
        w = 2 * math.pi
        eta = torch.stack([r0 * torch.cos(w * u[1]), r0 * torch.sin(w * u[1]), r2 * torch.cos(w * u[3])])
        b = sigma * eta.reshape(m.shape)
        k1 = ref.torque(m, b)
        k2 = ref.torque(m + dt * k1, b)
        m = _unit(m + dt / 2 * (k1 + k2))
    return m


def _network(w, m):
    """The spectral neural operator on m [B, 3, ny, nx], w the flat weights, everything in the type of w."""
    ny, nx = m.shape[-2:]
    at = 0

    def take(*shape):
        nonlocal at
        n = math.prod(shape)
        at += n
        return w[at - n:at].reshape(shape)

    def phase(k, n):
        return -2 * math.pi / n * (torch.outer(k, torch.arange(n, device="cuda")) % n).to(w.dtype)

    ax = phase(torch.arange(_KX, device="cuda"), nx)
    ay = phase(torch.arange(_KY, device="cuda") - _KY // 2, ny)
    fx, fy = torch.polar(torch.ones_like(ax), ax), torch.polar(torch.ones_like(ay), ay)
    wk = torch.full((_KX, 1), 2.0, device="cuda", dtype=w.dtype)
    wk[0] = 1.0
    big_p, small_p = take(_C, 3), take(_C, 1, 1)
    h = torch.tensordot(big_p, m, dims=([1], [1])).movedim(0, 1) + small_p
    for _ in range(_LAYERS):
        r, lw, lb = torch.view_as_complex(take(_KY, _KX, _C, _C, 2)), take(_C, _C), take(_C, 1, 1)
        hh = torch.matmul(fy, torch.matmul(h.to(fx.dtype), fx.T))  # [B, C, ky, kx]
        gh = torch.matmul(r, hh.permute(2, 3, 1, 0).contiguous()).permute(3, 2, 0, 1)
        g = torch.matmul(torch.matmul(fy.conj().T, gh), wk * fx.conj()).real / (nx * ny)
        z = g + torch.tensordot(lw, h, dims=([1], [1])).movedim(0, 1) + lb
        h = 0.5 * z * (1 + torch.erf(z / math.sqrt(2)))
    big_q, small_q = take(3, _C), take(3, 1, 1)
    return torch.tensordot(big_q, h, dims=([1], [1])).movedim(0, 1) + small_q


def exact(case, seed):
    kind = case["kind"]
    if kind in ("run", "observe", "field", "rk4"):
        region, p, m = _problem(case, seed)
        ref = _Reference(*_grid(case), _pbc(case), region, p)
        m = m.double()
        if kind == "run":
            m, t, dt, steps = _embedded(ref, m, case["solver"], case["dt"], case["attempts"], case["dt"])
            return {"m": m, "t": t, "dt": dt, "steps": steps}
        if kind == "observe":
            tau = ref.torque(m)
            return {"torque": tau, "energy": np.array(ref.energy(m)),
                    "max_torque": np.float64(tau.norm(dim=0).max().item())}
        if kind == "field":
            return {"beff": ref.beff(m), "bdemag": ref.demag(m)}
        h = case["dt"]
        for _ in range(case["steps"]):
            k1 = ref.torque(m)
            k2 = ref.torque(m + h / 2 * k1)
            k3 = ref.torque(m + h / 2 * k2)
            k4 = ref.torque(m + h * k3)
            m = _unit(m + h / 6 * (k1 + 2 * k2 + 2 * k3 + k4))
        return {"m": m}
    if kind == "ensemble":
        out = []
        for x in _members(case, seed):
            region = torch.as_tensor(x["region"], device="cuda")
            ref = _Reference(x["grid"], x["cell"], (0, 0, 0), region, x["params"])
            out.append(_embedded(ref, x["m"].double(), 45, case["dt"], case["attempts"])[0].reshape(-1))
        return {"m": torch.cat(out), "attempts": case["attempts"], "active": case["members"]}
    if kind == "thermal":
        t = 0.0
        for _ in range(case["steps"]):
            t += case["dt"]
        return {"m": _thermal(case, seed), "t": t, "steps": case["steps"]}
    if kind == "surrogate":
        w = torch.tensor(_weights(seed), device="cuda").bfloat16().double()
        m = _textures(1, case["nx"], case["ny"], seed)[:, :, 0].double()
        return {"bdemag": MU0 * 8e5 * _network(w, m)[0][:, None]}
    if kind == "train":
        m, t = (v[:, :, 0].double() for v in _batch(case, seed))
        w = torch.tensor(_weights(seed), device="cuda").double().requires_grad_()
        y = _network(w, m)
        loss = ((y - t).flatten(1).norm(dim=1) / t.flatten(1).norm(dim=1)).mean()
        return {"loss": np.float64(loss.item()), "grad": torch.autograd.grad(loss, w)[0]}
    s = prepare(case, seed)
    length = [_pad(n) for n in s["grid"]]
    k = _kernel(s["grid"], s["cell"], (0, 0, 0), length)
    kyh, kzh = length[1] // 2 + 1, length[2] // 2 + 1
    comps = [k[c][:kzh, :kyh].permute(2, 1, 0) for c in ((0, 1, 2, 3) if length[2] == 1 else range(6))]
    return {"kernel": (-MU0 / math.prod(length) * torch.stack(comps, dim=-1)).reshape(-1)}
