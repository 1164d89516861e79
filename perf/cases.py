"""What a user of this framework runs, as cases that can be timed and compared.

Each case is one pass through the public entry points of
``paper_1909_08354_amd.gsn``: a simulation from a state on the device (load,
step, read back, observables where a program would log them), a parameter
sweep through the batched solver, a run of corrected coarse steps, or the
forward and backward passes of corrector training.  Grids, boxes, kernels and
initial states are those of ``paper_1909_08354_amd/inputs.py`` or generic ones
of the same family; every state is drawn from the seed.

A case is a dict of plain values:

  kind     "grid", "sweep", "corrected" or "train"
  nz ny nx the grid (nz = 0: a 2-D grid)
  steps    split steps (coarse steps for "corrected") of one pass
  tuned    the schedule is autotuned on the first state, as programs that run
           long do; otherwise the grid is used as created
  storage  "c64" or "c128"
  model    "kerr" (Newton + Yukawa + Kerr term), "eq15" (the fluid of Eq. (15):
           pressure and Bohm terms) or "nmc" (that fluid under the
           position-dependent coupling of Eq. (9)-(12))
  observe  mass and energy are read after the steps
"""
import math

import numpy as np
import torch

from paper_1909_08354_amd import gsn

NET = ((3, 32), (32, 32), (32, 32), (32, 2))   # channels of the corrector's layers
RATIO = 8                                      # fine steps per coarse step


def _grid(name, nz, ny, nx, steps, tuned=True, storage="c64", model="kerr", g=0.0, box=0.0, dz=1e-3,
          observe=False):
    return dict(name=name, kind="grid", nz=nz, ny=ny, nx=nx, steps=steps, tuned=tuned, storage=storage,
                model=model, g=g, box=box, dz=dz, observe=observe)


def listed():
    return [
        # one step of a small 2-D grid with its observables: the interactive
        # call of a notebook or a parameter scan, launches and waits only
        _grid("one_step_64x128", 0, 64, 128, 1, tuned=False, g=-0.5, dz=2e-3, observe=True),
        # the paper's 2-D optics setting: a Kerr + Newton beam on [-20, 20)^2
        _grid("beam_128", 0, 128, 128, 200, g=-0.5, box=40.0),
        # a 2-D lump state at the corrector's mesh, its fine steps
        _grid("lumps_512sq", 0, 512, 512, 80, g=-0.5, dz=5e-3),
        # a large, unequal 2-D mesh
        _grid("sheet_1024x2048", 0, 1024, 2048, 20, g=-0.5),
        # a thin 3-D box of unequal extents on the schedule a grid starts with
        _grid("slab_32x256x64", 32, 256, 64, 20, tuned=False, dz=5e-4),
        # the 256^3 cloud with its logged mass and energy
        _grid("cloud_256", 256, 256, 256, 20, dz=5e-4, observe=True),
        # the largest single-GPU workload: moving lumps on 512^3
        _grid("lumps_512", 512, 512, 512, 8, dz=2.5e-4),
        # the paper's double-precision regime
        _grid("cloud_256_c128", 256, 256, 256, 8, storage="c128", dz=5e-4),
        # the full fluid model: pressure, Bohm potential, coupling fields
        _grid("fluid_nmc_256", 256, 256, 256, 6, model="nmc", dz=5e-4),
        # a sweep over the gravity model: 64 instances of uneven sizes
        dict(name="sweep_64", kind="sweep", count=64, small=256, large=1024, steps=200, tuned=True),
        # the learned corrector in use: coarse steps, each corrected
        dict(name="corrected_512", kind="corrected", ny=512, nx=512, steps=10, tuned=True),
        # one training batch of the corrector: features, forward, backward
        dict(name="train_512_b8", kind="train", ny=512, nx=512, batch=8),
    ]


def _pow2(rng, lo, hi):
    return 1 << rng.randint(lo, hi)


def draw(rng):
    """One more case of the same ranges."""
    r = rng.random()
    if r < 0.12:
        small = rng.choice((128, 256, 512))
        return dict(kind="sweep", count=rng.randint(3, 32), small=small, large=rng.choice((small, 2 * small, 1024)),
                    steps=rng.randint(20, 200), tuned=rng.random() < 0.7)
    if r < 0.2:
        return dict(kind="corrected", ny=_pow2(rng, 7, 10), nx=_pow2(rng, 7, 10), steps=rng.randint(2, 20), tuned=True)
    if r < 0.26:
        return dict(kind="train", ny=_pow2(rng, 6, 9), nx=_pow2(rng, 6, 9), batch=rng.randint(1, 7))
    model = "kerr" if r < 0.72 else ("eq15" if r < 0.8 else "nmc" if r < 0.88 else "kerr")
    storage = "c128" if r >= 0.88 else "c64"
    three = rng.random() < 0.6
    while True:   # points spread over their logarithm, 2^12 .. 2^27 (2^24 with more bytes per point)
        bits = rng.uniform(12, 24.4 if storage == "c128" or model != "kerr" else 27.4)
        if three:
            n = (_pow2(rng, 3, 10), _pow2(rng, 3, 10), _pow2(rng, 4, 10))
        else:
            n = (0, _pow2(rng, 5, 11), _pow2(rng, 5, 11))
        p = max(n[0], 1) * n[1] * n[2]
        least = 8 if model == "kerr" else 32      # the fluid's cloud needs some room
        if abs(math.log2(p) - bits) < 0.6 and p <= 1 << (24 if storage == "c128" or model != "kerr" else 27) \
                and min(n[0] or n[1], n[1], n[2]) >= least:
            break
        three = rng.random() < 0.6
    steps = rng.randint(1, max(1, min(100, int(3 * (1 << 27) / p))))
    return dict(kind="grid", nz=n[0], ny=n[1], nx=n[2], steps=steps, tuned=rng.random() < 0.7, storage=storage,
                model=model, g=0.0 if three else -0.5, box=0.0, dz=round(rng.uniform(2e-4, 2e-3), 6),
                observe=model != "nmc" and rng.random() < 0.25)


# ---------------------------------------------------------------- inputs
def _shape(case):
    return (case["ny"], case["nx"]) if not case.get("nz") else (case["nz"], case["ny"], case["nx"])


def _box(case):
    n = _shape(case)
    return tuple(float(case.get("box") or v) for v in n)


def _lumps(n, L, rng, device, dtype):
    """1-4 (3-D: 2-8) Gaussian lumps with phase-gradient velocities, built
    from their separable factors, as inputs.random_lumps draws them."""
    count = int(rng.integers(1, 5)) if len(n) == 2 else int(rng.integers(2, 9))
    least = min(L)
    psi = torch.zeros(n, dtype=dtype, device=device)
    for _ in range(count):
        c = rng.uniform(0.0, 1.0, size=len(n)) * np.array(L)
        w = rng.uniform(2.0, 6.0) if len(n) == 2 else rng.uniform(4.0, 10.0)
        w = min(w, least / 5.0)
        v = rng.uniform(-0.5, 0.5, size=len(n))
        f = []
        for ax in range(len(n)):
            x = -0.5 * L[ax] + np.arange(n[ax]) * (L[ax] / n[ax])
            d = (x - c[ax] + 0.5 * L[ax]) % L[ax] - 0.5 * L[ax]
            f.append(torch.from_numpy(np.exp(-(d * d) / (w * w)) * np.exp(1j * v[ax] * d)).to(device))
        yx = torch.outer(f[-2], f[-1])
        if len(n) == 2:
            psi += yx.to(dtype)
        else:
            psi += f[0].to(dtype)[:, None, None] * yx.to(dtype)
    return psi


def _fluid(n, L, rng, device, dtype):
    """sqrt of a Gaussian number density of mass 25 with 1e-3 phase noise."""
    w = min(6.0, min(L) / 10.0) * rng.uniform(0.9, 1.1)
    rho0 = 25.0 / (math.pi * w * w) ** (len(n) / 2)
    psi = torch.full(n, math.sqrt(rho0), dtype=torch.float64, device=device)
    for ax in range(len(n)):
        x = -0.5 * L[ax] + np.arange(n[ax]) * (L[ax] / n[ax])
        f = torch.from_numpy(np.exp(-x * x / (2 * w * w))).to(device)
        psi *= f.reshape([-1 if d == ax else 1 for d in range(len(n))])
    gen = torch.Generator(device=device)
    gen.manual_seed(int(rng.integers(1 << 31)))
    xi = torch.rand(n, dtype=torch.float64, device=device, generator=gen) * 2 - 1
    return torch.polar(psi, 1e-3 * xi).to(dtype)


def _state(case, seed, device="cuda"):
    """The initial state a case's program has on the device."""
    rng = np.random.default_rng(seed)
    dtype = torch.complex128 if case.get("storage") == "c128" else torch.complex64
    make = _lumps if case.get("model", "kerr") == "kerr" else _fluid
    return make(_shape(case), _box(case), rng, device, dtype)


def _kernel(case):
    """(c_N, c_Y, m_Y, c_0) of the case's model."""
    if case.get("model") == "eq15":
        return (0.5, 0.0, 0.0, 0.0)
    if case.get("model") == "nmc" or case.get("box"):
        return (1.0, 0.0, 0.0, 0.0)
    return (1.0, 0.3, 0.1, 0.0)


LOCAL = (-1.02, 1.0, -1.0, 1e-10)       # c_pressure, n, c_bohm, floor of the fluid
R0 = 25.0 / (4 * math.pi)


def _instances(case, seed, device="cuda"):
    """The sweep's instances: size, Yukawa coupling and mass, lump state."""
    sizes = []
    s = case["small"]
    while s <= case["large"]:
        sizes.append(s)
        s *= 2
    pick = np.random.default_rng(3)     # the same mix of sizes for every seed
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(case["count"]):
        n = int(sizes[pick.integers(0, len(sizes))])
        kern = (1.0, float(rng.uniform(0, 1)), float(rng.uniform(0.05, 0.5)), 0.0)
        out.append(((n, n), kern, _lumps((n, n), (float(n), float(n)), rng, device, torch.complex64)))
    return out


def _weights(seed):
    """Flat corrector parameters: scaled normal weights, small biases."""
    rng = np.random.default_rng(seed + 77)
    parts = []
    for ci, co in NET:
        parts += [rng.standard_normal((9, co, ci)) * math.sqrt(2.0 / (9 * ci)), rng.uniform(-0.05, 0.05, co)]
    return np.concatenate([p.ravel() for p in parts]).astype(np.float32)


SCALES, OUT_SCALE = (1.0, 1.0, 0.1), 1e-4


def _corrected_grid(case):
    return dict(nz=0, ny=case["ny"], nx=case["nx"], g=-0.5, dz=5e-3, box=0.0)


def _batch_tensors(case, seed, device="cuda"):
    """Coarse state, potential and fine state of every image of a batch (the
    residual is a small smooth field of the size the solver's has)."""
    rng = np.random.default_rng(seed)
    n = (case["ny"], case["nx"])
    L = tuple(float(v) for v in n)
    out = []
    for _ in range(case["batch"]):
        psi = _lumps(n, L, rng, device, torch.complex128)
        phi = 4.0 * (psi.real ** 2 + psi.imag ** 2) - 0.5
        fine = psi + 1e-4 * torch.roll(psi, (1, 1), (0, 1))
        out.append((psi.to(torch.complex64), phi.to(torch.float32), fine.to(torch.complex64)))
    return out


# ---------------------------------------------------------------- the program
def prepare(case, seed):
    kind = case["kind"]
    if kind == "grid":
        n, L = _shape(case), _box(case)
        psi = _state(case, seed)
        storage = np.complex128 if case["storage"] == "c128" else np.complex64
        grid = gsn.Grid(n, L, storage=storage)
        grid.set_kernel(*_kernel(case))
        grid.set_coefficients(0.5, case["g"], case["dz"])
        if case["model"] != "kerr":
            grid.set_local_terms(*LOCAL)
        if case["model"] == "nmc":
            grid.set_source_fields(*grid.nmc_fields(1.0, R0, 1.0))
        grid.set_psi(psi)
        if case["tuned"]:
            grid.autotune(5)
        return dict(case=case, grid=grid, psi=psi, dtype=storage)
    if kind == "sweep":
        inst = _instances(case, seed)
        batch = gsn.Batch([n for n, _, _ in inst], [(float(n[0]), float(n[1])) for n, _, _ in inst])
        if case["tuned"]:
            for i, (_, kern, psi) in enumerate(inst):
                batch.set(i, kern, 0.5, -0.5, 1e-3, psi)
            batch.autotune(3)
        return dict(case=case, batch=batch, inst=inst)
    corr = gsn.Corrector(case["ny"], case["nx"], case.get("batch", 1))
    corr.set_weights(_weights(seed))
    corr.set_scales(SCALES, OUT_SCALE)
    if kind == "corrected":
        g = _corrected_grid(case)
        psi = _state(g, seed)
        grid = gsn.Grid(_shape(g), _box(g))
        grid.set_kernel(1.0, 0.0, 0.0, 0.0)
        grid.set_coefficients(0.5, g["g"], g["dz"])
        grid.set_coarse_ratio(RATIO)
        grid.set_psi(psi)
        if case["tuned"]:
            grid.autotune(5)
        return dict(case=case, grid=grid, psi=psi, corr=corr)
    return dict(case=case, corr=corr, images=_batch_tensors(case, seed))


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "grid":
        grid = state["grid"]
        grid.set_psi(state["psi"])
        grid.step(case["steps"])
        out = {"psi": grid.get_psi(state["dtype"], device=True)}
        if case["observe"]:
            out["mass"] = np.float32(grid.mass())
            out["energy"] = np.float32(grid.energy()["total"])
        return out
    if kind == "sweep":
        batch = state["batch"]
        for i, (_, kern, psi) in enumerate(state["inst"]):
            batch.set(i, kern, 0.5, -0.5, 1e-3, psi)
        batch.step(case["steps"])
        return [batch.get(i, np.complex64) for i in range(batch.count)]
    if kind == "corrected":
        grid = state["grid"]
        grid.set_psi(state["psi"])
        grid.step_corrected(state["corr"], case["steps"])
        return {"psi": grid.get_psi(np.complex64, device=True)}
    corr = state["corr"]
    for b, (psi, phi, fine) in enumerate(state["images"]):
        corr.pack(b, psi, phi)
        corr.pack_target(b, fine, psi)
    out = corr.forward(case["batch"])
    loss, grad = corr.gradients(case["batch"])
    return {"out": out, "loss": np.float32(loss), "grad": grad}


def work(case):
    """Bytes and operations no split-step program can do without: the state
    read and written once a step, the transforms of psi (two complex) and of
    the density (two real) at 5 N log2 N, about 40 operations a point beside
    them; a 2 x 9 x cin x cout product per pixel and layer of the network."""
    def step(points, esize):
        return 2 * esize * points, points * (15 * math.log2(points) + 40)

    kind = case["kind"]
    net = 18 * sum(ci * co for ci, co in NET)
    if kind == "grid":
        p = math.prod(_shape(case))
        b, f = step(p, 16 if case["storage"] == "c128" else 8)
        more = {"kerr": (0, 0), "eq15": (0, 5 * math.log2(p) + 60), "nmc": (12, 10 * math.log2(p) + 70)}[case["model"]]
        return {"bytes": case["steps"] * (b + more[0] * p), "flops": case["steps"] * (f + more[1] * p)}
    if kind == "sweep":
        total = [0.0, 0.0]
        for n, _, _ in _sizes_only(case):
            b, f = step(n[0] * n[1], 8)
            total = [total[0] + case["steps"] * b, total[1] + case["steps"] * f]
        return {"bytes": total[0], "flops": total[1]}
    p = case["ny"] * case["nx"]
    if kind == "corrected":
        b, f = step(p, 8)
        return {"bytes": case["steps"] * b, "flops": case["steps"] * (f + net * p)}
    # forward once for the output, once more with the backward pass (twice its work)
    return {"bytes": case["batch"] * p * (8 + 4 + 8 + 8), "flops": 4.0 * net * p * case["batch"]}


def _sizes_only(case):
    sizes = []
    s = case["small"]
    while s <= case["large"]:
        sizes.append(s)
        s *= 2
    pick = np.random.default_rng(3)
    return [((int(sizes[pick.integers(0, len(sizes))]),) * 2, None, None) for _ in range(case["count"])]


# ---------------------------------------------------------------- in 64 bits
def _freq2(n, L, device):
    """|k|^2 on the grid."""
    k2 = torch.zeros(n, dtype=torch.float64, device=device)
    for ax in range(len(n)):
        k = 2 * math.pi * torch.fft.fftfreq(n[ax], d=L[ax] / n[ax], dtype=torch.float64, device=device)
        k2 = k2 + (k * k).reshape([-1 if d == ax else 1 for d in range(len(n))])
    return k2


def _kern_hat(k2, kern):
    cN, cY, mY, c0 = kern
    K = torch.zeros_like(k2)
    if cN:
        K += torch.where(k2 > 0, cN / torch.where(k2 > 0, k2, torch.ones_like(k2)), torch.zeros_like(k2))
    if cY:
        K += cY / (k2 + mY * mY)
    return K + c0


def _fields(n, L, device):
    """gamma, beta and V of the non-minimal coupling (lambda = 1), as float32."""
    r2 = torch.zeros(n, dtype=torch.float64, device=device)
    for ax in range(len(n)):
        x = -0.5 * L[ax] + torch.arange(n[ax], dtype=torch.float64, device=device) * (L[ax] / n[ax])
        r2 = r2 + (x * x).reshape([-1 if d == ax else 1 for d in range(len(n))])
    r = torch.sqrt(r2)
    u = R0 / (r + R0)
    rm = torch.clamp(r, min=0.5 * min(b / m for m, b in zip(n, L)))
    V = -torch.log(1 - R0 / (rm + R0))
    return [f.to(torch.float32).to(torch.float64) for f in ((1 - u) / 2, u / (r + R0), V)]


class _Exact:
    """The split step in complex128 with torch's transforms."""

    def __init__(self, n, L, kern, g, model="kerr"):
        self.n, self.L, self.kern, self.g, self.model = n, L, kern, g, model
        self.dev = "cuda" if torch.cuda.is_available() else "cpu"
        self.k2 = _freq2(n, L, self.dev)
        self.K = _kern_hat(self.k2, kern)
        self.fields = _fields(n, L, self.dev) if model == "nmc" else None

    def phi(self, rho):
        if self.fields is not None:
            gam, bet, _ = self.fields
            lap = torch.fft.ifftn(-self.k2 * torch.fft.fftn(rho)).real
            rho = gam * rho + bet * lap
        return torch.fft.ifftn(self.K * torch.fft.fftn(rho)).real

    def kinetic(self, psi, h):
        return torch.fft.ifftn(torch.fft.fftn(psi) * torch.polar(torch.ones_like(self.k2), -0.5 * h * self.k2))

    def nonlinear(self, psi, dz):
        rho = psi.real ** 2 + psi.imag ** 2
        u = self.g * rho + self.phi(rho)
        if self.model != "kerr":
            cp, _, cb, floor = LOCAL
            s = torch.sqrt(rho)
            lap = torch.fft.ifftn(-self.k2 * torch.fft.fftn(s)).real
            u = u + cp * torch.log(torch.clamp(rho, min=floor)) + cb * lap / (2 * torch.clamp(s, min=math.sqrt(floor)))
        if self.fields is not None:
            u = u + self.fields[2]
        return psi * torch.polar(torch.ones_like(u), u * dz)

    def steps(self, psi, dz, count):
        psi = self.kinetic(psi, 0.5 * dz)
        for i in range(count):
            psi = self.nonlinear(psi, dz)
            psi = self.kinetic(psi, dz if i + 1 < count else 0.5 * dz)
        return psi

    def observables(self, psi):
        dV = math.prod(b / m for m, b in zip(self.n, self.L))
        rho = psi.real ** 2 + psi.imag ** 2
        hat = torch.fft.fftn(psi)
        e = 0.5 * dV / psi.numel() * float((self.k2 * (hat.real ** 2 + hat.imag ** 2)).sum())
        e -= 0.5 * dV * float((rho * (self.g * rho + self.phi(rho))).sum())
        if self.model != "kerr":
            cp, _, cb, floor = LOCAL
            r = torch.clamp(rho, min=floor)
            # the antiderivative of the floored ln rho
            G = torch.where(rho > floor, r * (torch.log(r) - 1.0),
                            floor * (math.log(floor) - 1.0) + (rho - floor) * math.log(floor))
            s = torch.sqrt(rho)
            lap = torch.fft.ifftn(-self.k2 * torch.fft.fftn(s)).real
            e -= cp * dV * float(G.sum()) + 0.5 * cb * dV * float((s * lap).sum())
        return dV * float(rho.sum()), e


def _net(x, theta):
    """The corrector network on B x H x W x 3 images, parameters flat."""
    off = 0
    for li, (ci, co) in enumerate(NET):
        w = theta[off:off + 9 * ci * co].reshape(9, co, ci)
        off += 9 * ci * co
        b = theta[off:off + co]
        off += co
        y = b.expand(*x.shape[:3], co)
        for tap in range(9):
            y = y + torch.roll(x, (1 - tap // 3, 1 - tap % 3), (1, 2)) @ w[tap].T
        x = torch.relu(y) if li + 1 < len(NET) else y
    return x


def exact(case, seed):
    kind = case["kind"]
    if kind == "grid":
        ex = _Exact(_shape(case), _box(case), _kernel(case), case["g"], case["model"])
        psi = ex.steps(_state(case, seed, ex.dev).to(torch.complex128), case["dz"], case["steps"])
        out = {"psi": psi}
        if case["observe"]:
            out["mass"], out["energy"] = ex.observables(psi)
        return out
    if kind == "sweep":
        if case["count"] * case["steps"] > 16000 or not torch.cuda.is_available():
            return None
        out = []
        for n, kern, psi in _instances(case, seed):
            ex = _Exact(n, (float(n[0]), float(n[1])), kern, -0.5)
            out.append(ex.steps(psi.to(torch.complex128), 1e-3, case["steps"]).cpu().numpy())
        return out
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    theta = torch.from_numpy(_weights(seed).astype(np.float64)).to(dev)
    scale = torch.tensor(SCALES, dtype=torch.float64, device=dev)
    if kind == "corrected":
        g = _corrected_grid(case)
        ex = _Exact(_shape(g), _box(g), (1.0, 0.0, 0.0, 0.0), g["g"])
        psi = _state(g, seed, ex.dev).to(torch.complex128)
        for _ in range(case["steps"]):
            psi = ex.steps(psi, g["dz"] * RATIO, 1)
            phi = ex.phi(psi.real ** 2 + psi.imag ** 2)
            res = _net((torch.stack((psi.real, psi.imag, phi), -1) * scale)[None], theta)[0]
            psi = psi + OUT_SCALE * torch.complex(res[..., 0].contiguous(), res[..., 1].contiguous())
        return {"psi": psi}
    images = _batch_tensors(case, seed, dev)
    x = torch.stack([torch.stack((p.real.double(), p.imag.double(), f.double()), -1) for p, f, _ in images]) * scale
    t = torch.stack([torch.view_as_real((fine.to(torch.complex128) - p.to(torch.complex128))) for p, _, fine in images]) / OUT_SCALE
    theta.requires_grad_(True)
    out = _net(x, theta)
    loss = ((out - t) ** 2).mean()
    (grad,) = torch.autograd.grad(loss, theta)
    return {"out": out.detach(), "loss": float(loss.detach()), "grad": grad.cpu().numpy()}
