"""Rounding error of the solver against extended precision: the schedule and the
transforms may be chosen for speed only where the error does not grow."""
import numpy as np
import pytest
import scipy.fft

pytestmark = pytest.mark.gpu

KERN = (1.0, 0.3, 0.1, 0.0)
DZ, STEPS = 1e-3, 12


def say(*a):
    print(*a, flush=True)


def evolve_ld(psi, L, g):
    """STEPS split steps in extended precision (numpy's longdouble)."""
    ld = np.longdouble
    n = psi.shape
    two_pi = 2 * ld("3.14159265358979323846264338327950288")
    k2 = np.zeros(n, ld)
    for ax in range(len(n)):
        k = two_pi / ld(L[ax]) * np.fft.fftfreq(n[ax], 1.0 / n[ax]).astype(ld)
        k2 = k2 + (k * k).reshape([-1 if d == ax else 1 for d in range(len(n))])
    cN, cY, mY, _ = [ld(v) for v in KERN]
    K = np.zeros(n, ld)
    K[k2 > 0] = cN / k2[k2 > 0]
    K += cY / (k2 + mY * mY)

    def phase(t):
        return np.cos(t) + 1j * np.sin(t)

    def kinetic(p, m):
        return scipy.fft.ifftn(scipy.fft.fftn(p, workers=8) * m, workers=8)

    half, full = phase(-ld(0.25) * ld(DZ) * k2), phase(-ld(0.5) * ld(DZ) * k2)
    psi = kinetic(psi.astype(np.clongdouble), half)
    for i in range(STEPS):
        rho = psi.real ** 2 + psi.imag ** 2
        phi = scipy.fft.ifftn(K * scipy.fft.fftn(rho.astype(np.clongdouble), workers=8), workers=8).real
        psi = kinetic(psi * phase((ld(g) * rho + phi) * ld(DZ)), full if i + 1 < STEPS else half)
    return psi


def lumps(n, seed):
    from paper_1909_08354_amd import inputs
    L = tuple(float(v) for v in n)
    rng = np.random.default_rng(seed)
    cs, ws, vs = inputs.random_lumps(rng, n, L, 3, (min(n) / 8, min(n) / 5))
    return inputs.lumps(n, L, cs, ws, vs), L


def error(grid, psi, ref):
    grid.set_psi(psi)
    grid.step(STEPS)
    out = grid.get_psi(np.complex128)
    return float(np.sqrt((np.abs(out - ref) ** 2).sum() / (np.abs(ref) ** 2).sum()))


def make_grid(n, L, storage, g):
    from paper_1909_08354_amd import gsn
    grid = gsn.Grid(n, L, storage=storage)
    grid.set_kernel(*KERN)
    grid.set_coefficients(0.5, g, DZ)
    return grid


# Errors of the 16-point plan with every rotation inside a butterfly a product of
# its own, for the same inputs: the sum over seeds 1 to 3 in quadrature.
E16_C128 = {(128, 128): 7.8699e-15, (256, 256): 1.4449e-14, (512, 256): 2.1134e-14, (1024, 256): 3.0959e-14,
            (64, 64, 64): 6.8009e-15}


@pytest.mark.parametrize("n", list(E16_C128), ids=str)
def test_c128_error_of_the_16_point_plan(n):
    """A complex128 grid is as exact as with plain rotations.  The figures repeat
    exactly on one build; 2% is left for another order of the same roundings, which
    moved the errors of seven shapes by -1.0% to +1.3%."""
    total = 0.0
    for seed in (1, 2, 3):
        psi, L = lumps(n, seed)
        g = -0.5 if len(n) == 2 else 0.0
        grid = make_grid(n, L, np.complex128, g)
        grid.set_schedule(0)
        total += error(grid, psi, evolve_ld(psi, L, g)) ** 2
        grid.close()
    say(n, total ** 0.5)
    assert total ** 0.5 <= 1.02 * E16_C128[n]


# ---- read-outs and extra passes of the latency form against the 16-point plan
def wavenumbers2(n, L):
    k2 = np.zeros(n)
    for ax in range(len(n)):
        k = 2 * np.pi * np.fft.fftfreq(n[ax], d=L[ax] / n[ax])
        k2 = k2 + (k * k).reshape([-1 if d == ax else 1 for d in range(len(n))])
    return k2


SMALL = [(64, 2048), (64, 128), (32, 32, 32), (64, 64, 64), (32, 256, 64)]


def quadrature(errs):
    return float(np.sqrt(np.sum(np.square(errs))))


@pytest.mark.parametrize("n", SMALL, ids=str)
def test_potential_of_an_untuned_small_grid(n):
    """phi of a small grid's first schedule is no further off 64 bits than the
    16-point plan's (2% for the sample of roundings)."""
    errs = {}
    for seed in (1, 2, 3):
        psi, L = lumps(n, seed)
        psi = psi.astype(np.complex64)
        k2 = wavenumbers2(n, L)
        K = np.where(k2 > 0, KERN[0] / np.where(k2 > 0, k2, 1) + KERN[1] / (k2 + KERN[2] ** 2), 0.0)
        p = psi.astype(np.complex128)
        ref = np.fft.ifftn(K * np.fft.fftn(p.real ** 2 + p.imag ** 2)).real
        grid = make_grid(n, L, np.complex64, 0.0)
        grid.set_psi(psi)
        for name in ("first", "e16"):
            if name == "e16":
                grid.set_schedule(0)
            phi = grid.potential().cpu().numpy().astype(np.float64)
            errs.setdefault(name, []).append(np.linalg.norm(phi - ref) / np.linalg.norm(ref))
        grid.close()
    first, e16 = quadrature(errs["first"]), quadrature(errs["e16"])
    say(n, first, e16, first / e16)
    assert first <= 1.02 * e16


@pytest.mark.parametrize("fields", [False, True], ids=["bohm", "source"])
@pytest.mark.parametrize("n", SMALL, ids=str)
def test_laplacians_of_an_untuned_small_grid(n, fields):
    """One large step whose phase is the Laplacian term alone (the Bohm potential,
    or a potential of lap(rho)): no further off 64 bits than the 16-point plan's."""
    import torch
    errs = {}
    for seed in (1, 2, 3):
        L = tuple(float(v) for v in n)
        rng = np.random.default_rng(seed)
        rho = np.ones(n)
        for ax in range(len(n)):
            x = np.arange(n[ax]) * (2 * np.pi / n[ax])
            f = 1 + 0.3 * np.cos(3 * x + rng.uniform(0, 6)) + 0.1 * np.cos(int(n[ax] / 5) * x + rng.uniform(0, 6))
            rho = rho * f.reshape([-1 if d == ax else 1 for d in range(len(n))])
        psi = np.sqrt(rho).astype(np.complex64)
        p = psi.astype(np.complex128)
        rho = p.real ** 2 + p.imag ** 2
        k2 = wavenumbers2(n, L)
        grid = make_grid(n, L, np.complex64, 0.0)
        if fields:
            cN = 1.0
            grid.set_kernel(cN, 0.0, 0.0, 0.0)
            grid.set_source_fields(torch.zeros(n, device="cuda"), torch.ones(n, device="cuda"), None)
            # K = cN / k^2 takes lap(rho) back to -cN (rho - mean)
            U = -cN * (rho - rho.mean())
            dz = 1.0
        else:
            grid.set_kernel(0.0, 0.0, 0.0, 0.0)
            cb = -1.0
            grid.set_local_terms(0.0, 1.0, cb, 1e-10)
            s = np.sqrt(rho)
            U = cb * np.fft.ifftn(-k2 * np.fft.fftn(s)).real / (2 * s)
            dz = 1.0
        grid.set_coefficients(0.0, 0.0, dz)   # no kinetic term: the phase alone
        ref = p * np.exp(1j * U * dz)
        for name in ("first", "e16"):
            if name == "e16":
                grid.set_schedule(0)
            grid.set_psi(psi)
            grid.step(1)
            out = grid.get_psi(np.complex128)
            errs.setdefault(name, []).append(np.linalg.norm(out - ref) / np.linalg.norm(ref))
        grid.close()
    first, e16 = quadrature(errs["first"]), quadrature(errs["e16"])
    say(n, fields, first, e16, first / e16)
    assert first <= 1.02 * e16


# ---- the first schedule of large complex64 grids
LARGE = [(1024, 1024), (2048, 1024), (128, 128, 128), (64, 256, 128), (16, 1024, 128), (128, 16, 1024), (512, 64, 64),
         (8, 512, 512), (2048, 512), (32, 32, 2048)]


@pytest.mark.parametrize("model", ["kerr", "eq15"])
@pytest.mark.parametrize("n", LARGE, ids=str)
def test_untuned_large_grid_no_further_off_than_e16(n, model):
    """psi of an untuned grid after STEPS steps against the complex128 grid's (whose
    error is seven digits smaller) is no further off than on the 16-point plan.  One
    percent is left: a first schedule may run that plan in other kernels, whose
    compiler fuses other products."""
    g0 = -0.5 if len(n) == 2 else 0.0
    errs = {}
    for seed in (1, 2):
        psi, L = lumps(n, seed)
        psi = psi.astype(np.complex64)
        grid = make_grid(n, L, np.complex64, g0)
        if model == "eq15":
            grid.set_local_terms(-1.02, 2.0, 0.0, 0.0)   # a polytrope: 2 c_p rho
        exact = make_grid(n, L, np.complex128, g0 if model == "kerr" else g0 - 1.02 * 2.0)
        exact.set_psi(psi)
        exact.step(STEPS)
        ref = exact.get_psi(np.complex128)
        exact.close()
        for name in ("first", "e16"):
            if name == "e16":
                grid.set_schedule(0)
            errs.setdefault(name, []).append(error(grid, psi, ref))
        grid.close()
    first, e16 = quadrature(errs["first"]), quadrature(errs["e16"])
    say(n, model, first, e16, first / e16)
    assert first <= 1.01 * e16
