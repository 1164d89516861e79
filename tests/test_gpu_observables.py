"""Read-outs: the sums behind mass and energy reach the host in one launch.

A column holds from a handful of values to more than eight per thread of the
summing block; the grids below give lengths on both sides of 256 and 2048.
The mass bound: both sides sum the same P FP64 squares (each within 2^-52) in
another order, so they differ by at most P * 2^-53 relative (all terms are
positive) plus that."""
import numpy as np
import pytest

import paper_1909_08354_amd.gsn as gsn

pytestmark = pytest.mark.gpu


def make(n):
    g = gsn.Grid(n, [10.0] * len(n))
    g.set_kernel(4.0, 2.0, 1.5, 0.25)
    g.set_coefficients(0.5, 0.3, 1e-3)
    rng = np.random.default_rng(5)
    psi = (rng.standard_normal(n) + 1j * rng.standard_normal(n)).astype(np.complex64)
    g.set_psi(psi)
    return g, psi


@pytest.mark.parametrize("n", [(32, 32), (64, 2048), (1024, 128), (2048, 2048), (32, 64, 128)])
def test_mass_is_the_sum_over_the_points(n):
    g, psi = make(n)
    P = np.prod(n)
    ref = np.sum(np.abs(psi.astype(np.complex128)) ** 2) * 10.0 ** len(n) / P
    assert abs(g.mass() - ref) <= (P + 4) * 2.0 ** -53 * ref
    assert g.mass() == g.mass()
    assert g.energy() == g.energy()


@pytest.mark.parametrize("n", [(32, 32), (64, 2048), (1024, 128), (32, 64, 128)])
def test_kinetic_energy_matches_its_definition(n):
    """E_kin = a * sum |k|^2 |psi_k|^2; the entry transform is stored in complex64
    and carries at most (2 + 2 ln2 N) storage roundings of 2^-24 each, squared in
    the sum: relative error below 4 (2 + 2 * 11) 2^-24."""
    g, psi = make(n)
    P = np.prod(n)
    f = np.fft.fftn(psi.astype(np.complex128)) / P
    k2 = sum(np.meshgrid(*[(2 * np.pi * np.fft.fftfreq(m) * m / 10.0) ** 2 for m in n], indexing="ij"))
    ref = 0.5 * np.sum(k2 * np.abs(f) ** 2) * 10.0 ** len(n)
    assert abs(g.energy()["kinetic"] - ref) <= 4 * 24 * 2.0 ** -24 * ref


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_non_finite_values_are_reported(bad):
    g, psi = make((64, 64))
    psi[3, 5] = bad
    g.set_psi(psi)
    with pytest.raises(gsn.GsnError):
        g.mass()
    with pytest.raises(gsn.GsnError):
        g.step(1)
        g.sync()


@pytest.mark.parametrize("n", [(32, 32, 2048), (64, 64, 512), (128, 64, 512)])
def test_energies_from_long_columns_match_their_definition(n):
    """Columns of 2048 and 4096 values (s4: a partial per wave), both sides of what a
    block of 256 threads takes in one round of eight loads.  Kinetic as above; the
    non-local energy is of fourth order in psi, so twice that bar."""
    rng = np.random.default_rng(8)
    x = [np.arange(m) * (2 * np.pi / m) for m in n]
    amp = 1.0
    for ax in range(3):
        f = 1 + 0.4 * np.cos(x[ax] + rng.uniform(0, 6)) + 0.2 * np.cos(3 * x[ax] + rng.uniform(0, 6))
        amp = amp * f.reshape([-1 if d == ax else 1 for d in range(3)])
    psi = (amp * np.exp(0.5j * amp)).astype(np.complex64)
    L = [float(m) for m in n]
    g = gsn.Grid(n, L)
    g.set_kernel(1.0, 0.3, 0.5, 0.0)
    g.set_coefficients(0.5, 0.0, 1e-3)
    g.set_schedule(gsn.variant_names().index("s4"))
    g.set_psi(psi)
    e = g.energy()
    P = np.prod(n)
    p = psi.astype(np.complex128)
    k2 = sum(np.meshgrid(*[(2 * np.pi * np.fft.fftfreq(m)) ** 2 for m in n], indexing="ij"))
    kin = 0.5 * np.sum(k2 * np.abs(np.fft.fftn(p)) ** 2) / P   # dV = 1
    rho = np.abs(p) ** 2
    K = np.where(k2 > 0, 1.0 / np.where(k2 > 0, k2, 1.0), 0.0) + 0.3 / (k2 + 0.25)
    non = -0.5 * np.sum(rho * np.fft.ifftn(K * np.fft.fftn(rho)).real)
    assert abs(e["kinetic"] - kin) <= 4 * 24 * 2.0 ** -24 * abs(kin)
    assert abs(e["nonlocal"] - non) <= 8 * 24 * 2.0 ** -24 * abs(non)
    g.close()
