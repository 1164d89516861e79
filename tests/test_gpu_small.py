"""Schedule variant s4 (the latency form of the passes) against the FP64 oracle.

Tolerances: complex64 grids keep the solver's bar of 1e-5 relative L2 (every
pass rounds its values to complex64 once; s4 rounds nothing in between);
FP64-storage grids round nothing below FP64, bar 1e-12.  The mass and the
global phase are quadratic in psi: a relative L2 error e moves them by at most
2 e (relative), so their bar is twice psi's."""
import sys

import numpy as np
import pytest

from oracle import oracle as orc
from paper_1909_08354_amd import gsn, inputs

pytestmark = pytest.mark.gpu

KERN, G, DZ = (1.0, 0.3, 0.4, 0.05), -0.5, 2e-3
BAR = {np.complex64: 1e-5, np.complex128: 1e-12}
# the shortest and longest lines of each register form, fewer lines than a
# tile holds, and more partial sums than one round of the mass block's loads
SHAPES = [(8, 8), (16, 32), (64, 128), (8, 1024), (1024, 8), (256, 256), (512, 128), (128, 512),
          (8, 16, 32), (32, 8, 8), (8, 8, 512), (64, 32, 32), (8, 2048), (2048, 32), (64, 128, 64)]


def grid_for(n, storage=np.complex64, mode=0, seed=21):
    print("small", n, storage.__name__, "mode", mode, file=sys.stderr, flush=True)
    rng = np.random.default_rng(seed)
    L = tuple(float(v) for v in n)
    w = max(1.5, min(n) / 6.0)
    cs, ws, vs = inputs.random_lumps(rng, n, L, 2, (w, 1.5 * w))
    psi = inputs.as_oracle_input(inputs.phase_noise(inputs.lumps(n, L, cs, ws, vs), 1e-3, seed + 1))
    grid = gsn.Grid(n, L, storage=storage)
    grid.set_kernel(*KERN)
    grid.set_coefficients(0.5, G, DZ)
    grid.set_schedule(gsn.variant_names().index("s4"))
    grid.set_nonlinear_mode(mode)
    grid.set_psi(psi)
    return grid, psi, L


@pytest.mark.parametrize("storage,mode", [(np.complex64, 0), (np.complex64, 1), (np.complex128, 0),
                                          (np.complex128, 1)])
@pytest.mark.parametrize("n", SHAPES)
def test_s4_matches_oracle(n, storage, mode):
    grid, psi, L = grid_for(n, storage, mode)
    for c in (1, 12, 7):
        grid.step(c)
    ref = orc.evolve(psi, L, KERN, 0.5, G, DZ, 20)
    assert orc.rel_l2(grid.get_psi(), ref) < BAR[storage]
    obs = orc.observables(ref, L, KERN, 0.5, G)
    assert abs(grid.mass() / obs["mass"] - 1) < 2 * BAR[storage]
    assert grid.phase()[1] == 20
    # the global phase K(0) <rho> dz per step comes from the mass partials
    k0 = KERN[3] + KERN[1] / KERN[2] ** 2
    theta = 20 * DZ * k0 * obs["mass"] / np.prod(L)
    assert abs(grid.phase()[0] / theta - 1) < 2 * BAR[storage]


@pytest.mark.parametrize("n", [(32, 32), (16, 16, 32)])
def test_s4_energy_and_coarse_steps(n):
    """The energy and coarse passes in this variant's tiles (the energy's
    density partials are one per wave)."""
    grid, psi, L = grid_for(n)
    obs, e = orc.observables(psi, L, KERN, 0.5, G), grid.energy()
    scale = abs(obs["kinetic"]) + abs(obs["local"]) + abs(obs["nonlocal"])
    for k in ("kinetic", "local", "nonlocal", "total"):
        assert abs(e[k] - obs[k]) < 1e-6 * scale, k
    grid.set_coarse_ratio(4)
    grid.step_coarse(5)
    assert orc.rel_l2(grid.get_psi(), orc.evolve(psi, L, KERN, 0.5, G, 4 * DZ, 5)) < BAR[np.complex64]


def test_s4_nonfinite_mass_is_reported():
    grid, psi, _ = grid_for((32, 32), mode=1)
    bad = psi.copy()
    bad[3, 5] = np.nan
    grid.set_psi(bad)
    grid.step(3)
    with pytest.raises(gsn.GsnError) as e:
        grid.sync()
    assert e.value.status == gsn.GSN_ENONFINITE


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("n", [(8, 8), (16, 32), (64, 128), (32, 512), (8, 2048), (32, 8, 64)])
def test_local_terms_and_static_potential(n, mode):
    """The phase pass with every local term (logarithmic pressure, Bohm, Kerr)
    and a static potential; psi's bar, as the terms are evaluated in FP64 from
    spectra stored as complex64."""
    import torch
    print("small local", n, "mode", mode, file=sys.stderr, flush=True)
    L = tuple(0.5 * v for v in n)
    psi = inputs.as_oracle_input(inputs.fluid_gaussian(n, L, 25.0, 4.0, noise=1e-3, seed=8))
    V = np.random.default_rng(4).uniform(-1.0, 1.0, n).astype(np.float32)
    local = (-1.02, 1.0, -1.0, 1e-10)
    g = gsn.Grid(n, L)
    g.set_kernel(0.5, 0.3, 0.2, 0.0)
    g.set_coefficients(0.5, -0.2, 1e-3)
    g.set_local_terms(*local)
    g.set_source_fields(V_ext=torch.from_numpy(V).cuda())
    g.set_schedule(gsn.variant_names().index("s4"))
    g.set_nonlinear_mode(mode)
    g.set_psi(psi)
    g.step(12)
    ref = orc.evolve_fields(psi, L, (0.5, 0.3, 0.2, 0.0), 0.5, -0.2, 1e-3, 12, (None, None, V), local=local)
    assert orc.rel_l2(g.get_psi(), ref) < BAR[np.complex64]


@pytest.mark.parametrize("n", [(64, 64, 512), (128, 64, 512)])
def test_mass_block_sums_several_rounds(n):
    """2048 and 4096 partial sums in the block that sums them: one and two rounds of
    its eight loads a thread.  After one step theta = K(0) dz <rho>; the kinetic half
    step keeps the mass, and rho is quadratic in values stored as complex64 by at
    most four passes before the density pass: 2 * 4 * 3 roundings of 2^-24."""
    rng = np.random.default_rng(9)
    psi = (rng.standard_normal(n) + 1j * rng.standard_normal(n)).astype(np.complex64)
    grid = gsn.Grid(n, [float(v) for v in n])
    grid.set_kernel(0.0, 0.0, 0.0, 0.7)
    grid.set_coefficients(0.5, 0.0, DZ)
    grid.set_schedule(gsn.variant_names().index("s4"))
    grid.set_psi(psi)
    grid.step(1)
    theta, steps = grid.phase()
    want = 0.7 * DZ * np.mean(np.abs(psi.astype(np.complex128)) ** 2)
    assert steps == 1 and abs(theta - want) <= 24 * 2.0 ** -24 * want
    grid.close()
