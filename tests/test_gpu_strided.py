"""The two-butterfly strided pass of schedule p8 at every line length it serves
besides 512 points (whose cases are in test_gpu_solver.py): the same
butterflies, twiddles and roundings as the one-tile pass of the 8-point plan
(e8), so the two are compared bit for bit, and with the oracle (the solver's
1e-5 bar) where that is quick."""
import sys

import numpy as np
import pytest

from oracle import oracle as orc
from paper_1909_08354_amd import gsn, inputs

pytestmark = pytest.mark.gpu

STRIDED = ("kinetic_y", "kinetic", "y_fwd_rho", "kernel", "y_inv_phi")


# ragged tiles (fewer lines than a tile, half spectra plus the Nyquist line);
# 1024-point lines on both sides of the tile count that the 16-line tiles need;
# 2048-point lines, whose per-axis tables stay in global memory
@pytest.mark.parametrize("n,mode", [((256, 8), 0), ((256, 64), 1), ((8, 256, 8), 1), ((256, 16, 8), 0),
                                    ((16, 1024, 256), 1), ((1024, 32, 256), 0), ((1024, 16, 16), 1),
                                    ((2048, 8), 0), ((2048, 64), 1), ((8, 2048, 16), 0), ((2048, 8, 16), 1)])
def test_two_butterfly_lengths_bitwise(n, mode):
    print("strided", n, "mode", mode, file=sys.stderr, flush=True)
    rng = np.random.default_rng(3 + len(n))
    L = tuple(float(v) for v in n)
    cs, ws, vs = inputs.random_lumps(rng, n, L, 2, (max(1.5, min(n) / 6), max(2.0, min(n) / 4)))
    psi = inputs.lumps_3d(n, 3, 2, np.complex64) if np.prod(n) > 1 << 20 else inputs.lumps(n, L, cs, ws, vs)
    psi = inputs.as_oracle_input(psi)
    kern, g, dz, steps = (1.0, 0.3, 0.4, 0.05), -0.5, 2e-3, 5
    names, outs = gsn.variant_names(), []
    for variant in ("p8", "e8"):
        grid = gsn.Grid(n, L)
        grid.set_kernel(*kern)
        grid.set_coefficients(0.5, g, dz)
        grid.set_schedule([names.index(variant if p in STRIDED else "p8") for p in grid.pass_names()])
        grid.set_nonlinear_mode(mode)
        grid.set_psi(psi.astype(np.complex64))
        grid.step(steps)
        outs.append((grid.get_psi(np.complex64), grid.energy(), grid.phase()))
        grid.close()
    assert np.array_equal(outs[0][0], outs[1][0])
    assert outs[0][1] == outs[1][1] and outs[0][2] == outs[1][2]
    if np.prod(n) <= 1 << 18:
        ref = orc.evolve(psi, L, kern, 0.5, g, dz, steps)
        assert orc.rel_l2(outs[0][0].astype(np.complex128), ref) < 1e-5
