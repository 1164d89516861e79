"""The schedule a new grid starts with, on both sides of its rule: the line at
2^19 points, 256-point kinetic lines, complex128 storage.

A variant changes the order of roundings and nothing else, so the state must
agree with that of the one-tile 16-point schedule within the storage roundings
of both: each of the passes rounds once to 2^-24 (relative, per value; the LDS
exchanges of a line's transform likewise, at most two per pass), errors add in
L2, and a step has at most 9 passes: 2 * sqrt(3 * 9 * steps) * 2^-24.  With
complex128 storage everything is FP64: the same count of roundings at 2^-53,
plus ten per transform stage for the arithmetic itself, taken as 64 * 2^-53 *
(3 * 9 * steps)."""
import numpy as np
import pytest

import paper_1909_08354_amd.gsn as gsn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,storage", [
    ((32, 32), np.complex64), ((1024, 512), np.complex64), ((256, 2048), np.complex64), ((2048, 256), np.complex64),
    ((1024, 1024), np.complex64), ((2048, 512), np.complex64), ((32, 32, 32), np.complex64), ((32, 256, 64), np.complex64),
    ((128, 128, 64), np.complex64), ((256, 64, 128), np.complex64), ((64, 256, 128), np.complex64),
    ((512, 512), np.complex128), ((1024, 1024), np.complex128)])
def test_default_schedule_agrees_with_e16(n, storage):
    rng = np.random.default_rng(3)
    psi = (rng.standard_normal(n) + 1j * rng.standard_normal(n)).astype(np.complex64)
    steps, out = 3, []
    for explicit in (False, True):
        g = gsn.Grid(n, [float(m) for m in n], storage=storage)
        g.set_kernel(1.0, 0.3, 0.5, 0.1)
        g.set_coefficients(0.5, -0.5, 1e-3)
        if explicit:
            g.set_schedule([0] * len(g.pass_names()))
        g.set_psi(psi)
        g.step(steps)
        out.append(g.get_psi(np.complex128))
        names = set(g.schedule().values())
        assert names == {"e16"} if explicit else names <= {"s4", "s8", "p8", "p16", "e16"}
    d = np.linalg.norm(out[0] - out[1]) / np.linalg.norm(out[1])
    k = 3 * 9 * steps
    assert d <= (2 * np.sqrt(k) * 2.0 ** -24 if storage == np.complex64 else 64 * k * 2.0 ** -53)


@pytest.mark.parametrize("n,storage,entry,rest", [
    ((32, 32), np.complex64, "s8", "s4"), ((1024, 512), np.complex64, "s8", "s4"),
    ((128, 64, 64), np.complex64, "s8", "s4"), ((1024, 1024), np.complex64, "p16", "p16"),
    ((128, 128, 64), np.complex64, "p16", "p16"), ((8, 512, 256), np.complex64, "p16", "p16"),
    ((512, 1024), np.complex128, "s8", "s4"), ((1024, 1024), np.complex128, "e16", "e16"),
    ((64, 128, 128), np.complex128, "e16", "e16")])
def test_first_schedule_by_size_and_storage(n, storage, entry, rest):
    """The rule itself, on both sides of 2^19 points."""
    g = gsn.Grid(n, [float(m) for m in n], storage=storage)
    sched = g.schedule()
    assert sched.pop("x_entry_fft") == entry
    assert set(sched.values()) == {rest}
    assert g.nonlinear_mode() == 0
    g.close()
