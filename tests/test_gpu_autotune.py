"""What the autotuner times: the passes as a step runs them, on data that stay in
range.  The half spectrum lies in the caller's workspace behind psi and its scratch
copy, and holds what the last timed launches left there."""
import numpy as np
import pytest
import torch

import paper_1909_08354_amd.gsn as gsn
from paper_1909_08354_amd import inputs

pytestmark = pytest.mark.gpu

N, ITERS = (64, 32, 64), 6   # two untimed launches and six timed ones on each fill


def tuned_for(target, tmp_path, monkeypatch, n=N, kern=(1.0, 0.3, 0.1, 0.0)):
    """A grid tuned with every choice but the target pass's read from the file, the
    real-space state, and the half spectrum (two halves of a line's bins, Nyquist
    column apart) as the tuner leaves it."""
    L = tuple(float(v) for v in n)
    cs, ws, vs = inputs.random_lumps(np.random.default_rng(5), n, L, 3, (min(n) / 8, min(n) / 5))
    psi = inputs.lumps(n, L, cs, ws, vs).astype(np.complex64)
    cache = tmp_path / "autotune.txt"
    g = gsn.Grid(n, L)
    names = [p for p in g.pass_names() if p != target] + ["nonlinear_mode"]
    shape = f"gfx950 {len(n)}d " + "x".join(str(v) for v in n)
    cache.write_text("".join(f"{shape} {p} {0}\n" for p in names))
    monkeypatch.setenv("GSN_AUTOTUNE_CACHE", str(cache))
    g.set_kernel(*kern)
    g.set_coefficients(0.5, 0.0, 1e-3)
    g.set_psi(psi)
    g.autotune(ITERS)
    torch.cuda.synchronize()
    assert cache.read_text().count("\n") == len(names) + 1   # only the target was timed
    base = (g._ws.data_ptr() + 255 & ~255) - g._ws.data_ptr()
    P = int(np.prod(n))
    half = g._ws[base + 16 * P:base + 20 * P].cpu().numpy().view(np.complex64).reshape(n[:-1] + (n[-1] // 2,))
    assert np.array_equal(g.get_psi(np.complex64), psi)
    return g, psi.astype(np.complex128), half.astype(np.complex128)


def density_spectrum(psi):
    """The density pass's half spectrum of a state taken as x-spectral (twice the
    bins 0 .. N/2 - 1 of each row of rho)."""
    rho = np.abs(np.fft.ifft(psi, axis=-1)) ** 2
    return 2.0 * np.fft.fft(rho, axis=-1)[..., :psi.shape[-1] // 2]


@pytest.mark.parametrize("target", ["y_fwd_rho", "y_inv_phi"])
def test_plain_transforms_are_timed_at_their_own_scale(target, tmp_path, monkeypatch):
    """Eight unnormalised y transforms in place: each multiplies the norm by sqrt(Ny)
    (1e-4: eight complex64 roundings of 2^-24 each are far below)."""
    g, psi, half = tuned_for(target, tmp_path, monkeypatch)
    want = np.linalg.norm(density_spectrum(psi)) * float(N[1]) ** ((2 + ITERS) / 2)
    assert abs(np.linalg.norm(half) / want - 1) < 1e-4
    g.close()


@pytest.mark.parametrize("n", [N, (128, 256)], ids=str)
def test_kernel_pass_is_timed_on_data_in_range(n, tmp_path, monkeypatch):
    """The multiplier passes must not run the data into underflow: off k = 0 the
    spectrum of localised lumps has no empty bin, so after the timed launches
    nearly every bin is still a normal complex64 number."""
    g, _, half = tuned_for("kernel", tmp_path, monkeypatch, n)
    big = np.abs(half)
    assert np.isfinite(big).all()
    assert (big > 1.2e-38).mean() > 0.99
    g.close()
