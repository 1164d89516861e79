"""Calls while another HIP call of the process has failed: its error stays with the
thread until someone asks for it."""
import ctypes

import numpy as np
import pytest
import torch

import paper_1909_08354_amd.gsn as gsn
from paper_1909_08354_amd import inputs

pytestmark = pytest.mark.gpu


class ForeignError:
    """Leaves the error of a failed call behind (leave), and takes it away (take)."""

    def __init__(self):
        torch.cuda.synchronize()
        path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
        self.hip = ctypes.CDLL(path)
        self.current = ctypes.c_int(0)
        assert self.hip.hipGetDevice(ctypes.byref(self.current)) == 0

    def leave(self):
        assert self.hip.hipSetDevice(1 << 20) != 0   # no such device
        assert self.hip.hipPeekAtLastError() != 0

    def take(self):
        self.hip.hipGetLastError()
        assert self.hip.hipSetDevice(self.current.value) == 0
        assert self.hip.hipGetLastError() == 0


@pytest.fixture
def foreign():
    f = ForeignError()
    yield f
    f.take()


def make_grid(n, dz=1e-3):
    L = tuple(float(v) for v in n)
    cs, ws, vs = inputs.random_lumps(np.random.default_rng(2), n, L, 2, (min(n) / 8, min(n) / 5))
    g = gsn.Grid(n, L)
    g.set_kernel(1.0, 0.0, 0.0, 0.0)
    g.set_coefficients(0.5, -0.5, dz)
    g.set_psi(inputs.lumps(n, L, cs, ws, vs).astype(np.complex64))
    return g


def test_failed_network_leaves_the_coarse_state(foreign):
    """A corrected step whose network reports an error ends with the state of its
    coarse step, in real space."""
    n = (512, 512)
    corr = gsn.Corrector(*n, 1)
    corr.set_weights(np.random.default_rng(1).normal(0, 0.1, gsn.CORRECTOR_NPARAMS))
    corr.set_scales((1.0, 1.0, 0.1), 1e-2)
    out = []
    for corrected in (False, True):
        g = make_grid(n, 5e-3)
        g.set_coarse_ratio(8)
        if corrected:
            foreign.leave()
            with pytest.raises(gsn.GsnError):
                g.step_corrected(corr, 1, 0, 0.0)
            foreign.take()
        else:
            g.step_coarse(1)
        out.append(g.get_psi(np.complex64))
        g.close()
    d = np.linalg.norm(out[1] - out[0]) / np.linalg.norm(out[0])
    # the same passes but the last inverse transform: storage roundings only
    assert d < 2 * np.sqrt(3 * 9) * 2.0 ** -24


def test_state_read_outs_report_their_own_errors(foreign):
    """sync and phase succeed whatever another call of the thread has left."""
    g = make_grid((64, 128))
    g.step(3)
    want = g.phase()
    foreign.leave()
    g.sync()
    assert g.phase() == want
    foreign.take()
    g.close()
