"""Host-side check of the FFT butterflies' FP64 accuracy (inline
__host__ __device__ functions, compiled here for the CPU from the same header)."""
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_fp64_butterflies_no_further_off_than_rounded_products(tmp_path):
    """Where nothing is rounded to complex64, no twiddle's product may be fused
    into the addition and the subtraction at a cost in accuracy: over every plan and
    both kinds of line the error against extended precision stays at or below that
    of products rounded on their own.  Half a percent is left for the sample: a line
    set has 2^17 values, and the two errors share most of their roundings."""
    exe = tmp_path / "host_fft"
    subprocess.run([HIPCC, "-O2", "-std=c++17", "--offload-arch=gfx950",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I" + os.path.join(ROOT, "paper_1909_08354_amd", "csrc"),
                    "-o", str(exe), os.path.join(HERE, "host_fft.hip")],
                   check=True, capture_output=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, check=True, timeout=300).stdout
    rows = np.array([[float(v) for v in line.split()] for line in out.splitlines()])
    assert rows.shape == (7 * 3 * 2, 5)
    assert np.all(rows[:, 3] < 1e-15)
    ratio = rows[:, 3] / rows[:, 4]
    assert np.all(ratio < 1.005), rows[ratio >= 1.005]
    assert ratio.mean() <= 1.0
