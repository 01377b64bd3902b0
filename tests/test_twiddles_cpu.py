"""float32 twiddles of the reduced pair grids (tests/native/twiddle_check.hip,
host code): within one unit in the last place below 1 (2^-24) of the exact factors,
and with mean norm errors per leg, the energies' bias, at what the factors'
neighbours allow: on short legs the best of all choices (to a tenth of the 1e-9
that matters), on longer ones below 1e-9."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_balanced_twiddles(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "twiddle_check")
    subprocess.run([hipcc, "-std=c++17", "-O1", os.path.join(HERE, "native", "twiddle_check.hip"), "-o", exe],
                   check=True)
    out = subprocess.run([exe], capture_output=True, text=True, check=True).stdout.split()
    ulp, excess, longer, mean, plain = map(float, out)
    assert ulp <= 1.0 and excess <= 1e-10 and longer <= 1e-9, out
    assert mean < 0.5 * plain, out
