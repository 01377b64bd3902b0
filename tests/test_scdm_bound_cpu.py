"""The bound below which SCDM leaves a block of points out of a step: never
above the norm that the update computes for the candidate, however much of it
the new direction takes (tests/native/scdm_bound_check.cpp, host code)."""
import os
import re
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_bound_stays_below_the_updated_norm(tmp_path):
    exe = str(tmp_path / "scdm_bound_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off",
                    os.path.join(HERE, "native", "scdm_bound_check.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, check=True).stdout
    cases, over, relative, loose = map(int, re.findall(r"\d+", out))
    assert cases > 5000 and over == 0 and loose == 0, out
    assert relative > 0, out  # the cases reach where a relative margin fails
