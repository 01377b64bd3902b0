"""The host side of the reduced pair grids as the library compiles it: the
resampling matrices of every reduced pipeline, unpacked from both fragment orders,
against the direct cosine sum (tests/native/resample_check.cpp, linked with
libhfx.so; no device call)."""
import os
import shutil
import subprocess

import pytest

from paper_2309_00651_amd import hfx

HERE = os.path.dirname(os.path.abspath(__file__))


def test_matrices_of_every_reduced_pipeline(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc) or not os.path.exists(hfx.LIB_PATH):
        pytest.skip("hipcc or libhfx.so not available")
    exe = str(tmp_path / "resample_check")
    lib = os.path.dirname(hfx.LIB_PATH)
    subprocess.run([hipcc, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__",
                    os.path.join(HERE, "native", "resample_check.cpp"), "-L" + lib, "-lhfx",
                    "-Wl,-rpath," + lib, "-o", exe], check=True, timeout=600)
    lines = subprocess.run([exe], capture_output=True, text=True, check=True, timeout=600).stdout.split("\n")
    grids, matrices = set(), 0
    for line in lines:
        f = line.split()
        if not f:
            continue
        if f[0] == "variant":
            n, nz, m, mz, least = map(int, f[1:])
            grids.add((n, nz, m, mz))
            assert least >= 2
        elif f[0] == "band":
            nf, m, orbital = map(int, f[1:])
            k = 2 * orbital  # pair densities
            assert 2 * k + 1 <= nf and 3 * k + 1 <= m
            # the next band, one orbital frequency more, no longer fits the samples
            assert 2 * (k + 2) + 1 > nf
        else:
            a, b, kmax = map(int, f[1:4])
            plain, split, whole, row = float(f[4]), float(f[5]), int(f[6]), float(f[7])
            # plain: one rounding of values up to 1; split: two parts, the low one
            # rounded at 2^-25; and 80-bit arithmetic in both sums of up to 85 terms
            assert plain <= 2.0 ** -53 and split <= 1e-17, line
            # the exact product: below 2^53 units of 2^-50, see resample.hpp
            assert whole == 1 and row <= 8.0, line
            assert kmax < a / 2 and b % 2 == 0
            matrices += 1
    assert matrices == 64
    assert grids == {(64, 64, 48, 48), (72, 72, 60, 60), (80, 80, 60, 60), (96, 96, 72, 72),
                     (108, 108, 80, 80), (120, 120, 96, 96), (128, 128, 96, 96), (64, 128, 48, 96)}
