"""The refresh lets a bf16 matrix out of the second orthonormalisation pass on three bf16 plane products instead of an fp64
Gram matrix, if they come out within the tolerance less all that they can be off by: that margin against the kernel's arithmetic on
the columns that lose most (tests/host_refresh_check.cpp).  CPU only."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "host_refresh_check.cpp")


def test_the_margin_covers_what_the_plane_products_lose(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "host_refresh_check")
    # the device code is left out, and with it the symbol of its image
    res = subprocess.run([hipcc, "-x", "hip", "--cuda-host-only", "-std=c++17", "-O2", SRC, "-o", exe,
                          "-Wl,--unresolved-symbols=ignore-in-object-files"], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    print(run.stdout[-2000:], run.stderr[-2000:])
    assert run.returncode == 0 and "0 failure(s)" in run.stdout, (run.stdout[-3000:], run.stderr[-3000:])
