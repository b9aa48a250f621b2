"""The gate values of the Gram route on the host: the library's host code with a stand-in for the HIP runtime
(tests/host_gate_check.cpp).  CPU only."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "host_gate_check.cpp")


def test_gate_values_on_the_host(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "host_gate_check")
    # the device code is left out, and with it the symbol of its image, which the stand-in never looks at
    res = subprocess.run([hipcc, "-x", "hip", "--cuda-host-only", "-std=c++17", "-O1", "-g", "-Xarch_host", "-fsanitize=address",
                          SRC, "-o", exe, "-Wl,--unresolved-symbols=ignore-in-object-files"], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    print(run.stdout[-2000:], run.stderr[-2000:])
    assert run.returncode == 0 and "0 failure(s)" in run.stdout, (run.stdout[-3000:], run.stderr[-3000:])
