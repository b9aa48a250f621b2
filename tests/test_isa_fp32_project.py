"""The fp32 projection kernel requests its gradient blocks with inline-assembly loads as the bf16 ones do
(test_isa_async_loads.py): the same static check of its compiled code."""
import os
import shutil
import subprocess

import pytest

from paper_2410_01623_amd import build
import isa_async_check


def test_registers_of_the_fp32_projection_loads_are_untouched_until_their_wait(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    out = tmp_path / "fira.s"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    cmd = [hipcc, *flags, "--cuda-device-only", "-S", os.path.join(build.CSRC, "fira.hip"), "-o", str(out)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    ks = {k: v for k, v in isa_async_check.kernels(out.read_text()).items() if "fira_fp32_project" in k}
    assert len(ks) == 1, list(ks)
    for name, body in ks.items():
        n, loads, viol = isa_async_check.check_kernel(body)
        assert loads >= 8, f"{name}: expected the pipelined loads, found {loads}"
        assert not viol, f"{name}: {len(viol)} instruction(s) touch a pending register, e.g. {viol[:3]}"
