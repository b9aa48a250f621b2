"""Registers of the projector refresh's kernels: none of them keeps values in memory for want of a register.  The factorisation carries 64 doubles a
lane through its elimination, so that a mask or an offset too many shows there first."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2410_01623_amd import build


def test_refresh_kernels_do_not_spill(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    src, out = tmp_path / "refresh.hip", tmp_path / "refresh.s"
    # (templates are compiled where they are launched: the Gram matrices' two forms)
    src.write_text('#include <hip/hip_runtime.h>\n#include "fira_refresh.h"\n'
                   "template __global__ void fira_refresh_gram_kernel<true>(const FiraRefreshEnt* __restrict__, int);\n"
                   "template __global__ void fira_refresh_gram_kernel<false>(const FiraRefreshEnt* __restrict__, int);\n")
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    res = subprocess.run([hipcc, *flags, "--cuda-device-only", "-S", "-I", build.CSRC, str(src), "-o", str(out)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    found = {}
    for entry in re.findall(r"- \.agpr_count.*?\.wavefront_size", out.read_text(), re.S):
        name = re.search(r"\.name:\s+(\S+)", entry).group(1)
        if "fira_refresh_" in name:
            found[name] = [int(re.search(rf"\.{key}:\s+(\d+)", entry).group(1)) for key in ("private_segment_fixed_size", "vgpr_spill_count")]
    for kernel in ("fira_refresh_chol_kernel", "fira_refresh_chol_small_kernel", "fira_refresh_solve_kernel", "fira_refresh_gram_kernelILb0", "fira_refresh_gram_kernelILb1",
                   "fira_refresh_check_kernel", "fira_refresh_diaginv_kernel"):
        assert sum(kernel in name for name in found) == 1, (kernel, sorted(found))
    assert {name: spilt for name, spilt in found.items() if any(spilt)} == {}
