"""The fused projection/Adam kernel in the lists whose matrices all leave R in memory whatever their rank: residual route, Z in two planes, the first
step after an installation.  One and two rank tiles, the half tile, edges of tiles and ranks, both orientations, a limited step, against the CPU
oracle with the bounds of the bf16 stages (test_gpu_parity.py); and the assembly of its forms, as for the other projections."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2410_01623_amd import build, fira

import fira_harness as H
import isa_async_check
from test_gpu_fused_with_r import run


def filled(m, n, r):
    """Copies of a matrix that nearly fill one round of the kernel's workgroups, which it asks of a list (host_launch_check.cpp pins that for these)."""
    return (500 if r <= 256 else 250) // -(-max(m, n) // 128)


@pytest.mark.gpu
@pytest.mark.parametrize("option", [dict(norm_mode=fira.FIRA_NORM_RESIDUAL), dict(norm_mode=fira.FIRA_NORM_GRAM, z_planes=2),
                                    dict(norm_mode=fira.FIRA_NORM_RESIDUAL, z_planes=2)], ids=["residual", "planes", "residual-planes"])
@pytest.mark.parametrize("m,n,r", [(130, 1700, 68), (200, 1537, 128), (1665, 300, 252), (259, 1700, 256), (1665, 520, 508), (520, 1536, 512)])
def test_fused_kernel_on_every_route(m, n, r, option):
    count = filled(m, n, r)
    shapes = [(m, n)] * count + [(300, 260)]                # and a small rank, which has its own kernel
    ranks = [r] * count + [40]
    res = run(shapes, ranks, fira.FIRA_BF16, m + n + r, [0, count], **option)
    print(H.fmt(res), flush=True)
    gram = option["norm_mode"] == fira.FIRA_NORM_GRAM
    assert res.fused_steps == 0 and [rt for (_, i, rt) in res.routes if i == 0] == ([0, 1, 1, 1] if gram else [0, 0, 0, 0])
    assert max(res.w_err) <= 2e-2 and res.c_min < 1.0
    assert res.worst["R"] <= 1e-5 and res.worst["M"] <= 1e-5 and res.worst["V"] <= 1e-5 and res.worst["k"] <= 1e-4
    assert res.worst["s_pre"] <= 2e-3 and res.worst["c"] <= 2e-3
    # the same list in two kernels: the same R and the same W
    two = run(shapes, ranks, fira.FIRA_BF16, m + n + r, [0, count], fusion=False, **option)
    assert np.array_equal(res.ctx.fira_get_lowrank(0).numpy(), two.ctx.fira_get_lowrank(0).numpy())
    a, b = H.to_host(res.W_dev[0]), H.to_host(two.W_dev[0])
    assert np.array_equal(a, b)


@pytest.mark.gpu
@pytest.mark.parametrize("option", [dict(norm_mode=fira.FIRA_NORM_RESIDUAL), dict(norm_mode=fira.FIRA_NORM_GRAM, z_planes=2)], ids=["residual", "planes"])
@pytest.mark.parametrize("m,n,r", [(130, 1700, 68), (1665, 129, 124), (161, 1600, 96)])
def test_what_else_is_listed_does_not_show(m, n, r, option):
    """Below r = 128 both kernels take the same sums in the same order: the same bits in everything that a step leaves, in a list long enough for the
    fused kernel, in the same list in two kernels, and by itself."""
    count = filled(m, n, r)
    left = []
    for shapes, kw in [([(m, n)] * count, {}), ([(m, n)] * count, dict(fusion=False)), ([(m, n)], {})]:
        res = run(shapes, [r] * len(shapes), fira.FIRA_BF16, m + n, [0], **option, **kw)
        M, V, s_prev, _ = res.ctx.fira_get_state(0)
        left.append(dict(W=H.to_host(res.W_dev[0]), M=M.numpy(), V=V.numpy(), R=res.ctx.fira_get_lowrank(0).numpy(), k=res.ctx.fira_get_factors(0).numpy(),
                         s=np.array([s_prev, *res.ctx.fira_get_diag(0)])))
    for other in left[1:]:
        assert {name: int(np.sum(left[0][name] != other[name])) for name in left[0]} == {name: 0 for name in left[0]}


def test_registers_of_asynchronous_loads(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    out = tmp_path / "fira.s"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    res = subprocess.run([hipcc, *flags, "--cuda-device-only", "-S", os.path.join(build.CSRC, "fira.hip"), "-o", str(out)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    ks = {k: v for k, v in isa_async_check.kernels(out.read_text()).items() if "fira_fused_leave_r" in k}
    assert len(ks) == 2, list(ks)
    for name, body in ks.items():
        n, loads, viol = isa_async_check.check_kernel(body)
        assert loads >= 8 and not viol and "scratch_" not in body, (name, loads, viol[:3])
