"""What a matrix of rank 128 to 512 gets must not depend on what else is listed, whether that is enough for the fused projection/Adam kernel that leaves
R in memory, too little, or holds a matrix that cannot take it: the two norms of a factor are sums in one order in both kernels, so everything that
a step leaves has the same bits.  (test_gpu_fused_with_r.py and test_gpu_fused_every_route.py have the ranks below.)"""
import pytest
import torch

from paper_2410_01623_amd import fira

import fira_harness as H
from test_gpu_fused_every_route import filled

pytestmark = pytest.mark.gpu

OPTIONS = {"residual": dict(norm_mode=fira.FIRA_NORM_RESIDUAL), "planes": dict(z_planes=2), "residual-planes": dict(norm_mode=fira.FIRA_NORM_RESIDUAL, z_planes=2),
           "gram": {}}


def _left_after(shapes, ranks, option, fusion, limited):
    """What four steps leave of the first matrix; matrices of one shape and rank have the same inputs."""
    option = dict(option)
    ctx = fira.FiraContext(shapes, ranks, fira.FIRA_BF16, device=H.DEV)
    ctx.fira_set_z_planes(option.pop("z_planes", 1))
    ctx.fira_set_options(**{"norm_mode": fira.FIRA_NORM_GRAM, **option})
    ctx.fira_set_fusion(fusion)
    made = {}
    for (m, n), r in zip(shapes, ranks):
        if (m, n, r) not in made:
            gen = torch.Generator(device=H.DEV).manual_seed(m + n + r)
            rand = lambda *s: torch.randn(*s, device=H.DEV, generator=gen)
            G, P = 1e-2 * rand(m, n), torch.linalg.qr(rand(min(m, n), r).double())[0].float()
            inside = P @ (P.t() @ G) if m <= n else (G @ P) @ P.t()
            # (the second gradient: what lies outside the subspace has grown eightfold, and ||S|| with it)
            made[m, n, r] = ((0.02 * rand(m, n)).bfloat16(), G.bfloat16(), (8.0 * G - 7.0 * inside).bfloat16(), P.bfloat16().contiguous())
    key = [(m, n, r) for (m, n), r in zip(shapes, ranks)]
    W, idx, left = [made[k][0].clone() for k in key], list(range(len(shapes))), []
    ctx.fira_set_projectors(idx, [made[k][3] for k in key])
    for step in range(4):
        # one gradient throughout, so that the limiter acts where the step says so and nowhere else
        ctx.fira_step(idx, W, [made[k][2 if limited and step == 2 else 1] for k in key])
        M, V, s_prev, t = ctx.fira_get_state(0)
        d = dict(W=W[0].clone().cpu().view(torch.int16), M=M, V=V, k=ctx.fira_get_factors(0), s=torch.tensor([s_prev, *ctx.fira_get_diag(0)], dtype=torch.float64))
        if ctx.fira_get_gate(0)[2] != 2:         # (the fused kernel of the Gram route keeps no copy of R)
            d["R"] = ctx.fira_get_lowrank(0)
        left.append(d)
    torch.cuda.synchronize()
    return left


@pytest.mark.parametrize("option", OPTIONS)
@pytest.mark.parametrize("m,n,r", [(200, 1537, 128), (1665, 256, 128), (259, 1700, 132), (1665, 300, 240), (320, 1536, 256), (1665, 300, 260), (520, 1700, 484),
                                   (620, 1536, 512)])
def test_same_bits_whatever_is_listed(m, n, r, option):
    count = filled(m, n, r)                      # (at r = 132 and 260 the fused kernel serves the Gram route only)
    limited = option != "gram"                   # (a limited step of the Gram route forms Z from what its kernels have left: N alone, or N and R)
    lists = [([(m, n)] * count, [r] * count, True), ([(m, n)] * count, [r] * count, False), ([(m, n)], [r], True),
             ([(m, n)] * count + [(300, 260)], [r] * count + [97], True)]
    left = [_left_after(shapes, ranks, OPTIONS[option], fusion, limited) for shapes, ranks, fusion in lists]
    c = [d["s"][3].item() for d in left[0]]
    assert (c[2] < 1.0) == limited, c
    for which, other in enumerate(left[1:], 1):
        for step, (a, b) in enumerate(zip(left[0], other)):
            assert {name: int((a[name] != b[name]).sum()) for name in a if name in b} == {name: 0 for name in a if name in b}, (which, step)
