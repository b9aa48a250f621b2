"""The two fp32 projection kernels on either side of the short side (416) up to which a workgroup keeps its whole panel of the
gradient: last panel and first matrix past it, panels of 64 factors and tiles of 128 that end early, rank columns around 64, 128,
192 and 256 (one or two halves of a panel's rank columns, one or two rank tiles).  Against the CPU oracle with the bounds of
test_gpu_fp32_split.py."""
import numpy as np
import pytest
import torch

from paper_2410_01623_amd import fira

import fira_harness as H
import test_gpu_fp32_split as split

pytestmark = pytest.mark.gpu

CASES = [
    (416, 449, 64, 449), (449, 416, 65, 417),        # the largest panel
    (417, 545, 64, 545), (545, 417, 65, 419),        # the first matrix past it, one factor past whole tiles
    (430, 639, 129, 639), (639, 430, 257, 432),      # ... ragged k, middle and large rank tiles, two rank tiles
    (192, 193, 192, 193), (193, 191, 128, 191),      # whole blocks of k with full rank; a panel of one factor
    (255, 320, 193, 321), (320, 255, 254, 258),      # two passes over the rank columns, whole and half
    (63, 1030, 63, 1030), (1030, 65, 64, 66),        # few k, many panels
]


@pytest.mark.parametrize("norm", [fira.FIRA_NORM_GRAM, fira.FIRA_NORM_RESIDUAL], ids=["gram", "residual"])
@pytest.mark.parametrize("m,n,r,ld", CASES, ids=[f"{m}x{n}r{r}ld{ld}" for m, n, r, ld in CASES])
def test_fp32_step_around_the_panel(m, n, r, ld, norm):
    split.test_fp32_step_at_the_edges(m, n, r, ld, norm)


def test_a_list_with_matrices_on_either_side():
    """Panels, wider fp32 matrices and bf16 ones in one call give what they give in calls of their own, bit for bit."""
    shapes = [(200, 333), (450, 500), (333, 129), (500, 430), (150, 260), (300, 300)]
    dtypes = [fira.FIRA_F32] * 4 + [fira.FIRA_BF16] * 2
    gen = torch.Generator(device=H.DEV)
    gen.manual_seed(3)
    tt = {fira.FIRA_F32: torch.float32, fira.FIRA_BF16: torch.bfloat16}
    W0 = [torch.randn(s, device=H.DEV, generator=gen).to(tt[d]) for s, d in zip(shapes, dtypes)]
    Gs = [torch.randn(s, device=H.DEV, generator=gen).to(tt[d]) for s, d in zip(shapes, dtypes)]
    Ps = [torch.linalg.qr(torch.randn(min(s), 40, device=H.DEV, generator=gen))[0].contiguous() for s in shapes]
    out = []
    for lists in ([list(range(6))], [[i] for i in range(6)]):
        ctx = fira.FiraContext(shapes, 40, dtypes, device=H.DEV)
        ctx.fira_set_options(norm_mode=fira.FIRA_NORM_RESIDUAL)
        W = [w.clone() for w in W0]
        ctx.fira_set_projectors(list(range(6)), Ps)
        for _ in range(2):
            for idx in lists:
                ctx.fira_step(idx, [W[i] for i in idx], [Gs[i] for i in idx])
        torch.cuda.synchronize()
        out.append([(w, ctx.fira_get_lowrank(i)) for i, w in enumerate(W)])
    for (wa, ra), (wb, rb) in zip(*out):
        assert torch.equal(wa, wb) and torch.equal(ra, rb)
    for i, (s, g, p) in enumerate(zip(shapes, Gs, Ps)):
        R = (p.double().t() @ g.double() if s[0] <= s[1] else g.double() @ p.double()).cpu()
        if dtypes[i] == fira.FIRA_F32:
            # each product exact to 2^-24, sums of at most 450 of them in fp32
            assert (out[0][i][1].double() - R).abs().max() <= 1e-5 * R.abs().max()
