"""Projection at the edges of its tiles: factor counts and contraction lengths around a piece of 8, a K stage of 64 and a tile of 128, in both
orientations, for the three bf16 kernels (small ranks, two kernels, fused with Adam).  The gradient lies between NaNs, so what is read past an
edge and not cleared shows.  R, and M where R stays in registers, against the product in 64 bits."""
import numpy as np
import pytest
import torch

from paper_2410_01623_amd import fira

import fira_harness as H

pytestmark = pytest.mark.gpu

SHORT = [193, 199, 200, 201, 255, 256, 257]      # 64 k + 1, 7, 8, 9, 63, 64 and one more
LONG = [259, 263, 264, 265, 320, 383, 385]
SIZES = [(s, l) for i, s in enumerate(SHORT) for j, l in enumerate(LONG) if (i + j) % 2 == 0 or j == 6]


@pytest.mark.parametrize("right", [False, True], ids=["left", "right"])
@pytest.mark.parametrize("r", [20, 68, 128, 129, 132])
def test_projection_at_edges(r, right):
    gen = torch.Generator(device=H.DEV).manual_seed(r)
    shapes = [(l, s) if right else (s, l) for s, l in SIZES]
    lds = [n + 5 for _, n in shapes]
    ctx = fira.FiraContext(shapes, r, fira.FIRA_BF16, device=H.DEV, lds=lds)
    ctx.fira_set_options(norm_mode=fira.FIRA_NORM_GRAM)
    W, G, P = [], [], []
    for (m, n), ld in zip(shapes, lds):
        flat = torch.full((8 + m * ld + 8,), float("nan"), device=H.DEV, dtype=torch.bfloat16)
        g = flat[8:8 + m * ld].view(m, ld)[:, :n]
        g.copy_(torch.randn(m, n, device=H.DEV, generator=gen))
        G.append(g)
        W.append(torch.zeros(m, ld, device=H.DEV, dtype=torch.bfloat16)[:, :n])
        q, _ = torch.linalg.qr(torch.randn(min(m, n), r, device=H.DEV, generator=gen, dtype=torch.float64))
        P.append(q.to(torch.bfloat16).contiguous())
    idx = list(range(len(shapes)))
    ctx.fira_set_projectors(idx, P)
    lists = ctx.prepare(idx, W, G)
    for step in range(2):       # the first one after an installation takes two kernels, the second the fused one where there is one
        ctx.fira_step(prepared=lists)
        for i, (m, n) in enumerate(shapes):
            Pd, Gd = P[i].double(), G[i].double()
            R = (Gd @ Pd if right else Pd.t() @ Gd).cpu().numpy()
            M = ctx.fira_get_state(i)[0]
            M = np.asarray(M, dtype=np.float64)
            share = 0.1 if step == 0 else 0.19           # beta1 = 0.9, the same gradient twice
            # fp32 sums of at most 257 products and two roundings of M: 1e-5 of the largest entry
            assert np.abs(M - share * R).max() <= 1e-5 * share * np.abs(R).max(), (step, m, n)
            if step == 0 or r < 128:
                assert np.abs(np.asarray(ctx.fira_get_lowrank(i), dtype=np.float64) - R).max() <= 1e-5 * np.abs(R).max(), (step, m, n)
            k = np.asarray(ctx.fira_get_factors(i))
            assert np.all(np.isfinite(k)) and torch.isfinite(W[i].float()).all()
            assert np.isfinite(ctx.fira_get_diag(i)[0])
    assert ctx.fira_last_step_fused() == (r in (128, 132))
