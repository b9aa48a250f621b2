"""Projections at edges that test_gpu_project_edges.py leaves out, the gradient between NaNs as there: contractions of one K stage and of less than a
piece, sides below eight (whose gradients are read value by value), the 512-thread form of the fused kernel, its half tiles that leave R, and
the refresh, whose products take both orientations of a gradient."""
import numpy as np
import pytest
import torch

from oracle import fira_oracle as orc
from paper_2410_01623_amd import fira

import fira_harness as H
from test_gpu_project_edges import SIZES
from test_gpu_refresh import _gapped_gradient

pytestmark = pytest.mark.gpu


def _between_nans(m, n, ld):
    flat = torch.full((8 + m * ld + 8,), float("nan"), device=H.DEV, dtype=torch.bfloat16)
    return flat[8:8 + m * ld].view(m, ld)[:, :n]


STEPS = {   # rank, (short, long) sides, whether the second step's kernel keeps R in registers
    "one stage": (20, [(s, l) for s in (20, 21, 57, 63, 64, 65) for l in (65, 129, 200, 263)], False),
    "below eight": (3, [(3, 3), (3, 7), (3, 130), (5, 6), (5, 8), (5, 129), (7, 7), (7, 64), (7, 257), (4, 128)], False),
    "512 threads": (260, [(s, l) for s in (385, 391, 392, 449) for l in (450, 455, 513)], True),
    "half tiles that leave R": (68, 3 * SIZES, False),       # (200 tiles and more of 128 factors)
}


@pytest.mark.parametrize("right", [False, True], ids=["left", "right"])
@pytest.mark.parametrize("which", STEPS)
def test_step(which, right):
    r, sizes, drops_r = STEPS[which]
    if which == "half tiles that leave R":
        assert sum(-(-l // 128) for _, l in sizes) >= 200
    gen = torch.Generator(device=H.DEV).manual_seed(r)
    shapes = [(l, s) if right else (s, l) for s, l in sizes]
    lds = [n + 5 for _, n in shapes]
    ctx = fira.FiraContext(shapes, r, fira.FIRA_BF16, device=H.DEV, lds=lds)
    ctx.fira_set_options(norm_mode=fira.FIRA_NORM_GRAM)
    W, G, P = [], [], []
    for (m, n), ld in zip(shapes, lds):
        G.append(_between_nans(m, n, ld).copy_(torch.randn(m, n, device=H.DEV, generator=gen)))
        W.append(torch.zeros(m, ld, device=H.DEV, dtype=torch.bfloat16)[:, :n])
        q, _ = torch.linalg.qr(torch.randn(min(m, n), r, device=H.DEV, generator=gen, dtype=torch.float64))
        P.append(q.to(torch.bfloat16).contiguous())
    idx = list(range(len(shapes)))
    ctx.fira_set_projectors(idx, P)
    lists = ctx.prepare(idx, W, G)
    for step in range(2):
        ctx.fira_step(prepared=lists)
        for i, (m, n) in enumerate(shapes):
            # (a square matrix is projected from the left)
            R = (P[i].double().t() @ G[i].double() if m <= n else G[i].double() @ P[i].double()).cpu().numpy()
            M = np.asarray(ctx.fira_get_state(i)[0], dtype=np.float64)
            share = 0.1 if step == 0 else 0.19           # beta1 = 0.9, the same gradient twice
            # fp32 sums of at most 449 products and two roundings of M: 1e-5 of the largest entry
            assert np.abs(M - share * R).max() <= 1e-5 * share * np.abs(R).max(), (step, m, n)
            if step == 0 or not drops_r:
                assert np.abs(np.asarray(ctx.fira_get_lowrank(i), dtype=np.float64) - R).max() <= 1e-5 * np.abs(R).max(), (step, m, n)
            assert np.all(np.isfinite(np.asarray(ctx.fira_get_factors(i)))) and torch.isfinite(W[i].float()).all()
            assert np.isfinite(ctx.fira_get_diag(i)[0])
    assert ctx.fira_last_step_fused() == drops_r


@pytest.mark.parametrize("m,n,r", [(2, 2, 1), (3, 129, 2), (129, 3, 2), (5, 300, 3), (300, 5, 3), (7, 9, 4), (9, 7, 4), (8, 70, 5), (70, 8, 5), (20, 57, 12),
                                   (64, 63, 30), (321, 263, 68)])
def test_refresh(m, n, r):
    rng = np.random.default_rng(31 * m + n)
    G = _gapped_gradient(rng, m, n, r)
    ctx = fira.FiraContext([(m, n)], r, fira.FIRA_BF16, device=H.DEV, lds=[n + 5])
    Gd = _between_nans(m, n, n + 5).copy_(torch.from_numpy(G.astype(np.float32)))
    ws = torch.full((ctx.fira_refresh_workspace_bytes([0]),), 0xFF, dtype=torch.uint8, device=H.DEV)      # (NaNs)
    ctx.fira_refresh_projectors([0], [Gd], iters=3, seed=7, workspace=ws)
    torch.cuda.synchronize()
    P = ctx.fira_get_projector(0).numpy().astype(np.float64)
    assert np.all(np.isfinite(P))
    Pref = orc.top_r_projector(G, r)
    # (bounds as in test_gpu_refresh_edges.py)
    assert orc.subspace_sines(Pref, P).max() < 1e-2 and orc.captured_energy(G, P) > orc.captured_energy(G, Pref) - 1e-4
    # a basis that is orthonormal to 1e-4 (what its check asks), its entries rounded to bf16: eight significant bits, so that an entry moves by 2^-8 of
    # itself at most and p_a . p_b by 2^-8 (|p_a| . |p_b|) for each of the two, 2^-7 in all (few rows come near it: 4.2e-3 at 8 x 70, r = 5)
    assert np.max(np.abs(P.T @ P - np.eye(r))) <= 2.0 ** -7 + 2e-4
