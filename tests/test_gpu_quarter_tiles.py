"""The update on quarter tiles (128 columns x 64 rows, lists of few tiles) against the oracle where it can go wrong: matrices
that end inside the first, second, third and last quarter of a tile, both orientations, both types, Z in two planes.  Which
tiles a matrix is updated in, and in which direction the list is walked, is decided by the rest of the list (its number of tiles, its
largest rank): bit for bit the same, each element being the same sums in the same order."""
import numpy as np
import pytest
import torch

from oracle import fira_oracle as orc
from paper_2410_01623_amd import fira, synth

import fira_harness as H

pytestmark = pytest.mark.gpu

# m, n, r, ld
CASES = [(64, 128, 16, 128), (65, 129, 20, 129), (63, 127, 33, 130), (128, 256, 64, 256), (129, 257, 65, 257), (192, 384, 100, 385),
         (257, 130, 40, 131), (385, 193, 128, 193), (130, 65, 65, 65), (9, 300, 8, 300), (300, 7, 7, 9)]


@pytest.mark.parametrize("dtype,planes", [(fira.FIRA_BF16, 1), (fira.FIRA_BF16, 2), (fira.FIRA_F32, 1)], ids=["bf16", "bf16x2", "f32"])
@pytest.mark.parametrize("m,n,r,ld", CASES, ids=[f"{m}x{n}r{r}ld{ld}" for m, n, r, ld in CASES])
def test_update_on_quarter_tiles(m, n, r, ld, dtype, planes):
    rng = np.random.default_rng(77 * m + n)
    bf = dtype == fira.FIRA_BF16
    store = synth.as_bf16_values if bf else (lambda x: x.astype(np.float32))
    W0 = store(0.02 * rng.standard_normal((m, n)))
    Gs = [store(1e-2 * rng.standard_normal((m, n))) for _ in range(3)]
    P = synth.store_projector(np.linalg.qr(rng.standard_normal((min(m, n), r)))[0], "bf16" if bf else "f32")
    buf = torch.full((m, ld), 7.0, device=H.DEV, dtype=torch.bfloat16 if bf else torch.float32)
    buf[:, :n] = H.to_device(W0, dtype)
    ctx = fira.FiraContext([(m, n)], r, dtype, device=H.DEV, lds=[ld])
    ctx.fira_set_z_planes(planes)
    ctx.fira_set_projector(0, H.to_device(P, dtype))
    st, W = orc.OracleState.zeros(m, n, r), W0.astype(np.float64)
    for g in Gs:
        gd = torch.zeros_like(buf)
        gd[:, :n] = H.to_device(g, dtype)
        ctx.fira_step([0], [buf[:, :n]], [gd[:, :n]])
        W = orc.fira_step(W, g.astype(np.float64), P.astype(np.float64), st, orc.OracleHparams(), store_bf16=bf)["W"]
    assert H.rel_max(H.to_host(buf[:, :n]), W) <= (2e-2 if bf else 1e-4)        # the types' gates
    assert bool((buf[:, n:] == 7.0).all())


# Matrices that are updated alone (quarter tiles) and with others; rows that end with and inside a group of eight, and narrower ones
SMALL = [(200, 333), (333, 200), (300, 700), (64, 128), (277, 264), (300, 7), (40, 8), (41, 9)]
MANY, ONE_BIG = [(1024, 2736)] * 18, [(4096, 4096)]         # 1584 whole tiles; 512


def _updated(small, ranks, others, other_rank, dtype, planes):
    gen = torch.Generator(device=H.DEV)
    gen.manual_seed(5)
    tt = torch.bfloat16 if dtype == fira.FIRA_BF16 else torch.float32
    W, Gs, Ps = [], [], []
    shapes, ranks = small + others, ranks + [other_rank] * len(others)
    for s, r in zip(shapes, ranks):
        W.append((0.02 * torch.randn(s, device=H.DEV, generator=gen)).to(tt))
        Gs.append((1e-2 * torch.randn(s, device=H.DEV, generator=gen)).to(tt))
        Ps.append(torch.linalg.qr(torch.randn(min(s), r, device=H.DEV, generator=gen))[0].contiguous())
    ctx = fira.FiraContext(shapes, ranks, dtype, device=H.DEV)
    ctx.fira_set_z_planes(planes)
    ctx.fira_set_fusion(False)                              # (or it would depend on the other matrices' ranks)
    ids = list(range(len(shapes)))
    ctx.fira_set_projectors(ids, Ps)
    for _ in range(2):
        ctx.fira_step(ids, W, Gs)
    torch.cuda.synchronize()
    return W[:len(small)]


# rank of the small matrices (their short side if that is less), and what they are listed with
LISTS = {
    "many": (60, MANY, 60),                       # whole tiles, forwards
    "many, backwards": (60, MANY[:1], 65),        # quarter tiles, backwards
    "many above 64": (128, MANY, 128),            # whole tiles, backwards
    "one at 256": (256, ONE_BIG, 256),            # 512 tiles and the small ones': quarter tiles
    "one at 260": (256, ONE_BIG, 260),            # ... whole tiles of bf16 matrices: the largest rank decides
    "small at 260": (260, ONE_BIG, 260),
}


@pytest.mark.parametrize("dtype,planes", [(fira.FIRA_BF16, 1), (fira.FIRA_BF16, 2), (fira.FIRA_F32, 1)], ids=["bf16", "bf16x2", "f32"])
@pytest.mark.parametrize("name", LISTS)
def test_whole_and_quarter_tiles_agree_bit_for_bit(name, dtype, planes):
    rank, others, other_rank = LISTS[name]
    ranks = [min(rank, *s) for s in SMALL]
    alone = _updated(SMALL, ranks, [], 0, dtype, planes)
    listed = _updated(SMALL, ranks, others, other_rank, dtype, planes)
    for s, a, b in zip(SMALL, alone, listed):
        assert torch.equal(a, b), s


@pytest.mark.parametrize("m,n,r", [(192, 384, 100), (385, 193, 128), (130, 650, 64)], ids=["192x384r100", "385x193r128", "130x650r64"])
def test_quarter_tiles_multiply_both_planes(m, n, r):
    """One step from weights of zero is -lr (P N + c k S) rounded to bf16; what Z's rounding leaves of it is read off in fp64 against the
    oracle's unrounded step.  One plane leaves 2^-9 of Z's elements, two 2^-17 = 7.6e-6, and max |P Z| is within max |W|: 2e-5 holds with both
    and not with one."""
    rng = np.random.default_rng(m + n)
    G = synth.as_bf16_values(1e-2 * rng.standard_normal((m, n)))
    P = synth.store_projector(np.linalg.qr(rng.standard_normal((min(m, n), r)))[0], "bf16")
    want = orc.fira_step(np.zeros((m, n)), G.astype(np.float64), P.astype(np.float64), orc.OracleState.zeros(m, n, r), orc.OracleHparams(),
                         store_bf16=False)["W"]
    off = []
    for planes in (1, 2):
        ctx = fira.FiraContext([(m, n)], r, fira.FIRA_BF16, device=H.DEV)
        ctx.fira_set_z_planes(planes)
        ctx.fira_set_projector(0, H.to_device(P, fira.FIRA_BF16))
        W = torch.zeros((m, n), device=H.DEV, dtype=torch.bfloat16)
        ctx.fira_step([0], [W], [H.to_device(G, fira.FIRA_BF16)])
        got = H.to_host(W)
        # beyond half a unit in the last place of the stored value (2^-8 of it, at least)
        off.append(float(np.max(np.abs(got - want) - 2.0 ** -8 * np.abs(want))) / float(np.max(np.abs(want))))
    print(f"beyond the rounding of W: one plane {off[0]:.2e}, two {off[1]:.2e}", flush=True)
    assert off[1] <= 2e-5 < off[0]
