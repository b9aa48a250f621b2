"""The update on quarter tiles (128 columns x 64 rows, lists of few tiles) against the oracle where it can go wrong: matrices
that end inside the first, second, third and last quarter of a tile, both orientations, both types, Z in two planes, and at
either side of the rank above which bf16 lists take whole tiles (a list's largest rank decides, so the same matrix is updated
both ways: bit for bit the same, each element being the same sums in the same order)."""
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


@pytest.mark.parametrize("dtype", [fira.FIRA_BF16, fira.FIRA_F32], ids=["bf16", "f32"])
def test_whole_and_quarter_tiles_agree_bit_for_bit(dtype):
    """The small matrices alone, and in a list that is long enough for whole tiles."""
    shapes = [(200, 333), (333, 200), (300, 700), (64, 128)] + [(1024, 2736)] * 18
    r, few = 60, 4
    gen = torch.Generator(device=H.DEV)
    gen.manual_seed(5)
    tt = torch.bfloat16 if dtype == fira.FIRA_BF16 else torch.float32
    W0 = [(0.02 * torch.randn(s, device=H.DEV, generator=gen)).to(tt) for s in shapes]
    Gs = [(1e-2 * torch.randn(s, device=H.DEV, generator=gen)).to(tt) for s in shapes]
    Ps = [torch.linalg.qr(torch.randn(min(s), r, device=H.DEV, generator=gen))[0].contiguous() for s in shapes]
    out = []
    for listed in (few, len(shapes)):
        ctx = fira.FiraContext(shapes, r, dtype, device=H.DEV)
        W = [w.clone() for w in W0]
        ctx.fira_set_projectors(list(range(len(shapes))), Ps)
        for _ in range(2):
            ctx.fira_step(list(range(listed)), W[:listed], Gs[:listed])
        torch.cuda.synchronize()
        out.append(W[:few])
    for a, b in zip(*out):
        assert torch.equal(a, b)
