"""Refresh of lists whose largest rank is at most 128, factorised in LDS in one launch: ranks at the edges of its 32-wide blocks and 64-wide
inverses.  The same matrix listed with one of a larger rank takes the kernels that go through memory, with the same operations in
the same order: the two projectors are the same bit for bit, and orthonormal to what their storage holds."""
import numpy as np
import pytest
import torch

from paper_2410_01623_amd import fira

import fira_harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [fira.FIRA_BF16, fira.FIRA_F32], ids=["bf16", "f32"])
@pytest.mark.parametrize("r", [1, 16, 31, 32, 33, 63, 64, 65, 96, 97, 127, 128])
def test_small_ranks_factorised_in_lds(r, dtype):
    shapes, ranks = [(150, 203), (211, 140), (300, 310)], [r, r, 160]
    dt = torch.bfloat16 if dtype == fira.FIRA_BF16 else torch.float32
    gen = torch.Generator(device=H.DEV).manual_seed(r)
    G = [torch.randn(s, device=H.DEV, generator=gen).to(dt) for s in shapes]
    ctx = fira.FiraContext(shapes, ranks, dtype, device=H.DEV)
    seen = []
    for idx in ([0, 1], [0, 1, 2]):
        ctx.fira_refresh_projectors(idx, [G[i] for i in idx], iters=2, seed=5)
        seen.append([ctx.fira_get_projector(i).numpy().astype(np.float64) for i in (0, 1)])
    for small, general in zip(*seen):
        assert np.array_equal(small, general)
        # bf16 entries below 1 carry 2^-9 of themselves; fp32 ones 2^-24, and the orthonormalisation its 1e-6
        assert np.abs(small.T @ small - np.eye(r)).max() <= (2.0 ** -8 if dt == torch.bfloat16 else 2e-6)
