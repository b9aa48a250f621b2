"""bf16 projection with half a rank tile (64 < r <= 128, two kernels) at the ranks and sizes where it can go wrong: rank
columns past r, ranks that are no multiple of four, both orientations, tile edges and remainders along both sides, odd leading
dimensions.  Against the CPU oracle with the bounds of the bf16 stages (test_gpu_parity.py)."""
import numpy as np
import pytest

from oracle import fira_oracle as orc
from paper_2410_01623_amd import fira, synth

import fira_harness as H

pytestmark = pytest.mark.gpu

# m, n, r, ld
CASES = [
    (256, 384, 96, 384), (384, 256, 96, 256),        # whole tiles
    (127, 129, 65, 129), (130, 127, 66, 131),        # one past and one short of a tile, smallest rank of this form
    (193, 300, 100, 301), (300, 193, 127, 193),      # ragged k; one short of the largest rank
    (161, 385, 128, 388), (385, 162, 128, 163),      # the largest rank, ragged factors
    (96, 131, 96, 131), (131, 99, 99, 102),          # full rank
]


@pytest.mark.parametrize("norm", [fira.FIRA_NORM_GRAM, fira.FIRA_NORM_RESIDUAL], ids=["gram", "residual"])
@pytest.mark.parametrize("m,n,r,ld", CASES, ids=[f"{m}x{n}r{r}ld{ld}" for m, n, r, ld in CASES])
def test_bf16_step_at_half_a_rank_tile(m, n, r, ld, norm):
    rng = np.random.default_rng(1000 * m + n)
    W0 = synth.as_bf16_values(0.02 * rng.standard_normal((m, n)))
    Gs = [synth.as_bf16_values(1e-2 * rng.standard_normal((m, n))) for _ in range(4)]
    P = synth.store_projector(np.linalg.qr(rng.standard_normal((min(m, n), r)))[0], "bf16")
    full = r == min(m, n)
    if not full:                    # the third step is limited: its part outside the subspace is eight times larger
        g, p = Gs[2].astype(np.float64), P.astype(np.float64)
        Gs[2] = synth.as_bf16_values(8.0 * g - 7.0 * (p @ (p.T @ g) if m <= n else (g @ p) @ p.T))
    res = H.run_case([(m, n)], r, fira.FIRA_BF16, 4, lambda i: W0, lambda i, s: Gs[s], lambda i, s: P if s == 0 else None,
                     orc.OracleHparams(), lds=[ld], norm_mode=norm, fusion=False)
    print(H.fmt(res), flush=True)
    assert max(res.w_err) <= 2e-2
    assert res.worst["R"] <= 1e-5 and res.worst["M"] <= 1e-5 and res.worst["V"] <= 1e-5 and res.worst["k"] <= 1e-4
    if norm == fira.FIRA_NORM_GRAM and not full:
        assert [rt for (_, _, rt) in res.routes] == [0, 1, 1, 1]      # ||G_i||^2 from both waves of the first columns
    if not full:                    # at full rank S is what rounding leaves of it
        # the Gram route's ||S|| carries the ~1e-3 orthonormality defect of a bf16 P
        assert res.c_min < 1.0 and res.worst["s_pre"] <= 2e-3 and res.worst["c"] <= 2e-3
