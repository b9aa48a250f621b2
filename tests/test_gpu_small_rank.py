"""bf16 matrices with r <= 64, whose projection and Adam are one kernel on every route: ranks around its two forms (up to 32 and above), ranks that
are no multiple of four, both orientations, tile edges and remainders along both sides, odd leading dimensions, and every option that
decides what the kernel leaves behind.  Against the CPU oracle with the bounds of the bf16 stages (test_gpu_parity.py)."""
import numpy as np
import pytest

from oracle import fira_oracle as orc
from paper_2410_01623_amd import fira, synth

import fira_harness as H

pytestmark = pytest.mark.gpu

# m, n, r, ld
CASES = [
    (128, 256, 32, 256), (256, 128, 64, 128),        # whole tiles, whole K blocks
    (97, 129, 33, 129), (130, 97, 31, 99),           # one past and one short of a form, one past a tile
    (65, 161, 1, 161), (159, 70, 2, 71),             # a row of less than four values; ragged k
    (70, 260, 63, 261), (385, 66, 61, 66),           # tails of three and one value
    (20, 31, 20, 31), (9, 5, 5, 5),                  # full rank; less than a wavefront's factors, fewer than eight columns
]
OPTIONS = {
    "gram": {}, "residual": dict(norm_mode=fira.FIRA_NORM_RESIDUAL), "planes": dict(z_planes=2), "planes residual": dict(z_planes=2, norm_mode=fira.FIRA_NORM_RESIDUAL),
    "matrix factor": dict(scaling="matrix"), "matrix factor residual": dict(scaling="matrix", norm_mode=fira.FIRA_NORM_RESIDUAL),
    "no factor": dict(scaling="none"), "only scaling": dict(variant="only_scaling"),
}


@pytest.mark.parametrize("option", OPTIONS)
@pytest.mark.parametrize("m,n,r,ld", CASES, ids=[f"{m}x{n}r{r}ld{ld}" for m, n, r, ld in CASES])
def test_bf16_step_at_a_small_rank(m, n, r, ld, option):
    rng = np.random.default_rng(1000 * m + n)
    W0 = synth.as_bf16_values(0.02 * rng.standard_normal((m, n)))
    Gs = [synth.as_bf16_values(1e-2 * rng.standard_normal((m, n))) for _ in range(4)]
    P = synth.store_projector(np.linalg.qr(rng.standard_normal((min(m, n), r)))[0], "bf16")
    full = r == min(m, n)
    if not full:                    # the third step is limited: its part outside the subspace is eight times larger
        g, p = Gs[2].astype(np.float64), P.astype(np.float64)
        Gs[2] = synth.as_bf16_values(8.0 * g - 7.0 * (p @ (p.T @ g) if m <= n else (g @ p) @ p.T))
    res = H.run_case([(m, n)], r, fira.FIRA_BF16, 4, lambda i: W0, lambda i, s: Gs[s], lambda i, s: P if s == 0 else None,
                     orc.OracleHparams(), lds=[ld], **{"norm_mode": fira.FIRA_NORM_GRAM, **OPTIONS[option]})
    print(H.fmt(res), flush=True)
    assert res.fused_steps == 0 and all(route != 2 for (_, _, route) in res.routes)      # R is left behind on every route
    assert max(res.w_err) <= 2e-2
    # (k of a factor with one or two values carries their own relative error: fp32 sums that cancel leave up to 2^-24 sqrt(S) of the largest)
    assert res.worst["R"] <= 1e-5 and res.worst["M"] <= 1e-5 and res.worst["V"] <= 1e-5 and res.worst["k"] <= 1e-4
    if not full:                    # at full rank S is what rounding leaves of it
        # the Gram route's ||S|| carries the ~1e-3 orthonormality defect of a bf16 P
        assert res.c_min < 1.0 and res.worst["s_pre"] <= 2e-3 and res.worst["c"] <= 2e-3
