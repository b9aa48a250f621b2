"""The fused projection/Adam kernel at the ranks whose R it leaves in memory (64 < r < 128, r a multiple of four), and rows that are no multiple of
four values in the Adam kernel of its own, up to the largest rank it keeps in registers: edges of tiles and ranks, both orientations, a
limited step.  Against the CPU oracle with the bounds of the bf16 and fp32 stages (test_gpu_parity.py)."""
import numpy as np
import pytest

from oracle import fira_oracle as orc
from paper_2410_01623_amd import fira, synth

import fira_harness as H

pytestmark = pytest.mark.gpu

FILL = 200      # tiles of 128 factors from which on a list takes the fused kernel at these ranks


def run(shapes, ranks, dtype, seed, check, **kw):
    """Four steps of the listed matrices, the third one limited; matrices of one shape and rank share their inputs."""
    rng = np.random.default_rng(seed)
    name = "bf16" if dtype == fira.FIRA_BF16 else "f32"
    store = synth.as_bf16_values if name == "bf16" else (lambda x: x.astype(np.float32))
    first = {}
    alias = {i: first.setdefault((s, r), i) for i, (s, r) in enumerate(zip(shapes, ranks))}
    W, G, P = {}, {}, {}
    for i in set(alias.values()):
        (m, n), r = shapes[i], ranks[i]
        W[i] = store(0.02 * rng.standard_normal((m, n)))
        G[i] = [store(1e-2 * rng.standard_normal((m, n))) for _ in range(4)]
        P[i] = synth.store_projector(np.linalg.qr(rng.standard_normal((min(m, n), r)))[0], name)
        g, p = G[i][2].astype(np.float64), P[i].astype(np.float64)
        G[i][2] = store(8.0 * g - 7.0 * (p @ (p.T @ g) if m <= n else (g @ p) @ p.T))
    return H.run_case(shapes, ranks, dtype, 4, lambda i: W[i], lambda i, s: G[i][s], lambda i, s: P[i] if s == 0 else None,
                      orc.OracleHparams(), check=check, alias={i: j for i, j in alias.items() if i != j}, **kw)


@pytest.mark.parametrize("m,n,r", [(130, 1700, 68), (1665, 129, 124), (161, 1600, 96), (200, 1537, 100)])
def test_fused_kernel_leaves_r_behind(m, n, r):
    count = -(-FILL // -(-max(m, n) // 128))
    shapes = [(m, n)] * count + [(300, 260)]                # and a small rank, which leaves its own
    res = run(shapes, [r] * count + [40], fira.FIRA_BF16, m + n, [0, count], norm_mode=fira.FIRA_NORM_GRAM)
    print(H.fmt(res), flush=True)
    assert res.fused_steps == 0 and [rt for (_, i, rt) in res.routes if i == 0] == [0, 1, 1, 1]
    assert max(res.w_err) <= 2e-2 and res.c_min < 1.0
    assert res.worst["R"] <= 1e-5 and res.worst["M"] <= 1e-5 and res.worst["V"] <= 1e-5 and res.worst["k"] <= 1e-4
    assert res.worst["s_pre"] <= 2e-3 and res.worst["c"] <= 2e-3      # a bf16 P's orthonormality defect
    # the same list in two kernels: the same R
    two = run(shapes, [r] * count + [40], fira.FIRA_BF16, m + n, [0, count], norm_mode=fira.FIRA_NORM_GRAM, fusion=False)
    assert np.array_equal(res.ctx.fira_get_lowrank(0).numpy(), two.ctx.fira_get_lowrank(0).numpy())


@pytest.mark.parametrize("option", [{}, dict(norm_mode=fira.FIRA_NORM_RESIDUAL), dict(z_planes=2)], ids=["gram", "residual", "planes"])
@pytest.mark.parametrize("m,n,r", [(130, 300, 65), (259, 300, 255), (300, 290, 257), (520, 600, 514), (700, 620, 511)])
def test_bf16_rows_of_any_length(m, n, r, option):
    res = run([(m, n)], [r], fira.FIRA_BF16, m + n, [0], **{"norm_mode": fira.FIRA_NORM_GRAM, **option})
    print(H.fmt(res), flush=True)
    assert max(res.w_err) <= 2e-2 and res.c_min < 1.0
    assert res.worst["R"] <= 1e-5 and res.worst["M"] <= 1e-5 and res.worst["V"] <= 1e-5 and res.worst["k"] <= 1e-4
    assert res.worst["s_pre"] <= 2e-3 and res.worst["c"] <= 2e-3


@pytest.mark.parametrize("norm", [fira.FIRA_NORM_GRAM, fira.FIRA_NORM_RESIDUAL], ids=["gram", "residual"])
@pytest.mark.parametrize("m,n,r", [(40, 130, 3), (130, 97, 33), (300, 131, 66), (270, 330, 258), (520, 530, 511)])
def test_fp32_rows_of_any_length(m, n, r, norm):
    res = run([(m, n)], [r], fira.FIRA_F32, m + n, [0], norm_mode=norm)
    print(H.fmt(res), flush=True)
    assert max(res.w_err) <= 1e-4 and res.c_min < 1.0
    assert res.worst["R"] <= 1e-5 and res.worst["M"] <= 1e-5 and res.worst["V"] <= 1e-5 and res.worst["k"] <= 1e-4
    assert res.worst["s_pre"] <= 1e-3 and res.worst["c"] <= 1e-3


@pytest.mark.parametrize("m,n,r", [(130, 1700, 68), (1665, 129, 124), (161, 1600, 96), (200, 1537, 100), (1540, 300, 72), (128, 1664, 112)])
def test_what_else_is_listed_does_not_show(m, n, r):
    """The same matrix in a list long enough for the fused kernel, in the same list in two kernels, and by itself: sums in one order, so the same
    bits in everything that a step leaves."""
    count = -(-FILL // -(-max(m, n) // 128))
    left = []
    for shapes, kw in [([(m, n)] * count, {}), ([(m, n)] * count, dict(fusion=False)), ([(m, n)], {})]:
        ctx, W = (lambda res: (res.ctx, res.W_dev[0]))(run(shapes, [r] * len(shapes), fira.FIRA_BF16, m + n, [0], norm_mode=fira.FIRA_NORM_GRAM, **kw))
        M, V, s_prev, _ = ctx.fira_get_state(0)
        left.append(dict(W=H.to_host(W), M=M.numpy(), V=V.numpy(), R=ctx.fira_get_lowrank(0).numpy(), k=ctx.fira_get_factors(0).numpy(),
                         s=np.array([s_prev, *ctx.fira_get_diag(0)])))
    for other in left[1:]:
        assert {name: int(np.sum(left[0][name] != other[name])) for name in left[0]} == {name: 0 for name in left[0]}
