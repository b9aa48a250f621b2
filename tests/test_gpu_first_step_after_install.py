"""The first step after a projector was installed does not wait for the gate values' way back to the host: it knows that
the second one is unmeasured.  Routes, gates and weights must be what a caller gets who synchronises after every call."""
import numpy as np
import pytest
import torch

from paper_2410_01623_amd import fira, synth

import fira_harness as H

pytestmark = pytest.mark.gpu

SHAPES = [(192, 320), (320, 192), (130, 259)]


def _run(dtype, wait, r):
    rng = np.random.default_rng(5)
    st = synth.as_bf16_values if dtype == fira.FIRA_BF16 else (lambda x: x.astype(np.float32))
    W = [H.to_device(st(0.02 * rng.standard_normal(s)), dtype) for s in SHAPES]
    G = [[H.to_device(st(1e-2 * rng.standard_normal(s)), dtype) for s in SHAPES] for _ in range(3)]
    bad = H.to_device(st(rng.standard_normal((130, r))), dtype)          # not orthonormal: fails the first gate
    ctx = fira.FiraContext(SHAPES, r, dtype, device=H.DEV)
    seen = []

    def sync():
        if wait:
            torch.cuda.synchronize()
            seen.append([ctx.fira_get_gate(i)[:2] for i in range(3)])

    def step(lst, g):
        ctx.fira_step(lst, [W[i] for i in lst], [G[g][i] for i in lst])
        sync()

    ws = ctx.fira_refresh_projectors([0, 1, 2], G[0], iters=2, seed=3); sync()
    step([0, 1], 0)                                   # all unmeasured
    step([0, 1, 2], 1)                                # one of them still is
    ctx.fira_set_projector(2, bad); sync()
    step([2], 0)
    step([0, 1, 2], 2)
    ws = ctx.fira_refresh_projectors([1, 2], [G[2][1], G[2][2]], iters=2, seed=4, workspace=ws); sync()
    ws = ctx.fira_refresh_projectors([0, 1, 2], G[1], iters=1, seed=9, workspace=ws); sync()   # tables rewritten at once
    step([0, 1, 2], 0)
    step([0, 1, 2], 1)
    torch.cuda.synchronize()
    return [w.clone() for w in W], [ctx.fira_get_gate(i) for i in range(3)], seen


@pytest.mark.parametrize("r", [40, 128])
@pytest.mark.parametrize("dtype", [fira.FIRA_BF16, fira.FIRA_F32], ids=["bf16", "f32"])
def test_steps_after_installation_need_no_synchronisation(dtype, r):
    Wa, ga, _ = _run(dtype, False, r)
    Wb, gb, seen = _run(dtype, True, r)
    assert ga == gb
    assert all(torch.equal(a, b) for a, b in zip(Wa, Wb))
    assert all(np.isinf(g[1]) for g in seen[0]) and all(np.isfinite(seen[1][i][1]) for i in (0, 1))


@pytest.mark.usefixtures("no_automatic_collection")
def test_what_a_graph_cannot_hold_is_refused_under_capture():
    """A refresh and a first step after an installation are refused while the stream is being captured; the capture goes on
    without them, replays, and the context goes on as a twin that was never asked."""
    side = torch.cuda.Stream(device=H.DEV)
    out = []
    for ask in (True, False):
        rng = np.random.default_rng(8)
        W = [H.to_device(synth.as_bf16_values(0.02 * rng.standard_normal(s)), fira.FIRA_BF16) for s in SHAPES]
        G = [[H.to_device(synth.as_bf16_values(1e-2 * rng.standard_normal(s)), fira.FIRA_BF16) for s in SHAPES] for _ in range(3)]
        ctx = fira.FiraContext(SHAPES, 40, fira.FIRA_BF16, device=H.DEV, stream=side)
        ws = torch.empty(ctx.fira_refresh_workspace_bytes([0, 1, 2]), dtype=torch.uint8, device=H.DEV)
        x = torch.zeros(64, device=H.DEV)

        def asked(*calls):
            if not ask:
                return
            x.zero_()
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side):
                for call in calls:
                    with pytest.raises(fira.FiraError) as ei:
                        call()
                    assert ei.value.status == fira.FIRA_ERR_HIP and "captured" in str(ei.value)
                x.add_(1.0)
            for rep in range(3):
                graph.replay()
                torch.cuda.synchronize()
                assert float(x.sum()) == 64.0 * (rep + 1)

        refresh = lambda: ctx.fira_refresh_projectors([0, 1, 2], G[0], iters=2, seed=3, workspace=ws)
        refresh_static = lambda: ctx.fira_refresh_projectors_static([0, 1, 2], G[0], iters=2, seed=3)
        step = lambda: ctx.fira_step([0, 1, 2], W, G[0])
        asked(refresh, refresh_static)
        torch.cuda.synchronize()
        refresh()
        asked(step, refresh)
        torch.cuda.synchronize()
        for g in G:
            ctx.fira_step([0, 1, 2], W, g)
        torch.cuda.synchronize()
        out.append(([w.clone() for w in W], [ctx.fira_get_gate(i) for i in range(3)], [ctx.fira_get_projector(i) for i in range(3)]))
    assert out[0][1] == out[1][1]
    assert all(torch.equal(a, b) for k in (0, 2) for a, b in zip(out[0][k], out[1][k]))
