"""What is timed: the optimizer step and the projector refresh as a training loop calls them.

A case is a list of transformer blocks (per block: four d x d matrices, two d x f, one f x d), stepped together by
one context, with the rank, storage type and options that the case names:

  op        "step":    one fira_step over every matrix (what a training loop calls once per iteration)
            "refresh": fira_refresh_projectors over every matrix, then the first fira_step with the new projectors
                       (what it calls every T iterations; that step measures the Gram gate on the residual route)
  blocks    0: a single d x f matrix
  per_block which matrices of a block are listed: 7 (all) or 5 (Q, K, V, up, down: the fine-tuning setting)
  dtype     storage type of W and G
  norm      how ||S|| is obtained: "gram" (the default) or "residual" (exact for any projector)
  planes    bf16 planes of the back-projection operand (1, or 2 for long bf16 runs)
  limited   the limiter (Eq. 12) acts on every matrix, as in the steps after a loss spike or at the start of a run
  grad      distribution of the gradients: "gauss", "colscale" (a scale per column), "student_t" (heavy tails),
            "decay" (a decaying spectrum over noise)
  pad       leading dimension of W and G rounded up to this many elements (1: dense rows)

W and G are views of flat buffers, as an optimizer that owns its parameters lays them out; two gradient sets
alternate from call to call.  Before the first timed call the optimizer has taken enough steps to be in its steady
state (from zero moments the limiter acts on the first thirty or so)."""
import math

import torch

from paper_2410_01623_amd import fira

DEV = "cuda:0"
ALIGN = 128   # elements between the starts of two matrices are a multiple of this


def _case(name, d, f, blocks, r, dtype="bf16", op="step", per_block=7, norm="gram", planes=1, limited=False, grad="gauss", pad=1):
    c = dict(op=op, d=d, f=f, blocks=blocks, per_block=per_block, r=r, dtype=dtype, norm=norm, planes=planes,
             limited=limited, grad=grad, pad=pad)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one small fp32 matrix: launches and latency
        _case("single_256x688_r64_f32", 256, 688, 0, 64, "f32"),
        # a small model, bf16: a few hundred tiles, less than the chip holds at once
        _case("llama60m_r128_bf16", 512, 1376, 8, 128, grad="colscale"),
        # a medium model, heavy-tailed gradients
        _case("llama350m_r256_bf16", 1024, 2736, 24, 256, grad="student_t"),
        # the headline workload: odd n
        _case("llama1b_r512_bf16", 2048, 5461, 24, 512),
        # a large model, rank above what one workgroup holds
        _case("llama7b_r1024_bf16", 4096, 11008, 32, 1024),
        # fine-tuning: a very small rank on large matrices, almost a pure stream
        _case("llama7b_finetune_r32_bf16", 4096, 11008, 32, 32, per_block=5),
        # fp32 weights and gradients over a whole model
        _case("llama350m_r256_f32", 1024, 2736, 24, 256, "f32"),
        # ||S|| from the residual itself (projectors that are not orthonormal, gradients inside the subspace)
        _case("llama350m_r256_bf16_residual", 1024, 2736, 24, 256, norm="residual", grad="student_t"),
        # long bf16 runs: back-projection operand in two planes
        _case("llama350m_r256_bf16_two_planes", 1024, 2736, 24, 256, planes=2, grad="student_t"),
        # the steps after a spike: the limiter acts on every matrix
        _case("llama1b_r512_bf16_limited", 2048, 5461, 24, 512, limited=True),
        # every T steps: new projectors for a small and for the headline model
        _case("refresh_llama60m_r128_bf16", 512, 1376, 8, 128, op="refresh", grad="decay"),
        _case("refresh_llama1b_r512_bf16", 2048, 5461, 24, 512, op="refresh", grad="decay"),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    op = "refresh" if rng.random() < 0.2 else "step"
    dtype = "f32" if rng.random() < 0.2 else "bf16"
    big = op == "step" and dtype == "bf16"
    d = int(_log_uniform(rng, 192, 4096 if big else 2048))
    if rng.random() < 0.5:
        d = max(192, d // 64 * 64)          # hidden sizes are mostly round, feed-forward sizes often are not
    f = int(d * rng.uniform(1.0, 3.0))
    r = int(_log_uniform(rng, 16, d / 2 if big else min(512, d / 2)))
    if rng.random() < 0.7:
        r = max(16, r // 16 * 16)
    per_block = 5 if rng.random() < 0.2 else 7
    blocks = int(_log_uniform(rng, 1, 32))
    per = 4 * d * d + 3 * d * f if per_block == 7 else 3 * d * d + 2 * d * f
    # no more memory or work than the largest listed case of the same kind
    elements = {("step", "bf16"): 6.4e9, ("step", "f32"): 3.0e8, ("refresh", "bf16"): 1.2e9, ("refresh", "f32"): 1.5e8}[op, dtype]
    blocks = max(1, min(blocks, int(elements / per)))
    kind = rng.choice(["gram", "gram", "gram", "residual", "planes", "limited"]) if op == "step" else "gram"
    if dtype == "f32" and kind == "planes":
        kind = "gram"
    return _case(None, d, f, blocks, r, dtype, op, per_block, "residual" if kind == "residual" else "gram",
                 2 if kind == "planes" else 1, kind == "limited",
                 "decay" if op == "refresh" else rng.choice(["gauss", "colscale", "student_t"]), rng.choice([1, 1, 64]))


def _shapes(case):
    d, f = case["d"], case["f"]
    if case["blocks"] == 0:
        return [(d, f)]
    block = [(d, d)] * 4 + [(d, f)] * 2 + [(f, d)] if case["per_block"] == 7 else [(d, d)] * 3 + [(d, f), (f, d)]
    return block * case["blocks"]


class _Flat:
    """One flat buffer and its matrix views."""

    def __init__(self, shapes, lds, dtype):
        starts, total = [], 0
        for (m, _), ld in zip(shapes, lds):
            starts.append(total)
            total += -(-m * ld // ALIGN) * ALIGN
        self.flat = torch.empty(total, dtype=dtype, device=DEV)
        self.views = [self.flat[s:s + m * ld].view(m, ld)[:, :n] for s, (m, n), ld in zip(starts, shapes, lds)]


def _fill_normal(flat, scale, gen):
    for part in flat.split(1 << 28):
        part.normal_(0.0, scale, generator=gen)


def _fill_gradients(case, g, scale, gen):
    _fill_normal(g.flat, scale, gen)
    if case["grad"] == "student_t":        # three degrees of freedom: normal / sqrt(chi2_3 / 3)
        for part in g.flat.split(1 << 24):
            chi2 = torch.zeros(part.numel(), device=DEV)
            for _ in range(3):
                chi2.addcmul_(*[torch.randn(part.numel(), device=DEV, generator=gen)] * 2)
            part.copy_(part.float() * (chi2 / 3.0).rsqrt())
    elif case["grad"] == "colscale":
        for v in g.views:
            v.mul_((10.0 ** (2.0 * torch.rand(v.shape[1], device=DEV, generator=gen) - 1.0)).to(v.dtype))
    elif case["grad"] == "decay":          # leading directions of falling weight over the noise, about the noise's energy
        for v in g.views:
            q = min(min(v.shape), max(64, 2 * case["r"]))
            s = torch.arange(1, q + 1, device=DEV, dtype=torch.float32).rsqrt()
            s *= scale * (s.square().sum().rsqrt())
            a = torch.randn(v.shape[0], q, device=DEV, generator=gen) * s
            v.add_((a @ torch.randn(q, v.shape[1], device=DEV, generator=gen)).to(v.dtype))


def _orthonormal(rows, r, gen):
    """A random orthonormal basis (rows x r), fp32: Cholesky QR in fp64."""
    x = torch.randn(rows, r, device=DEV, dtype=torch.float64, generator=gen)
    low = torch.linalg.cholesky(x.t() @ x)
    return torch.linalg.solve_triangular(low, x.t(), upper=False).t().float().contiguous()


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    shapes = _shapes(case)
    f32 = case["dtype"] == "f32"
    dtype = torch.float32 if f32 else torch.bfloat16
    scale = 2e-2 if case["blocks"] == 0 else 1e-3
    pad = case["pad"]
    lds = [-(-n // pad) * pad for _, n in shapes]
    idx = list(range(len(shapes)))
    w = _Flat(shapes, lds, dtype)
    _fill_normal(w.flat, 0.02, gen)
    g = [_Flat(shapes, lds, dtype) for _ in range(2)]
    for x in g:
        _fill_gradients(case, x, scale, gen)
    ctx = fira.FiraContext(shapes, case["r"], fira.FIRA_F32 if f32 else fira.FIRA_BF16, fira.make_hparams(), device=DEV, lds=lds)
    ctx.fira_set_options(norm_mode=fira.FIRA_NORM_RESIDUAL if case["norm"] == "residual" else fira.FIRA_NORM_GRAM)
    ctx.fira_set_z_planes(case["planes"])
    lists = [ctx.prepare(idx, w.views, x.views) for x in g]
    state = dict(case=case, ctx=ctx, W=w.flat, G=[x.views for x in g], idx=idx, lists=lists, calls=0, keep=(w, g))
    if case["op"] == "refresh":
        state["workspace"] = torch.empty(ctx.fira_refresh_workspace_bytes(idx), dtype=torch.uint8, device=DEV)
        state["workspace"] = ctx.fira_refresh_projectors(idx, state["G"][0], iters=2, seed=0, workspace=state["workspace"])
        for k in range(10):
            ctx.fira_step(prepared=lists[k % 2])
        return state
    bases = {}
    for m, n in shapes:
        if (min(m, n), m <= n) not in bases:
            p = _orthonormal(min(m, n), case["r"], gen)
            bases[min(m, n), m <= n] = p if f32 else p.to(dtype)
    ps = [bases[min(m, n), m <= n] for m, n in shapes]
    ctx.fira_set_projectors(idx, ps)
    for k in range(40):
        ctx.fira_step(prepared=lists[k % 2])
    if case["limited"]:                    # the part of the gradients outside the subspace grows eightfold: limited for 200 steps
        for x in g:
            for v, p in zip(x.views, ps):
                inside = p @ (p.t() @ v) if v.shape[0] <= v.shape[1] else (v @ p) @ p.t()
                v.mul_(8.0).sub_(inside, alpha=7.0)
        for k in range(2):
            ctx.fira_step(prepared=lists[k])
    state["keep"] += (ps,)
    return state


def run(state):
    ctx, k = state["ctx"], state["calls"] % 2
    state["calls"] += 1
    if state["case"]["op"] == "refresh":
        ctx.fira_refresh_projectors(state["idx"], state["G"][k], iters=2, seed=state["calls"], workspace=state["workspace"])
    ctx.fira_step(prepared=state["lists"][k])
    return state["W"]


def work(case):
    """Bytes: G read, W read and written, P read (written by a refresh, which also reads G), the two moments read and
    written in fp32.  Flops: R = P^T G and the back-projection, 2 m n r each, and one more such product where ||S||
    comes from the residual itself.  A refresh adds two rounds of two products with G and, per round, the
    orthonormalisation of its result (Gram matrix and triangular solve, S r^2 each, and r^3 / 3)."""
    size, r = (4 if case["dtype"] == "f32" else 2), case["r"]
    refresh = case["op"] == "refresh"
    nbytes = flops = 0.0
    for m, n in _shapes(case):
        long, short = max(m, n), min(m, n)
        nbytes += (3 * m * n + short * r) * size + 16 * long * r
        flops += 2.0 * m * n * r * (3 if refresh or case["norm"] == "residual" else 2)
        if refresh:
            nbytes += (m * n + short * r) * size
            flops += 2 * (4.0 * m * n * r + 2.0 * short * r * r + r ** 3 / 3)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times what was measured on W after a few calls: the same precision with the sums in another order
    (fused against two kernels), either route to ||S||, and fp32 against an fp64 restatement of the step (3.6e-7).  A
    limited bf16 step may also round its back-projection operand once or twice (6.4e-4), and a refresh hands every
    rounding on to the new basis (bf16 7.5e-4; fp32, whose way back runs in bf16, 1.3e-4 for gradients that
    differ by 1e-7).  The largest single differences are a bf16 weight that rounds to the other side."""
    refresh = case["op"] == "refresh"
    if case["dtype"] == "f32":
        return {"rel": 6e-4, "max": 0.1} if refresh else {"rel": 1.5e-6, "max": 1e-4}
    if refresh:
        return {"rel": 3e-3, "max": 0.3}
    return {"rel": 2.5e-3 if case["limited"] else 5e-4, "max": 0.6}
