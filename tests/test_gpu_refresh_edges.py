"""The projector refresh at the edges of its tiles, in a workspace that holds NaNs beforehand: what the kernels read of it
they must have written.  Against the SVD of the gradient (subspace and kept energy, as in test_gpu_refresh.py)."""
import numpy as np
import pytest
import torch

from oracle import fira_oracle as orc
from paper_2410_01623_amd import fira

import fira_harness as H
from test_gpu_refresh import _gapped_gradient

pytestmark = pytest.mark.gpu

# long sides one past, one short of and well inside the 32, 64 and 128 factors of a block, a K stage and a tile; ranks around
# the 64, 128 and 256 columns of a rank tile's forms
CASES = [(70, 97, 5, 97), (97, 70, 64, 71), (100, 129, 65, 129), (130, 127, 66, 128), (191, 130, 128, 131), (130, 193, 129, 200),
         (257, 140, 130, 140), (260, 321, 256, 321), (330, 290, 257, 290)]


@pytest.mark.parametrize("dtype", [fira.FIRA_BF16, fira.FIRA_F32], ids=["bf16", "f32"])
@pytest.mark.parametrize("m,n,r,ld", CASES, ids=[f"{m}x{n}r{r}ld{ld}" for m, n, r, ld in CASES])
def test_refresh_reads_only_what_it_wrote(m, n, r, ld, dtype):
    rng = np.random.default_rng(31 * m + n)
    G = _gapped_gradient(rng, m, n, r)
    ctx = fira.FiraContext([(m, n)], r, dtype, device=H.DEV, lds=[ld])
    Gd = torch.full((m, ld), float("nan"), device=H.DEV, dtype=torch.bfloat16 if dtype == fira.FIRA_BF16 else torch.float32)
    Gd[:, :n] = torch.from_numpy(G.astype(np.float32)).to(H.DEV).to(Gd.dtype)
    ws = torch.full((ctx.fira_refresh_workspace_bytes([0]),), 0xFF, dtype=torch.uint8, device=H.DEV)
    ctx.fira_refresh_projectors([0], [Gd[:, :n]], iters=3, seed=7, workspace=ws)
    torch.cuda.synchronize()
    P = ctx.fira_get_projector(0).numpy().astype(np.float64)
    assert np.all(np.isfinite(P))
    Pref = orc.top_r_projector(G, r)
    sines = orc.subspace_sines(Pref, P)
    defect = np.max(np.abs(P.T @ P - np.eye(r)))
    e_ref, e_gpu = orc.captured_energy(G, Pref), orc.captured_energy(G, P)
    print(f"max sine {sines.max():.2e}  defect {defect:.2e}  energy svd {e_ref:.6f} device {e_gpu:.6f}", flush=True)
    # three rounds leave (0.05)^6 of the tail; the way back runs in bf16 for both types, and bf16 entries of P add ~4e-3
    assert sines.max() < 1e-2 and e_gpu > e_ref - 1e-4
    assert defect < (3e-3 if dtype == fira.FIRA_BF16 else 1e-5)
