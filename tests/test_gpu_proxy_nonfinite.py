"""Features or matrices that are not finite make the objective's loss and error not finite, on both routes: a search that
minimises it must not take them for a perfect reconstruction.  The sparsity does not depend on them."""
import math

import numpy as np
import pytest
import torch

import paper_2604_20470_amd as dr
from paper_2604_20470_amd import proxy_eval

pytestmark = pytest.mark.gpu

BAD = [float("nan"), float("inf"), -float("inf"), 1e30]      # (1e30: the logits overflow)


@pytest.mark.parametrize("bad", BAD)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("where", ["Q", "K"])
def test_objective_of_one_bad_feature(d, where, bad):
    B, H, N, Sb = 2, 2, 3 * 9 * 5, 5
    g = torch.Generator(device="cuda").manual_seed(d)
    x = dict(Q=torch.randn(B, H, N, d, generator=g, device="cuda"), K=torch.randn(B, H, N, d, generator=g, device="cuda"))
    rowptr = (torch.arange(Sb + 1, dtype=torch.int32, device="cuda") * 2).repeat(B, 1, 1).contiguous()
    colidx = torch.stack([torch.tensor(sorted({i, (i + 1) % Sb})) for i in range(Sb)]).flatten().int().repeat(B, 1, 1).contiguous().cuda()
    nnz = torch.full((B, 1), 2 * Sb, dtype=torch.int64, device="cuda")
    out = torch.zeros(3, dtype=torch.float64, device="cuda")
    ctx, shape = dr.Context(0), dr.shape_of(x["Q"], 3, 9, 5, 32)
    call = lambda: dr.dr_proxy_objective(ctx, shape, x["Q"], x["K"], rowptr, colidx, 1, 2 * Sb, nnz, 0.8, 10.0, out)
    call()
    clean = out.tolist()
    assert all(math.isfinite(v) for v in clean)
    x[where][1, 0, 70, 3] = bad
    if bad == 1e30:
        x["K" if where == "Q" else "Q"][1, 0, :, 3] = 1e30
    call()
    loss, nmse, sparsity = out.tolist()
    assert not math.isfinite(loss) and not math.isfinite(nmse) and sparsity == clean[2]
    loss, nmse, _ = proxy_eval.proxy_loss(ctx, x["Q"], x["K"], 3, 9, 5, 32, dr.MODE_UNIFORM, 0.5, 1.0, dr.MaskParams(head_fuse=1))
    assert not math.isfinite(loss) and not math.isfinite(nmse)


@pytest.mark.parametrize("bad", BAD[:3])
@pytest.mark.parametrize("which", [0, 1])
def test_loss_of_one_bad_entry(which, bad):
    B, H, N = 1, 3, 50
    A = [torch.rand(B, H, N, N, device="cuda") for _ in range(2)]
    A[0][0, 1], A[1][0, 1] = 0.0, 0.0                        # a head whose dense matrix is 0 contributes 0
    nnz = torch.full((B, 1), 3, dtype=torch.int64, device="cuda")
    out = torch.zeros(3, dtype=torch.float64, device="cuda")
    ctx = dr.Context(0)
    dr.dr_proxy_loss(ctx, *A, nnz, 2, 0.8, 10.0, out)
    dense, sparse = (t.double().cpu().numpy() for t in A)
    want = np.mean([0.0 if h == 1 else ((dense[0, h] - sparse[0, h]) ** 2).sum() / (dense[0, h] ** 2).sum() for h in range(H)])
    assert abs(out[1].item() - want) <= 1e-12 * want
    A[which][0, 2, 7, 9] = bad
    dr.dr_proxy_loss(ctx, *A, nnz, 2, 0.8, 10.0, out)
    assert not math.isfinite(out[0].item()) and not math.isfinite(out[1].item()) and out[2].item() == 1.0 - 3 / 4
