"""dr_proxy_objective sums in 64 bits: with the same key everywhere a row's logits are equal to the last bit, its exponentials p too,
and the error of a row that keeps n of N keys is N / n - 1 whatever p is.  Sums of n terms in 64 bits are off by at most
n 2^-53 of theirs; sums in 32 bits by some 2^-24, which shows."""
import numpy as np
import pytest
import torch

import paper_2604_20470_amd as dr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("frames,hg,wg,bs", [(1, 1, 5, 32), (7, 9, 21, 32), (7, 9, 21, 64), (5, 24, 32, 128), (8, 32, 32, 32)])
@pytest.mark.parametrize("d", [64, 128])
def test_equal_logits(frames, hg, wg, bs, d):
    B, H, N = 1, 2, frames * hg * wg
    Sb = -(-N // bs)
    g = torch.Generator(device="cuda").manual_seed(N + d)
    Q = torch.randn(B, H, N, d, generator=g, device="cuda")
    K = torch.randn(B, H, 1, d, generator=g, device="cuda").expand(-1, -1, N, -1).contiguous()
    keep = np.random.default_rng(N).random((Sb, Sb)) < 0.4
    keep[:, 0] = True
    rowptr = torch.from_numpy(np.concatenate([[0], keep.sum(1).cumsum()]).astype(np.int32)).view(1, 1, -1).cuda()
    colidx = torch.from_numpy(np.nonzero(keep)[1].astype(np.int32)).view(1, 1, -1).contiguous().cuda()
    nnz = torch.tensor([[int(keep.sum())]], device="cuda")
    out = torch.zeros(3, dtype=torch.float64, device="cuda")
    dr.dr_proxy_objective(dr.Context(0), dr.shape_of(Q, frames, hg, wg, bs), Q, K, rowptr, colidx, 1, colidx.shape[2], nnz, 0.8, 10.0, out)
    width = np.minimum(np.arange(1, Sb + 1) * bs, N) - np.arange(Sb) * bs
    n = (keep * width).sum(1).astype(np.float64)                       # kept keys of a query block's rows
    # ||a_dense||^2 = 1 / N, ||a_dense - a_sparse||^2 = 1 / n - 1 / N
    want = float((width * (N / n - 1.0)).sum() / N)
    assert abs(out[1].item() - want) <= 16 * N * 2.0 ** -53 * (1.0 + want)
