"""dr_proxy_objective against the two softmax matrices in 64 bits: both head dimensions, ragged ends (a last group of 32 keys
and a last tile of 16 queries that are not full), one mask and one per head, rows that list nothing and rows that list all,
tensors that are not contiguous, logits far enough apart that the two rows of sums need their own references."""
import numpy as np
import pytest
import torch

import paper_2604_20470_amd as dr
from paper_2604_20470_amd import proxy_eval

pytestmark = pytest.mark.gpu


def _csr(keep):
    """int32 CSR of bool [B, M, Sb, Sb] with a few spare entries a mask."""
    B, M, Sb, _ = keep.shape
    cap = int(keep.sum((2, 3)).max()) + 3
    rowptr = np.zeros((B, M, Sb + 1), np.int32)
    rowptr[..., 1:] = keep.sum(-1).cumsum(-1)
    colidx = np.full((B, M, cap), -1, np.int32)
    for b in range(B):
        for m in range(M):
            cols = np.nonzero(keep[b, m])[1]
            colidx[b, m, :cols.size] = cols
    return tuple(torch.from_numpy(x).cuda() for x in (rowptr, colidx, keep.sum((2, 3)).astype(np.int64))) + (cap,)


@pytest.mark.parametrize("frames,hg,wg,bs", [(1, 1, 1, 32), (3, 3, 5, 32), (5, 6, 11, 64), (4, 8, 8, 32), (3, 11, 13, 128), (6, 10, 17, 32)])
@pytest.mark.parametrize("d,per_head,contiguous,gain", [(64, False, True, 1.0), (64, True, False, 6.0), (128, True, True, 1.0), (128, False, False, 6.0)])
def test_objective_matches_the_matrices(frames, hg, wg, bs, d, per_head, contiguous, gain):
    B, H, N = 2, 3, frames * hg * wg
    Sb = -(-N // bs)
    g = torch.Generator().manual_seed(N * d)
    q, k = (gain * torch.randn(B, H, N, d, generator=g) for _ in range(2))
    Q, K = (t.cuda() if contiguous else t.cuda().transpose(1, 2).contiguous().transpose(1, 2) for t in (q, k))
    rng = np.random.default_rng(N + d)
    keep = rng.random((B, H if per_head else 1, Sb, Sb)) < 0.5
    keep[0, 0, 0] = False                       # a row that lists nothing
    keep[1, -1, Sb - 1] = True                  # and one that lists everything
    rowptr, colidx, nnz, cap = _csr(keep)
    ctx, shape = dr.Context(0), dr.shape_of(Q, frames, hg, wg, bs)
    out = torch.full((3,), -7.0, dtype=torch.float64, device="cuda")
    got = []
    for _ in range(2):                          # the same bits on every run
        dr.dr_proxy_objective(ctx, shape, Q, K, rowptr, colidx, keep.shape[1], cap, nnz, 0.8, 10.0, out)
        got.append(out.tolist())
    assert got[0] == got[1]
    loss, nmse, sparsity = got[0]
    ratio, most = [], 0.0
    for b in range(B):
        for h in range(H):
            allowed = torch.from_numpy(keep[b, h if per_head else 0]).repeat_interleave(bs, 0)[:N].repeat_interleave(bs, 1)[:, :N]
            s = q[b, h].double() @ k[b, h].double().T / d ** 0.5
            most = max(most, float((q[b, h].abs().double() @ k[b, h].abs().double().T).max()) / d ** 0.5)
            dense = torch.softmax(s, 1)
            sparse = torch.softmax(s.masked_fill(~allowed, -torch.inf), 1).nan_to_num(0.0)
            ratio.append(float(((dense - sparse) ** 2).sum() / (dense ** 2).sum()))
    want = sum(ratio) / len(ratio)
    # A logit is off by at most (d / 16 + 4) roundings (a sum of d / 16 steps of four terms, four sums, the scale) of its terms'
    # sum of magnitudes; a probability by twice that, relatively, and 2^-20 for the exponentials and sums; a squared norm by twice
    # a probability, and the quotient of two by twice that.
    tol = 8.0 * ((d / 16 + 4) * 2.0 ** -24 * most + 2.0 ** -20)
    assert abs(nmse - want) <= tol * max(want, 1e-30), (nmse, want, tol)
    kept = float(keep.mean())
    assert abs(sparsity - (1.0 - kept)) <= 1e-12
    assert abs(loss - (nmse + 10.0 * max(0.0, 0.8 - sparsity))) <= 1e-12 * max(1.0, loss)
    if N > 1:                                   # the route over the matrices gives the same
        matrices = [proxy_eval.attention_matrix(ctx, shape, Q, K, rowptr, colidx, keep.shape[1], cap)]
        full = torch.arange(Sb, dtype=torch.int32, device="cuda").repeat(B, 1, Sb).contiguous()
        starts = (torch.arange(Sb + 1, dtype=torch.int32, device="cuda") * Sb).repeat(B, 1, 1).contiguous()
        matrices.append(proxy_eval.attention_matrix(ctx, shape, Q, K, starts, full, 1, Sb * Sb))
        dr.dr_proxy_loss(ctx, matrices[1], matrices[0], nnz, Sb, 0.8, 10.0, out)
        assert abs(out[1].item() - want) <= 4 * tol * max(want, 1e-6)


def test_arguments_are_checked():
    N, d = 64, 64
    Q = torch.zeros(1, 2, N, d, device="cuda")
    rowptr, colidx, nnz, cap = _csr(np.ones((1, 1, 2, 2), bool))
    out = torch.zeros(3, dtype=torch.float64, device="cuda")
    ctx, shape = dr.Context(0), dr.shape_of(Q, 1, 8, 8, 32)
    call = lambda **kw: dr.dr_proxy_objective(*{**dict(ctx=ctx, shape=shape, Q=Q, K=Q, rowptr=rowptr, colidx=colidx, mask_heads=1,
                                                        colidx_stride=cap, nnz=nnz, target=0.8, alpha=10.0, out=out), **kw}.values())
    call()
    for bad in (dict(Q=None), dict(out=None), dict(mask_heads=3), dict(colidx_stride=-1), dict(target=float("nan")),
                dict(Q=Q.flatten()[1:]), dict(shape=dr.shape_of(Q.bfloat16(), 1, 8, 8, 32))):
        with pytest.raises(dr.DRError):
            call(**bad)
    torch.cuda.synchronize()
