"""Evaluation utility on the GPU path: the objective of the paper's offline parameter search on its proxy task
(App. C: drift-proxy features, proxy attention matrix, Eq. 22).  The loss is formed by dr_proxy_objective from the features and the mask; neither
attention matrix is held.

attention_matrix gives the matrix itself, which is not an output of the hot path: it is read off the attention kernel
column block by column block.  With V set to the one-hot columns of a key range, O = A V is that column range of A.  fp32
tensors keep the read-out exact to fp32 rounding (they run the fp32 attention kernel).  Meant for the small N of the
proxy task (N x N floats are materialised).
"""
from __future__ import annotations

from typing import Tuple

from . import binding as dr

MODE_TOKENS = -1     # proxy_loss: build the mask with Algorithm 1 in its own order (token links, then aggregation)


def attention_matrix(ctx: dr.Context, shape: dr.Shape, Q, K, rowptr, colidx, mask_heads: int, capacity: int):
    """A[b, h, p, q] under the block CSR, float32 torch tensor on Q's device.  Q, K: [B, H, N, d] float32."""
    import torch
    B, H, N, d = Q.shape
    assert Q.dtype == torch.float32 and K.dtype == torch.float32, "the read-out uses the fp32 attention path"
    A = torch.empty((B, H, N, N), dtype=torch.float32, device=Q.device)
    O = torch.empty_like(Q)
    # One-hot values for the key range c0 .. c0 + w - 1 (key c0 + j carries the unit vector e_j).  With the heads' rows one
    # after the other the range is moved by moving the start of the view: every head's w unit rows sit at its last rows,
    # and a view that starts s rows later shows them s keys earlier (what it shows of the next head is zero).  The last
    # range may overlap the one before it.
    w = min(d, N)
    flat = torch.zeros((B * H * N + N, d), dtype=torch.float32, device=Q.device)
    flat[:B * H * N].view(B * H, N, d)[:, N - w:, :w] = torch.eye(w, dtype=torch.float32, device=Q.device)
    straight = Q.is_contiguous()
    V = None if straight else torch.empty_like(Q)
    for c0 in sorted({min(c, N - w) for c in range(0, N, w)}):
        s = N - w - c0
        view = flat[s:s + B * H * N].view(B, H, N, d)
        if not straight:                               # V shares the strides of Q
            V.copy_(view)
            view = V
        dr.dr_sparse_attn_fwd(ctx, shape, Q, K, view, rowptr, colidx, mask_heads, capacity, O)
        A[:, :, :, c0:c0 + w] = O[:, :, :, :w]
    torch.cuda.synchronize()
    return A


def proxy_loss(ctx: dr.Context, Q, K, Nf: int, Hg: int, Wg: int, Bs: int, mode: int, ratio_or_tau: float, lam: float,
               params: dr.MaskParams, target: float = 0.80, alpha: float = 10.0) -> Tuple[float, float, float]:
    """(loss, normalised squared error, effective sparsity) of one configuration on given features, averaged over
    (batch, head); `mode` is one of the library's selection rules or MODE_TOKENS: ||A_dense - A_sparse||_F^2 / ||A_dense||_F^2 + alpha * max(0, target - sparsity)."""
    import torch
    B, H, N, d = Q.shape
    assert Q.dtype == torch.float32 and K.dtype == torch.float32, "the objective is computed from fp32 features"
    shape = dr.shape_of(Q, Nf, Hg, Wg, Bs)
    Sb = shape.Sb
    masks = 1 if params.head_fuse > 0 else H
    # the scores are under way while the host prepares the rest
    tokens = mode == MODE_TOKENS     # ratio_or_tau is tau_1; tau_2 comes from params
    side = N if tokens else Sb
    scores = torch.empty((B, masks, side, side), dtype=torch.float32, device=Q.device)
    (dr.dr_token_scores if tokens else dr.dr_block_scores)(ctx, shape, Q, K, params.head_fuse, scores)
    cap, _ = dr.dr_mask_capacity(ctx, shape, lam, params)
    rowptr = torch.empty((B, masks, Sb + 1), dtype=torch.int32, device=Q.device)
    colidx = torch.empty((B, masks, cap), dtype=torch.int32, device=Q.device)
    nnz = torch.empty((B, masks), dtype=torch.int64, device=Q.device)
    if tokens:
        dr.dr_build_mask_tokens(ctx, shape, ratio_or_tau, lam, params, scores, rowptr, colidx, cap, nnz)
    else:
        dr.dr_build_mask(ctx, shape, mode, ratio_or_tau, lam, params, scores, rowptr, colidx, cap, nnz)
    out = torch.empty(3, dtype=torch.float64, device=Q.device)
    dr.dr_proxy_objective(ctx, shape, Q, K, rowptr, colidx, masks, cap, nnz, target, alpha, out)
    loss, nmse, sparsity = out.tolist()
    return loss, nmse, sparsity
