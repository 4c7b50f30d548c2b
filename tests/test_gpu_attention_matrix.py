"""The attention matrix read off the kernel with one-hot values: column ranges that divide the sequence, that overlap at its
end, a sequence shorter than one range, several heads, and tensors that are not contiguous."""
import numpy as np
import pytest
import torch

import paper_2604_20470_amd as dr
from oracle import dynamicrad_oracle as o
from paper_2604_20470_amd import proxy_eval

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("frames,hg,wg", [(4, 8, 8), (5, 6, 11), (3, 3, 5)])      # N = 256, 330, 45
@pytest.mark.parametrize("contiguous", [True, False])
def test_matrix_matches_the_oracle(frames, hg, wg, contiguous):
    B, H, N, d, bs = 2, 3, frames * hg * wg, 64, 32
    g = torch.Generator().manual_seed(N)
    q, k = (torch.randn(B, H, N, d, generator=g) for _ in range(2))
    Q, K = (t.cuda() if contiguous else t.cuda().transpose(1, 2).contiguous().transpose(1, 2) for t in (q, k))
    assert Q.is_contiguous() == contiguous
    Sb = -(-N // bs)
    rng = np.random.default_rng(N)
    rows = [sorted({qb} | set(np.nonzero(rng.random(Sb) < 0.5)[0].tolist())) for qb in range(Sb)]
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])])
    ci = np.asarray([c for r in rows for c in r], dtype=np.int64)
    rowptr = torch.from_numpy(rp.astype(np.int32)).view(1, 1, -1).repeat(B, 1, 1).cuda()
    colidx = torch.from_numpy(ci.astype(np.int32)).view(1, 1, -1).repeat(B, 1, 1).cuda()
    A = proxy_eval.attention_matrix(dr.Context(0), dr.shape_of(Q, frames, hg, wg, bs), Q, K, rowptr, colidx, 1, len(ci))
    for b in range(B):
        for h in range(H):
            want = o.attention_matrix(q[b, h].double().numpy(), k[b, h].double().numpy(), rp, ci, bs)
            # a logit is good to 2^-22 of its terms (at most 64 * 4.5^2 / 8); a probability is at most 1
            assert np.abs(A[b, h].cpu().numpy() - want).max() <= 2.0 ** -22 * 162 + 2.0 ** -20
