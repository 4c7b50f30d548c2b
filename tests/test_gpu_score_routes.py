"""Block scores with one wavefront per 16 x 16 outputs and with 64 x 64 tiles: rows that end inside a tile, one to five fused heads,
both head dimensions, on both sides of the rule that chooses (1700 wavefronts, 1450 where every head has its mask)."""
import pytest
import torch

import paper_2604_20470_amd as dr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks,heads,fuse", [(1, 1, 1), (15, 2, 2), (16, 3, 3), (17, 5, 5), (33, 4, 4), (33, 4, 0), (63, 2, 1), (177, 16, 0),
                                               (177, 17, 0), (720, 2, 2), (721, 2, 2), (464, 2, 2), (465, 2, 2), (177, 5, 0), (177, 6, 0)])
@pytest.mark.parametrize("d,dtype", [(64, torch.float32), (128, torch.bfloat16)])
def test_scores_match_64_bits(blocks, heads, fuse, d, dtype):
    bs = 32
    N = blocks * bs - (5 if blocks > 1 else 0)
    g = torch.Generator(device="cuda").manual_seed(blocks * 8 + heads)
    q, k = (torch.randn(2, heads, N, d, generator=g, device="cuda").to(dtype) for _ in range(2))
    masks = 1 if fuse else heads
    scores = torch.full((2, masks, blocks, blocks), float("nan"), device="cuda")
    dr.dr_block_scores(dr.Context(0), dr.shape_of(q, 1, 1, N, bs), q, k, fuse, scores)

    def pool(x):
        y = torch.zeros(2, heads, blocks * bs, d, dtype=torch.float64, device="cuda")
        y[:, :, :N] = x.double()
        n = torch.full((blocks, 1), float(bs), dtype=torch.float64, device="cuda")
        n[-1] = N - (blocks - 1) * bs
        return y.view(2, heads, blocks, bs, d).sum(3) / n

    a, b = pool(q), pool(k)
    want = torch.stack([torch.stack([a[i, h] @ b[i, h].T for h in range(heads)]) for i in range(2)]) / d ** 0.5
    size = torch.stack([torch.stack([a[i, h].abs() @ b[i, h].abs().T for h in range(heads)]) for i in range(2)]) / d ** 0.5
    if fuse:
        want, size = want[:, :fuse].mean(1, keepdim=True), size[:, :fuse].mean(1, keepdim=True)
    # pooled means are good to a few roundings of sums of 32, the product to its roundings in a row: (8 + heads * d / 8) of 2^-24
    # of the terms' sum of magnitudes is beyond either
    bound = (8 + max(fuse, 1) * d / 8) * 2.0 ** -24 * size + 2.0 ** -24 * 8 * size.mean()
    assert ((scores.double() - want).abs() <= bound).all()
