"""Masks of few rows, selected and written out in one launch, and just beyond (33 rows, 257 masks): static top-k with one and two
ratios and cumulative mass, with ties, a capacity that is too small, and what lies behind the written entries untouched."""
import pytest
import torch

import paper_2604_20470_amd as dr
from oracle import dynamicrad_oracle as o

from helpers import assert_masks_equal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("frames,hg,wg,bs,B,H", [
    (1, 3, 7, 32, 1, 1),         # one block
    (8, 4, 8, 32, 2, 3),         # 8 rows
    (16, 4, 8, 32, 1, 5),        # 16: one per wave
    (17, 4, 8, 32, 1, 1),        # 17
    (13, 7, 11, 32, 1, 2),       # 32 rows, the last block partial, blocks that straddle frames
    (33, 4, 8, 32, 1, 2),        # 33: apart
    (9, 5, 8, 32, 2, 128),       # 256 masks
    (9, 5, 8, 32, 1, 257),       # 257: apart
    (16, 8, 16, 64, 1, 2),       # 32 rows of block size 64
])
@pytest.mark.parametrize("mode,par,far", [("static", 0.3, None), ("static", 0.5, 0.2), ("static", 1.0, None), ("dynamic", 0.8, None), ("dynamic", 1.0, None)])
def test_masks_bit_exact(frames, hg, wg, bs, B, H, mode, par, far):
    N = frames * hg * wg
    Sb = -(-N // bs)
    shape = dr.Shape(B, H, N, 64, frames, hg, wg, bs, 0, 0, N * 64 * H, N * 64, 64)
    params = dr.MaskParams(head_fuse=0, gamma=2.0) if far is None else dr.MaskParams(head_fuse=0, gamma=2.0, ratio_far=far)
    ctx = dr.Context(0)
    some = (torch.randn(min(B * H, 6), Sb, Sb, generator=torch.Generator().manual_seed(Sb)) * 4).round() / 4      # ties
    scores = some.repeat(-(-B * H // some.shape[0]), 1, 1)[:B * H].view(B, H, Sb, Sb).contiguous()
    cap, _ = dr.dr_mask_capacity(ctx, shape, 1.0, params)
    code = dr.MODE_STATIC if mode == "static" else dr.MODE_DYNAMIC
    tab = o.frame_table(frames, hg * wg, bs, 2.0, 1.0)
    want = o.build_mask(scores.numpy(), o.classify_blocks(N, hg * wg, bs, tab, 0.15, 0.60), mode, par, ratio_far=far)
    most = max(int(w[0][-1]) for per in want for w in per)
    for room in (cap, max(1, most // 2)):
        rowptr = torch.full((B, H, Sb + 1), -7, dtype=torch.int32, device="cuda")
        colidx = torch.full((B * H * room + 64,), -7, dtype=torch.int32, device="cuda")
        nnz = torch.full((B, H), -7, dtype=torch.int64, device="cuda")
        dr.dr_build_mask(ctx, shape, code, par, 1.0, params, scores.cuda(), rowptr, colidx, room, nnz)
        assert (colidx[B * H * room:] == -7).all()
        got = colidx[:B * H * room].view(B, H, room).cpu()
        if room == cap:
            assert_masks_equal(rowptr, got.cuda(), nnz, want)
        for b in range(B):
            for h in range(H):
                rp, ci = want[b][h]
                assert int(nnz[b, h]) == rp[-1] and (rowptr[b, h].cpu().numpy() == rp).all()
                n = min(room, int(rp[-1]))
                assert (got[b, h, :n].numpy() == ci[:n]).all() and (got[b, h, n:] == -7).all()
