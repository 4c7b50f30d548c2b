"""Token links, density rule and safeguard of frames above 128 tokens, and of many smaller ones: both widths of the workgroup, steps of 1024 columns that end
inside a key block's word, query blocks that straddle frames, several masks, ties for the safeguard.  Bit for bit."""
import numpy as np
import pytest
import torch

import paper_2604_20470_amd as dr
from oracle import dynamicrad_oracle as o
from workloads import Workload

from helpers import GpuRun, assert_masks_equal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bs", [32, 64, 128])
@pytest.mark.parametrize("frames,hg,wg,B,H", [
    (4, 3, 43, 1, 1),       # N = 516: one step
    (4, 8, 32, 1, 1),       # N = 1024: exactly one
    (4, 11, 23, 2, 2),      # N = 1012
    (5, 5, 41, 1, 1),       # N = 1025: a step of one column
    (3, 1, 499, 2, 1),      # N = 1497: at block size 128 the steps leave bytes of the only word
    (9, 10, 23, 2, 2),      # N = 2070; more than 512 workgroups at block size 32
    (5, 27, 31, 2, 2),      # N = 4185; more than 512 at every block size
    (45, 5, 16, 1, 1), (29, 8, 15, 1, 1), (200, 1, 18, 1, 1),      # small frames on both sides of 12 * 2^20 token pairs
])
@pytest.mark.parametrize("tau", [0.3, 40.0])      # 40: nothing passes, the first of the best is kept
def test_masks_bit_exact(bs, frames, hg, wg, B, H, tau):
    wl = Workload("blocks", 93, B, H, 64, frames, hg, wg, bs, "f32", "iid", "dynamic", 0.5, 0.9, 1.0, head_fuse=0)
    run = GpuRun(wl, params=dr.MaskParams(gamma=1.5, head_fuse=0))
    N = wl.N
    g = torch.Generator().manual_seed(N + bs)
    scores = (torch.randn(B, H, N, N, generator=g) * 2).round() / 2      # steps of a half: many ties
    cap, _ = dr.dr_mask_capacity(run.ctx, run.shape, wl.lam, run.params)
    rowptr = torch.zeros((B, H, wl.Sb + 1), dtype=torch.int32, device="cuda")
    colidx = torch.zeros((B, H, cap), dtype=torch.int32, device="cuda")
    nnz = torch.zeros((B, H), dtype=torch.int64, device="cuda")
    # the context's bitmaps are full of bits beforehand
    big = dr.Shape(B, H, N + 4096 * frames, 64, frames, 1, N // frames + 4096, 32, 0, 0, 64, 64, 64)
    room, _ = dr.dr_mask_capacity(run.ctx, big, 1.0, run.params)
    out = [torch.zeros(n, dtype=t, device="cuda") for n, t in ((B * H * (big.Sb + 1), torch.int32), (B * H * room, torch.int32), (B * H, torch.int64))]
    dr.dr_build_mask(run.ctx, big, dr.MODE_STATIC, 1.0, 1.0, run.params, torch.zeros(B, H, big.Sb, big.Sb, device="cuda"), out[0], out[1], room, out[2])
    links = torch.full((B, H, N, N), 9, dtype=torch.uint8, device="cuda")
    dr.dr_build_mask_tokens(run.ctx, run.shape, tau, wl.lam, run.params, scores.cuda(), rowptr, colidx, cap, nnz, links)
    tab = o.frame_table(wl.Nf, wl.Nt, wl.Bs, 1.5, wl.lam)
    sc, got = scores.numpy(), links.cpu().numpy()
    assert got.max() <= 1
    for b in range(B):
        for m in range(H):
            assert (got[b, m].astype(bool) == o.select_token_links(sc[b, m], N, wl.Nt, tab, tau, tau)).all()
    assert_masks_equal(rowptr, colidx, nnz, o.build_mask_from_tokens(sc, N, wl.Nt, wl.Bs, tab, 0.15, 0.60, tau))
