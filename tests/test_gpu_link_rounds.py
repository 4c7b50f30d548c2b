"""Sums and statistics of the frame pairs' candidate sets where a workgroup's rows end inside a run of sixteen, a round of 48 or a tile of
64 columns, where the windows are narrower than a run, and with both numbers of feeding wavefronts; three calls on one context, so that the pairs' arrival counts start anew."""
import pytest
import torch

import paper_2604_20470_amd as dr
from oracle import dynamicrad_oracle as o
from workloads import Workload

from helpers import GpuRun, assert_masks_equal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("frames,hg,wg,gamma", [
    (4, 1, 129, 0.25), (5, 1, 191, 0.25), (5, 1, 192, 1.0), (5, 1, 193, 4.0),      # windows of a block size up to whole frames
    (9, 3, 85, 1.0), (4, 16, 16, 1.0), (4, 1, 257, 0.5), (3, 1, 1087, 1.0),
    (17, 1, 199, 1.0), (18, 1, 200, 1.0), (19, 7, 19, 0.5), (17, 1, 449, 1.0),      # 1680 workgroups and more
])
def test_links_and_masks_bit_exact_call_after_call(frames, hg, wg, gamma):
    B, H = 1, 2
    wl = Workload("rounds", 95, B, H, 64, frames, hg, wg, 32, "f32", "iid", "dynamic", 0.5, 0.9, 1.0, head_fuse=0)
    run = GpuRun(wl, params=dr.MaskParams(gamma=gamma, head_fuse=0))
    N = wl.N
    cap, _ = dr.dr_mask_capacity(run.ctx, run.shape, wl.lam, run.params)
    rowptr = torch.zeros((B, H, wl.Sb + 1), dtype=torch.int32, device="cuda")
    colidx = torch.zeros((B, H, cap), dtype=torch.int32, device="cuda")
    nnz = torch.zeros((B, H), dtype=torch.int64, device="cuda")
    tab = o.frame_table(wl.Nf, wl.Nt, wl.Bs, gamma, wl.lam)
    for call, tau in enumerate((0.1, 30.0, 0.8)):                                  # 30: nothing passes
        scores = torch.randn(B, H, N, N, generator=torch.Generator().manual_seed(N + call))
        links = torch.full((B, H, N, N), 9, dtype=torch.uint8, device="cuda")
        dr.dr_build_mask_tokens(run.ctx, run.shape, tau, wl.lam, run.params, scores.cuda(), rowptr, colidx, cap, nnz, links)
        sc, got = scores.numpy(), links.cpu().numpy()
        for m in range(H):
            assert (got[0, m].astype(bool) == o.select_token_links(sc[0, m], N, wl.Nt, tab, tau, tau)).all()
        assert_masks_equal(rowptr, colidx, nnz, o.build_mask_from_tokens(sc, N, wl.Nt, wl.Bs, tab, 0.15, 0.60, tau))
