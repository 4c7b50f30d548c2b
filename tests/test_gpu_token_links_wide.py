"""Token-level links and their aggregation where a row is longer than one step of the aggregation (4096 columns), frames are
no multiple of a wavefront, and rows are aligned to nothing: bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import paper_2604_20470_amd as dr
from oracle import dynamicrad_oracle as o
from workloads import Workload

from helpers import GpuRun, assert_masks_equal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bs", [32, 64, 128])
@pytest.mark.parametrize("frames,hg,wg,tau", [
    (5, 31, 33, 0.2), (9, 3, 157, 60.0),                      # N = 5115 and 4239; the second: safeguard only
    (3, 1, 5, 0.2), (2, 2, 4, 0.2), (4, 9, 11, 0.2),          # N = 15, 16, 396: rows shared out over idle threads
    (16, 8, 16, 0.2), (23, 1, 89, 0.2),                       # N = 2048 and 2047: half of the threads have a row of their own
    (5, 1, 127, 0.2), (5, 3, 43, 0.2), (5, 3, 43, 60.0),      # frames of 127 and 129 tokens: one launch and five
    (70, 1, 1, 0.2), (40, 1, 3, 60.0),                        # frames of one token and of three
])
def test_links_and_masks_bit_exact(bs, frames, hg, wg, tau):
    wl = Workload("wide", 91, 1, 1, 64, frames, hg, wg, bs, "f32", "field", "dynamic", 0.5, 0.9, 1.0, head_fuse=1)
    run = GpuRun(wl, params=dr.MaskParams(gamma=1.5, head_fuse=1))
    scores = torch.empty((1, 1, wl.N, wl.N), dtype=torch.float32, device="cuda")
    dr.dr_token_scores(run.ctx, run.shape, run.Q, run.K, 1, scores)
    cap, _ = dr.dr_mask_capacity(run.ctx, run.shape, wl.lam, run.params)
    rowptr = torch.zeros((1, 1, wl.Sb + 1), dtype=torch.int32, device="cuda")
    colidx = torch.zeros((1, 1, cap), dtype=torch.int32, device="cuda")
    nnz = torch.zeros((1, 1), dtype=torch.int64, device="cuda")
    links = torch.full((1, 1, wl.N, wl.N), 9, dtype=torch.uint8, device="cuda")
    dr.dr_build_mask_tokens(run.ctx, run.shape, tau, wl.lam, run.params, scores, rowptr, colidx, cap, nnz, links)
    tab = o.frame_table(wl.Nf, wl.Nt, wl.Bs, 1.5, wl.lam)
    sc = scores.cpu().numpy()
    want = o.select_token_links(sc[0, 0], wl.N, wl.Nt, tab, tau, tau)
    got = links[0, 0].cpu().numpy()
    assert got.max() <= 1 and (got.astype(bool) == want).all()
    assert_masks_equal(rowptr, colidx, nnz, o.build_mask_from_tokens(sc, wl.N, wl.Nt, wl.Bs, tab, 0.15, 0.60, tau))


INF, NAN = float("inf"), float("nan")


@pytest.mark.parametrize("hg,wg", [(8, 16), (3, 43)])        # a pair's links in one launch, and in five
@pytest.mark.parametrize("edits,kept", [
    ({(3, 4): INF, (5, 5): INF, (9, 8): INF}, (3, 4)),       # nothing is above a mean of infinity: the first of the best
    ({(3, 4): INF, (5, 6): -INF}, (3, 4)),
    ({(3, 4): -INF}, None),
    ({(3, 4): NAN}, None),                                    # None: the highest number of the set
    ({(3, 4): -NAN, (7, 12): NAN}, None),
])
def test_a_set_with_scores_that_are_not_finite_keeps_its_best_alone(edits, kept, hg, wg):
    """The mean or the deviation is then no number, no score passes the test, and the safeguard's one link is left."""
    frames, bs = 4, 32
    Nt, N = hg * wg, frames * hg * wg
    wl = Workload("nonfinite", 92, 1, 1, 64, frames, hg, wg, bs, "f32", "field", "dynamic", 0.5, 0.9, 1.0, head_fuse=1)
    run = GpuRun(wl, params=dr.MaskParams(gamma=1.0, head_fuse=1))
    scores = torch.randn(1, 1, N, N, generator=torch.Generator().manual_seed(3))
    tile = scores[0, 0, 0:Nt, 2 * Nt:3 * Nt]                  # frames 0 and 2: a judged pair
    for at, value in edits.items():
        tile[at] = value
    tab = o.frame_table(frames, Nt, bs, 1.0, wl.lam)
    w = int(tab["w"][2])
    assert tab["retained"][2] and all(abs(u - v) <= w for u, v in edits)
    if kept is None:
        u = torch.arange(Nt)
        inside = (u[:, None] - u[None, :]).abs() <= w
        ranked = torch.where(inside & ~tile.isnan(), tile, torch.tensor(-INF))
        kept = divmod(int(ranked.argmax()), Nt)
    cap, _ = dr.dr_mask_capacity(run.ctx, run.shape, wl.lam, run.params)
    rowptr = torch.zeros((1, 1, wl.Sb + 1), dtype=torch.int32, device="cuda")
    colidx = torch.zeros((1, 1, cap), dtype=torch.int32, device="cuda")
    nnz = torch.zeros((1, 1), dtype=torch.int64, device="cuda")
    links = torch.full((1, 1, N, N), 9, dtype=torch.uint8, device="cuda")
    dr.dr_build_mask_tokens(run.ctx, run.shape, 0.5, wl.lam, run.params, scores.cuda(), rowptr, colidx, cap, nnz, links)
    got = links[0, 0, 0:Nt, 2 * Nt:3 * Nt].cpu()
    assert [tuple(x) for x in got.nonzero().tolist()] == [kept]
