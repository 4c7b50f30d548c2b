"""CSR emission on both sides of the number of rows from which a workgroup takes eight: masks against the oracle, and lists cut short by the
capacity of colidx, of which every entry below it is written and none beyond (stretches that end inside it included)."""
import dataclasses

import pytest
import torch

import paper_2604_20470_amd as dr
from workloads import tiny_case

from helpers import GpuRun, assert_masks_equal, oracle_class_map, oracle_masks_from

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("frames,hg,wg,heads", [
    (15, 32, 20, 3),         # 300 rows: a wavefront a row, then four and eight rows a workgroup (19 and 20 masks), then offsets apart
    (15, 32, 20, 19), (15, 32, 20, 20), (15, 32, 20, 122),
    (5, 7, 30, 181), (5, 7, 30, 182),                # 33 rows, no multiple of eight: 5973 and 6006
    (16, 64, 64, 3),         # rows of 2048 key blocks
    (5, 16, 16, 100),        # 40 rows
])
@pytest.mark.parametrize("mode,par", [("static", 0.3), ("dynamic", 0.8)])
def test_lists_against_the_oracle_and_cut_short(frames, hg, wg, heads, mode, par):
    wl = dataclasses.replace(tiny_case("tiny8"), Nf=frames, Hg=hg, Wg=wg, Bs=32, H=heads, index=133)
    ctx, params = dr.Context(0), dr.MaskParams(head_fuse=0)
    shape = dr.Shape(1, heads, wl.N, 64, frames, hg, wg, 32, 0, 0, wl.N * 64 * heads, wl.N * 64, 64)
    scores = torch.randn(1, heads, wl.Sb, wl.Sb, generator=torch.Generator().manual_seed(heads))
    full, _ = dr.dr_mask_capacity(ctx, shape, wl.lam, params)

    def build(cap):
        rowptr = torch.zeros(1, heads, wl.Sb + 1, dtype=torch.int32, device="cuda")
        colidx = torch.full((1, heads, cap), -7, dtype=torch.int32, device="cuda")
        nnz = torch.zeros(1, heads, dtype=torch.int64, device="cuda")
        dr.dr_build_mask(ctx, shape, dr.MODE_STATIC if mode == "static" else dr.MODE_DYNAMIC, par, wl.lam, params, scores.cuda(), rowptr,
                         colidx, cap, nnz)
        return rowptr, colidx, nnz

    rowptr, colidx, nnz = build(full)
    last = heads - 1
    assert_masks_equal(rowptr[:, last:], colidx[:, last:], nnz[:, last:], oracle_masks_from(scores[:, last:], oracle_class_map(wl), mode, par))
    for cap in (1, int(nnz.min()) // 2 + 1, int(nnz.max()) - 1):
        r, c, n = build(cap)
        assert torch.equal(r, rowptr) and torch.equal(n, nnz)
        written = torch.arange(cap, device="cuda") < nnz[..., None]
        assert torch.equal(c, torch.where(written, colidx[:, :, :cap], torch.full_like(c, -7)))
