"""CSR emission with the row offsets in the same launch and in one of their own: many masks at once, on both sides of the
rule that chooses, give every mask what the oracle gives one."""
import dataclasses

import pytest
import torch

import paper_2604_20470_amd as dr
from workloads import tiny_case

from helpers import GpuRun, assert_masks_equal, oracle_class_map, oracle_masks_from

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("frames,hg,wg,heads", [
    (15, 32, 20, 95),        # 300 rows: 121 and 122 masks are the rule's two sides
    (15, 32, 20, 96),
    (15, 32, 20, 121),
    (15, 32, 20, 122),
    (16, 64, 64, 8),         # 2048 rows, the longest of one wavefront: 64 and 65
    (16, 64, 64, 9),
    (16, 64, 64, 64),
    (16, 64, 64, 65),
    (4, 16, 20, 749),        # 40 rows: 749 and 750
    (4, 16, 20, 750),
    (5, 7, 30, 911),         # 33 rows, no multiple of a workgroup's four: 909 and 910
])
@pytest.mark.parametrize("mode,par", [("static", 0.1), ("uniform", 0.1)])
def test_every_mask_alike(frames, hg, wg, heads, mode, par):
    wl = dataclasses.replace(tiny_case("tiny8"), Nf=frames, Hg=hg, Wg=wg, Bs=32, H=heads, index=131)
    run = GpuRun.__new__(GpuRun)
    run.wl, run.heads, run.params, run.device, run.Sb = wl, list(range(heads)), dr.MaskParams(head_fuse=0), "cuda:0", wl.Sb
    run.ctx = dr.Context(0)
    run.shape = dr.Shape(1, heads, wl.N, 64, frames, hg, wg, 32, 0, 0, wl.N * 64 * heads, wl.N * 64, 64)
    one = torch.randn(1, 1, wl.Sb, wl.Sb, generator=torch.Generator().manual_seed(heads))
    rowptr, colidx, nnz, _ = run.build_mask(one.cuda().expand(1, heads, -1, -1).contiguous(), mode, par)
    if mode == "static":
        assert_masks_equal(rowptr[:, :1], colidx[:, :1], nnz[:, :1],
                           oracle_masks_from(one, oracle_class_map(wl), mode, par))
    total = int(nnz[0, 0])
    assert total == int(rowptr[0, 0, -1]) and bool((nnz == total).all())
    assert torch.equal(rowptr, rowptr[:, :1].expand_as(rowptr))
    assert torch.equal(colidx[:, :, :total], colidx[:, :1, :total].expand(1, heads, total))
