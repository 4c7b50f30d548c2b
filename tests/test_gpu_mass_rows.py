"""The cumulative-mass rule for rows of at most 1024 key blocks: the crossing found with fixed-point masses and bins, and the
literal chain where the target lies too close to it, bit for bit against the oracle."""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2604_20470_amd as dr
from workloads import tiny_case

from helpers import GpuRun, assert_masks_equal, oracle_class_map, oracle_masks_from

pytestmark = pytest.mark.gpu


# rows on both sides of every register width, with one row per workgroup (one mask) and four (thirty)
@pytest.mark.parametrize("frames,hg,wg", [(8, 8, 16), (16, 10, 25), (15, 16, 30), (32, 20, 23), (40, 20, 25), (33, 31, 32)])
@pytest.mark.parametrize("heads", [1, 30])
def test_prefix_bit_exact(frames, hg, wg, heads):
    wl = dataclasses.replace(tiny_case("tiny8"), Nf=frames, Hg=hg, Wg=wg, H=heads, index=101)
    params = dr.MaskParams(head_fuse=0, gamma=3.0)
    run = GpuRun.__new__(GpuRun)
    run.wl, run.heads, run.params, run.device, run.Sb = wl, list(range(heads)), params, "cuda:0", wl.Sb
    run.ctx = dr.Context(0)
    run.shape = dr.Shape(1, heads, wl.N, 64, frames, hg, wg, wl.Bs, 0, 0, wl.N * 64 * heads, wl.N * 64, 64)
    assert wl.Sb <= 1024
    g = torch.Generator().manual_seed(frames)
    scores = torch.randn(1, heads, wl.Sb, wl.Sb, generator=g)
    scores[:, 0, 1::7] = 0.25                                     # all equal: the sum hits tau * n exactly for some tau
    scores[:, 0, 2::7] *= 40.0                                    # one key holds nearly everything
    scores[:, 0, 3::7] = (scores[:, 0, 3::7] * 2).round()         # many ties, signed zeros
    scores[:, 0, 4::7] *= 1e30                                    # masses of 0 and 1 only
    scores = scores.cuda()
    cls = oracle_class_map(wl, gamma=3.0)
    for tau in (0.5, 0.9, 0.99, 1.0, 1e-9):
        rowptr, colidx, nnz, cap = run.build_mask(scores, "dynamic", tau)
        few = [0] if heads == 1 else [0, heads - 1]
        want = oracle_masks_from(scores[:, few], cls, "dynamic", tau)
        assert_masks_equal(rowptr[:, few], colidx[:, few], nnz[:, few], want)


@pytest.mark.parametrize("bits", [0x7f800000, 0xff800000, 0x7fc00000, 0xffc00000])      # infinities and NaN of both signs
@pytest.mark.parametrize("tau", [0.3, 1.0])
def test_scores_that_are_not_finite_take_the_chain(bits, tau):
    """Beyond the contract, but defined by the rule as written: where the whole sum is not a number no prefix reaches its
    share and the row keeps every block; a mass of exp(-inf) = 0 is left out of a prefix that ends before it."""
    wl = dataclasses.replace(tiny_case("tiny8"), Nf=8, Hg=10, Wg=17, Bs=32, H=1, index=102)
    run = GpuRun.__new__(GpuRun)
    run.wl, run.heads, run.params, run.device, run.Sb = wl, [0], dr.MaskParams(head_fuse=0, gamma=3.0), "cuda:0", wl.Sb
    run.ctx = dr.Context(0)
    run.shape = dr.Shape(1, 1, wl.N, 64, 8, 10, 17, 32, 0, 0, wl.N * 64, wl.N * 64, 64)
    scores = torch.randn(1, 1, wl.Sb, wl.Sb, generator=torch.Generator().manual_seed(7))
    special = torch.zeros(wl.Sb, dtype=torch.bool)
    special[::5] = True
    scores.view(torch.int32)[..., special] = bits - (1 << 32) if bits >> 31 else bits
    rowptr, colidx, _, _ = run.build_mask(scores.cuda(), "dynamic", tau)
    rp, ci, cls = rowptr[0, 0].cpu().numpy(), colidx[0, 0].cpu().numpy(), oracle_class_map(wl, gamma=3.0)
    for qb in range(wl.Sb):
        free = np.nonzero((cls[qb] == 1) | (cls[qb] == 2))[0]
        forced = np.nonzero(cls[qb] == 3)[0]
        kept = free
        if bits == 0xff800000 or not special.numpy()[free].any():
            s = scores[0, 0, qb].numpy()[free].astype(np.float64)
            order = np.lexsort((free, -s))
            run_sum = np.add.accumulate(np.exp(s[order] - s.max())) if free.size else np.zeros(0)
            kept = free[order[:1 + int(np.argmax(run_sum >= tau * run_sum[-1]))]] if free.size else free
        assert np.array_equal(ci[rp[qb]:rp[qb + 1]], np.union1d(kept, forced)), qb


@pytest.mark.parametrize("frames,hg,wg", [(8, 8, 16), (15, 16, 30), (33, 31, 32)])
@pytest.mark.parametrize("heads", [1, 30])                    # bins that are binned again (few rows), and not
def test_crossing_among_many_keys_of_one_bin(frames, hg, wg, heads):
    wl = dataclasses.replace(tiny_case("tiny8"), Nf=frames, Hg=hg, Wg=wg, H=heads, index=103)
    run = GpuRun.__new__(GpuRun)
    run.wl, run.heads, run.params, run.device, run.Sb = wl, list(range(heads)), dr.MaskParams(head_fuse=0, gamma=3.0), "cuda:0", wl.Sb
    run.ctx = dr.Context(0)
    run.shape = dr.Shape(1, heads, wl.N, 64, frames, hg, wg, wl.Bs, 0, 0, wl.N * 64 * heads, wl.N * 64, 64)
    g = torch.Generator().manual_seed(frames)
    noise = torch.randn(1, 1, wl.Sb, wl.Sb, generator=g)
    scores = 2.0 + 1e-3 * noise                               # a cluster, which fills one bin
    scores[:, :, 0::5, ::17] = 2.5                            # beside a few ahead of it
    scores[:, :, 1::5] = (noise[:, :, 1::5] > 0.3).float()    # two values
    scores[:, :, 2::5, ::2] = 2.0 + 1e-6 * noise[:, :, 2::5, ::2]                     # a cluster in the cluster's bin
    scores[:, :, 3::5] = (noise[:, :, 3::5] * 64).round() / 64                        # groups of equal scores in every bin
    scores[:, :, 4::5, ::31] = -30.0                          # everything else in one bin
    scores = scores.expand(1, heads, -1, -1).contiguous()
    cls = oracle_class_map(wl, gamma=3.0)
    for tau in (0.1, 0.5, 0.9, 0.999):
        rowptr, colidx, nnz, _ = run.build_mask(scores.cuda(), "dynamic", tau)
        few = [0] if heads == 1 else [0, heads - 1]
        assert_masks_equal(rowptr[:, few], colidx[:, few], nnz[:, few], oracle_masks_from(scores[:, few], cls, "dynamic", tau))
