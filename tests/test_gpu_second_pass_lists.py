"""The lists of flagged query blocks: blocks that one or both wavefronts flag, odd block counts (a pair without its second block), two
batches, fewer pairs than queues, and more flagged blocks than workgroups of the second pass.  Every flagged block has the bits of
the kernel that takes one query block per workgroup, whose second pass looks at flag words; call after call, from either scratch."""
import dataclasses
import os

import numpy as np
import pytest
import torch

import paper_2604_20470_amd as dr
from workloads import tiny_case

from helpers import GpuRun

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,frames,share", [(1, 1, 3, 1.0), (2, 3, 5, 0.5), (1, 5, 9, 0.4), (2, 40, 11, 1.0), (2, 40, 11, 0.1)])
def test_listed_blocks_have_the_bits_of_the_flag_words_pass(B, H, frames, share):
    wl = dataclasses.replace(tiny_case("ragged128"), Nf=frames, Hg=9, Wg=15, B=B, H=H, index=73)      # 135 tokens a frame
    run = GpuRun(wl, threads=8)
    Sb, N = wl.Sb, wl.N
    halves = np.random.default_rng(frames).random((B, H, 2 * Sb)) < share            # of 64 queries: a wavefront's
    hot = torch.from_numpy(halves).repeat_interleave(64, 2)[:, :, :N].cuda()
    Q = torch.where(hot[..., None], run.Q.float() * 14, run.Q.float()).bfloat16()
    rowptr = (torch.arange(Sb + 1, dtype=torch.int32) * Sb).repeat(B, 1, 1).cuda()
    colidx = torch.arange(Sb, dtype=torch.int32).repeat(B, 1, Sb).cuda()
    cap = colidx.shape[2]

    def attend(ctx, entry=dr.dr_sparse_attn_fwd):
        O, lse = torch.full_like(Q, 7.0), torch.zeros(B, H, N, device="cuda")
        entry(ctx, run.shape, Q, run.K, run.V, rowptr, colidx, 1, cap, O, lse)
        return O, lse

    os.environ["DR_ATTN_PAIRS"] = "0"
    try:
        words = dr.Context(0)
    finally:
        del os.environ["DR_ATTN_PAIRS"]
    want_O, want_lse = attend(words)
    flagged = torch.nn.functional.pad(want_lse.abs() > 45.0, (0, Sb * 128 - N)).view(B, H, Sb, 128).any(-1)
    assert int(flagged.sum()) >= share * 0.5 * B * H * Sb
    rows = flagged.repeat_interleave(128, 2)[:, :, :N]
    ctx = dr.Context(0)
    for entry in (dr.dr_sparse_attn_fwd, dr.dr_sparse_attn_fwd, dr.dr_sparse_attn_fwd_static):
        O, lse = attend(ctx, entry)
        assert torch.equal(O[rows], want_O[rows]) and torch.equal(lse[rows], want_lse[rows])
        assert (O.float() - want_O.float()).abs().max() < 4e-2
