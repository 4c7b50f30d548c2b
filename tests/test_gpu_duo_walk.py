"""Block size 64 with one mask per head: the kernel of two wavefronts per workgroup, with the bits that the kernel of four
gives for the same head and mask (they take a row's chunks in the same order), and against the oracle."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import dynamicrad_oracle as o
from workloads import tiny_case

from helpers import GpuRun, to_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,frames,hg,wg", [
    (1, 3, 7, 9, 21),       # N = 1323: the last block of 43 keys, 21 blocks: a last group of one row
    (2, 2, 8, 10, 17),      # N = 1360: the last block of 16 keys
    (1, 2, 10, 8, 16),      # N = 1280: every block full
    (1, 2, 2, 7, 5),        # N = 70: two blocks, one group
    (1, 24, 23, 16, 24),    # N = 8832: 1656 groups, more than two per compute unit; lists beyond a register window
])
def test_bits_of_the_four_wavefront_kernel(B, H, frames, hg, wg):
    wl = dataclasses.replace(tiny_case("ragged128"), B=B, H=H, Nf=frames, Hg=hg, Wg=wg, Bs=64, index=111)
    run = GpuRun(wl, threads=8)
    Sb = wl.Sb
    rng = np.random.default_rng(Sb)
    keep = rng.random((B, H, Sb, Sb)) < 0.55
    keep[:, :, 0] = False                                    # an empty row, a full one beside it, an empty pair
    if Sb > 4:
        keep[:, :, 1] = True
        keep[:, :, 2:4] = False
    rp = np.concatenate([np.zeros((B, H, 1), dtype=np.int64), keep.sum(-1).cumsum(-1)], -1)
    cap = int(rp[..., -1].max())
    ci = np.zeros((B, H, cap), dtype=np.int64)
    for b in range(B):
        for h in range(H):
            ci[b, h, :rp[b, h, -1]] = np.nonzero(keep[b, h])[1]
    rowptr, colidx = (torch.from_numpy(x.astype(np.int32)).cuda() for x in (rp, ci))
    run.Q[0, 0, :20] *= 14                                   # rows for the second pass
    O, lse = run.attention(rowptr, colidx, cap, want_lse=True)
    alone = GpuRun(dataclasses.replace(wl, B=1, H=1))
    alone.shape.stride_b = alone.shape.stride_h
    for b in range(B):
        for h in range(H):
            alone.Q, alone.K, alone.V = (t[b:b + 1, h:h + 1].contiguous() for t in (run.Q, run.K, run.V))
            Oa, la = alone.attention(rowptr[b:b + 1, h:h + 1].contiguous(), colidx[b:b + 1, h:h + 1].contiguous(), cap, want_lse=True)
            assert torch.equal(Oa[0, 0], O[b, h]) and torch.equal(la[0, 0], lse[b, h]), (b, h)
    q, k, v = (to_f64(t[0, 0]) for t in (run.Q, run.K, run.V))
    want = o.masked_attention(q, k, v, rp[0, 0], ci[0, 0], 64)
    for qb, blk in want.items():
        assert np.abs(to_f64(O[0, 0, qb * 64: qb * 64 + blk.shape[0]]) - blk).max() <= 2e-2, qb
