"""The 256-query kernel on launches with more items than compute units: every item is taken once, whichever workgroup
draws it, with the bits that a launch of its head alone gives (few items: no queue is drawn from)."""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2604_20470_amd as dr
from oracle import dynamicrad_oracle as o
from workloads import tiny_case

from helpers import GpuRun, to_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,bs,frames,hg,wg", [
    (40, 128, 9, 16, 23),       # N = 3312: 13 items per head, 65 per queue
    (30, 32, 9, 16, 23),        # 390 items: a queue ends inside a head
    (9, 64, 33, 16, 21),        # N = 11088: 396 items, the last queue is shorter
])
def test_every_item_once(H, bs, frames, hg, wg):
    wl = dataclasses.replace(tiny_case("ragged128"), Nf=frames, Hg=hg, Wg=wg, H=H, Bs=bs, index=81)
    run = GpuRun(wl, threads=8)
    Sb = wl.Sb
    assert -(-wl.N // 256) * H > 256
    rng = np.random.default_rng(H)
    rows = [np.nonzero(rng.random(Sb) < 0.1)[0].tolist() for _ in range(Sb)]
    per = 256 // bs
    for qb in range(Sb):                                     # whole items without a key block, in a row and alone
        if qb // per in (1, 2, 3, 7):
            rows[qb] = []
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])])
    ci = np.asarray([c for r in rows for c in r], dtype=np.int64)
    rowptr = torch.from_numpy(rp.astype(np.int32)).view(1, 1, -1).cuda()
    colidx = torch.from_numpy(ci.astype(np.int32)).view(1, 1, -1).cuda()
    O = run.attention(rowptr, colidx, colidx.shape[2])
    assert torch.equal(O, run.attention(rowptr, colidx, colidx.shape[2]))
    alone = GpuRun(dataclasses.replace(wl, H=1))
    for h in range(H):
        alone.Q, alone.K, alone.V = (t[:, h:h + 1].contiguous() for t in (run.Q, run.K, run.V))
        alone.shape.stride_b = alone.Q.stride(0)
        assert torch.equal(alone.attention(rowptr, colidx, colidx.shape[2])[0, 0], O[0, h]), h
    for h in (0, H - 1):
        want = o.masked_attention(to_f64(run.Qc[0, h]), to_f64(run.Kc[0, h]), to_f64(run.Vc[0, h]), rp, ci, bs)
        for qb, blk in want.items():
            assert np.abs(to_f64(O[0, h, qb * bs: qb * bs + blk.shape[0]]) - blk).max() <= 2e-2, (h, qb)


@pytest.mark.parametrize("bs", [128, 64, 32])
def test_every_item_once_with_batches_and_masks_of_their_own(bs):
    """312 items of 256 queries (at block size 64 between one and two rounds: four wavefronts, not two), B = 2, one mask per
    head: the drawn item's batch, head and list, from the context's queue and from the static area's, twice."""
    B, H = 2, 12
    wl = dataclasses.replace(tiny_case("ragged128"), B=B, H=H, Nf=9, Hg=16, Wg=23, Bs=bs, index=82)      # N = 3312
    run = GpuRun(wl, threads=8)
    Sb = wl.Sb
    assert 256 < -(-wl.N // 256) * H * B <= 512
    keep = np.random.default_rng(bs).random((B, H, Sb, Sb)) < 0.15
    keep[:, :, 3] = False
    rp = np.concatenate([np.zeros((B, H, 1), dtype=np.int64), keep.sum(-1).cumsum(-1)], -1)
    cap = int(rp[..., -1].max())
    ci = np.zeros((B, H, cap), dtype=np.int64)
    for b in range(B):
        for h in range(H):
            ci[b, h, :rp[b, h, -1]] = np.nonzero(keep[b, h])[1]
    rowptr, colidx = (torch.from_numpy(x.astype(np.int32)).cuda() for x in (rp, ci))
    O, lse = run.attention(rowptr, colidx, cap, want_lse=True)
    for _ in range(2):
        Os, ls = torch.full_like(O, float("nan")), torch.full_like(lse, float("nan"))
        dr.dr_sparse_attn_fwd_static(run.ctx, run.shape, run.Q, run.K, run.V, rowptr, colidx, H, cap, Os, ls)
        torch.cuda.synchronize()
        assert torch.equal(Os, O) and torch.equal(ls, lse)
    alone = GpuRun(dataclasses.replace(wl, B=1, H=1))
    alone.shape.stride_b = alone.shape.stride_h
    for b in range(B):
        for h in range(H):
            alone.Q, alone.K, alone.V = (t[b:b + 1, h:h + 1].contiguous() for t in (run.Q, run.K, run.V))
            Oa, la = alone.attention(rowptr[b:b + 1, h:h + 1].contiguous(), colidx[b:b + 1, h:h + 1].contiguous(), cap, want_lse=True)
            assert torch.equal(Oa[0, 0], O[b, h]) and torch.equal(la[0, 0], lse[b, h]), (b, h)
    want = o.masked_attention(to_f64(run.Q[1, H - 1]), to_f64(run.K[1, H - 1]), to_f64(run.V[1, H - 1]), rp[1, H - 1], ci[1, H - 1], bs)
    for qb, blk in want.items():
        assert np.abs(to_f64(O[1, H - 1, qb * bs: qb * bs + blk.shape[0]]) - blk).max() <= 2e-2, qb
