"""The fp32-accuracy kernel in launches that do not fill the chip or end in a round that does not (one workgroup walks a query
block's whole list there too): rows of very different lengths (none, one, three), a partial last block, infinities, O over Q, and
the entry point with static scratch bit for bit."""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2604_20470_amd as dr
from oracle import dynamicrad_oracle as o
from workloads import tiny_case

from helpers import GpuRun, to_f64

pytestmark = pytest.mark.gpu


def _launch(run, rowptr, colidx, fn, O=None, lse=True):
    O = torch.full_like(run.Q, float("nan")) if O is None else O
    out = torch.full(run.Q.shape[:3], float("nan"), dtype=torch.float32, device="cuda") if lse else None
    fn(run.ctx, run.shape, run.Q, run.K, run.V, rowptr, colidx, 1, colidx.shape[2], O, out)
    torch.cuda.synchronize()
    return O, out


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 64)])
@pytest.mark.parametrize("bs", [64, 128])
@pytest.mark.parametrize("frames,hg,wg,heads", [
    (9, 17, 19, 1),        # N = 2907: a few blocks, many pieces
    (9, 17, 19, 5),
    (17, 19, 21, 2),       # N = 6783: up to a round and a half
    (11, 24, 32, 6),       # N = 8448
])
def test_shared_lists_against_the_oracle(dtype, d, bs, frames, hg, wg, heads):
    wl = dataclasses.replace(tiny_case("ragged128"), dtype=dtype, d=d, Bs=bs, Nf=frames, Hg=hg, Wg=wg, H=heads, index=63)
    run = GpuRun(wl)
    N, Sb = wl.N, wl.Sb
    rng = np.random.default_rng(N + bs + heads)
    rows = [sorted(np.nonzero(rng.random(Sb) < 0.6)[0].tolist()) for _ in range(Sb)]
    rows[0], rows[1], rows[2], rows[Sb - 1] = [], [Sb - 1], [3, 5, 7], list(range(Sb))
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])])
    ci = np.asarray([c for r in rows for c in r])
    rowptr, colidx = (torch.from_numpy(x.astype(np.int32)).view(1, 1, -1).contiguous().cuda() for x in (rp, ci))
    O, lse = _launch(run, rowptr, colidx, dr.dr_sparse_attn_fwd)
    for other in (_launch(run, rowptr, colidx, dr.dr_sparse_attn_fwd_static), _launch(run, rowptr, colidx, dr.dr_sparse_attn_fwd)):
        assert torch.equal(O.view(torch.uint8), other[0].view(torch.uint8)) and torch.equal(lse, other[1])
    assert torch.equal(_launch(run, rowptr, colidx, dr.dr_sparse_attn_fwd, lse=False)[0].view(torch.uint8), O.view(torch.uint8))
    if dtype == "f32":                       # (blocks that share Q with O: nothing of Q is read after O is written)
        over = run.Q.clone()
        keep, run.Q = run.Q, over
        assert torch.equal(_launch(run, rowptr, colidx, dr.dr_sparse_attn_fwd, O=over)[0], O)
        run.Q = keep
    h = heads - 1
    q, k, v = (to_f64(t[0, h]) for t in (run.Qc, run.Kc, run.Vc))
    qb_seen = sorted({0, 1, 2, 3, Sb // 2, Sb - 2, Sb - 1})
    want, want_lse = o.masked_attention(q, k, v, rp, ci, bs, rows=qb_seen, return_lse=True)
    # a logit is good to 2^-22 of its terms' magnitudes, a probability to twice that and 2^-20 for exponentials and sums
    logit = 2.0 ** -22 * float((np.abs(q[::7]) @ np.abs(k).T).max()) * 1.5 / np.sqrt(d)
    tol = np.abs(v).max() * (2.0 * logit + 2.0 ** -20) + (np.abs(v).max() * 2.0 ** -8 if dtype == "bf16" else 0.0)
    for qb in qb_seen:
        blk, span = want[qb], slice(qb * bs, qb * bs + want[qb].shape[0])
        assert np.abs(to_f64(O[0, h, span]) - blk).max() <= tol, qb
        got = lse[0, h, span].cpu().numpy()
        if rows[qb]:
            assert np.abs(got - want_lse[qb]).max() <= logit + 2.0 ** -20 + 2.0 ** -23 * 16, qb
        else:
            assert np.isneginf(got).all() and (to_f64(O[0, h, span]) == 0).all()


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 64)])
@pytest.mark.parametrize("bs", [64, 128])
def test_infinities_in_a_shared_block_go_the_plain_way(dtype, d, bs):
    wl = dataclasses.replace(tiny_case("ragged128"), dtype=dtype, d=d, Bs=bs, Nf=9, Hg=17, Wg=19, H=1, index=64)
    run = GpuRun(wl)
    Sb = wl.Sb
    rp, ci = np.arange(Sb + 1) * Sb, np.tile(np.arange(Sb), Sb)
    rowptr, colidx = (torch.from_numpy(x.astype(np.int32)).view(1, 1, -1).contiguous().cuda() for x in (rp, ci))
    clean, _ = _launch(run, rowptr, colidx, dr.dr_sparse_attn_fwd)
    run.V[0, 0, 70, 5] = float("inf")
    O, lse = _launch(run, rowptr, colidx, dr.dr_sparse_attn_fwd)
    assert torch.isposinf(O[0, 0, :, 5].float()).all() and torch.isfinite(lse).all()
    O[..., 5] = clean[..., 5]
    scale = float(run.V[torch.isfinite(run.V)].abs().max())
    assert float((O.float() - clean.float()).abs().max()) <= scale * (2.0 ** -8 if dtype == "bf16" else 2.0 ** -16)
    if dtype == "f32":                       # queries beyond the range of three parts, flagged by every piece
        run.V[0, 0, 70, 5] = 0.0
        run.Q[0, 0, 5] = 0.0
        run.Q[0, 0, 5, 0] = 2.0 ** 101
        run.K[..., 0] = 0.0
        O, lse = _launch(run, rowptr, colidx, dr.dr_sparse_attn_fwd)
        mean = run.V[0, 0].double().mean(0)
        assert float((O[0, 0, 5].double() - mean).abs().max()) <= scale * 2.0 ** -16
