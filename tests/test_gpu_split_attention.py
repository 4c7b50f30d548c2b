"""Attention at fp32 accuracy (fp32 storage, and bf16 storage at d = 64): 32-bit operands as three bf16 parts on the
matrix cores, against the oracle on every row, at the edges of its tiles, streams and list windows."""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2604_20470_amd as dr
from oracle import dynamicrad_oracle as o
from workloads import tiny_case

from helpers import GpuRun, to_f64

pytestmark = pytest.mark.gpu

STORAGE = [("f32", 64), ("f32", 128), ("bf16", 64)]


def _run(dtype, d, bs, frames, hg, wg, scale=1.0):
    wl = dataclasses.replace(tiny_case("ragged128"), dtype=dtype, d=d, Bs=bs, Nf=frames, Hg=hg, Wg=wg, H=2, index=61)
    run = GpuRun(wl)
    if scale != 1.0:
        run.Qc = (run.Qc.float() * scale).to(run.Qc.dtype)
        run.Q = run.Qc.cuda()
    return run


def _csr(rows):
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])])
    return rp, np.asarray([c for r in rows for c in r] or [0], dtype=np.int64)


def _attend(run, rp, ci):
    rowptr = torch.from_numpy(rp.astype(np.int32)).view(1, 1, -1).contiguous().cuda()
    colidx = torch.from_numpy(ci.astype(np.int32)).view(1, 1, -1).contiguous().cuda()
    return run.attention(rowptr, colidx, colidx.shape[2], want_lse=True)


def _bounds(run, h):
    """Rounding bounds for O and the log-sum-exp: a logit is a sum of d products, each correct to 2^-23, accumulated in
    fp32; a relative change e of every probability moves O by at most 2 e max|V|; bf16 output rounds once more."""
    q, k, v = (np.abs(to_f64(t[0, h])) for t in (run.Qc, run.Kc, run.Vc))
    logit = 2.0 ** -22 * float((q @ k.T).max()) / np.sqrt(q.shape[1])
    out = v.max() * (2.0 * logit + 2.0 ** -20)
    return out + (v.max() * 2.0 ** -8 if run.wl.dtype == "bf16" else 0.0), logit + 2.0 ** -20


def _check(run, rp, ci, O, lse):
    for h in range(run.wl.H):
        want, want_lse = o.masked_attention(to_f64(run.Qc[0, h]), to_f64(run.Kc[0, h]), to_f64(run.Vc[0, h]), rp, ci,
                                            run.wl.Bs, return_lse=True)
        tol, tol_lse = _bounds(run, h)
        for qb, blk in want.items():
            rows = slice(qb * run.wl.Bs, qb * run.wl.Bs + blk.shape[0])
            assert np.abs(to_f64(O[0, h, rows]) - blk).max() <= tol, (h, qb, tol)
            g, w = lse[0, h, rows].cpu().numpy().astype(np.float64), want_lse[qb]
            with np.errstate(invalid="ignore"):
                close = np.abs(g - w) <= tol_lse + 2.0 ** -23 * np.abs(w)
            assert (close | (np.isinf(g) & np.isinf(w) & (g < 0) & (w < 0))).all(), (h, qb)


@pytest.mark.parametrize("dtype,d", STORAGE)
@pytest.mark.parametrize("bs", [32, 64, 128])
@pytest.mark.parametrize("frames,hg,wg,scale", [
    (7, 9, 21, 1.0),        # N = 1323: a partial last block and a partial last tile at every block size
    (3, 5, 11, 8.0),        # N = 165; large logits: the exponent reference moves
    (7, 16, 24, 1.0),       # N = 2688 = 84 * 32: full lists outgrow the register window at block size 32
    (1, 3, 7, 1.0),         # N = 21: one tile, and not a full one
])
def test_random_lists_against_the_oracle(dtype, d, bs, frames, hg, wg, scale):
    run = _run(dtype, d, bs, frames, hg, wg, scale)
    Sb = run.wl.Sb
    rng = np.random.default_rng(frames * 100 + bs)
    rows = [sorted(np.nonzero(rng.random(Sb) < 0.4)[0].tolist()) for _ in range(Sb)]
    rows[-1] = list(range(Sb))
    if Sb > 3:
        rows[0], rows[1], rows[2] = [], [Sb - 1], list(range(Sb))[::-1]     # nothing; the partial block alone; not ascending
    rp, ci = _csr(rows)
    _check(run, rp, ci, *_attend(run, rp, ci))


@pytest.mark.parametrize("dtype,d", STORAGE)
@pytest.mark.parametrize("bs", [32, 64, 128])
def test_infinite_inputs_give_what_fp32_arithmetic_gives(dtype, d, bs):
    run = _run(dtype, d, bs, 5, 9, 13)                       # N = 585
    Sb = run.wl.Sb
    rp, ci = _csr([list(range(Sb))] * Sb)
    run.Qc[..., 3] = run.Qc[..., 3].abs() + 0.5
    run.Kc[:, 0, 40] = 0.0                                   # head 0: a key whose logit is -inf in every row
    run.Vc[:, 1, 70, 5] = float("inf")                       # head 1: one infinite value
    clean = {n: getattr(run, n).clone() for n in ("Qc", "Kc", "Vc")}
    run.Kc[:, 0, 40, 3] = -float("inf")
    clean["Kc"][:, 0, 40, 3] = -1e4                          # the same key out of reach by a finite logit
    clean["Vc"][:, 1, 70, 5] = 0.0
    run.Q, run.K, run.V = run.Qc.cuda(), run.Kc.cuda(), run.Vc.cuda()
    O, lse = _attend(run, rp, ci)
    assert torch.isposinf(O[0, 1, :, 5].float()).all()
    O[0, 1, :, 5] = 0.0
    run.Qc, run.Kc, run.Vc = clean["Qc"], clean["Kc"], clean["Vc"]
    bounds = _bounds(run, 1)                                  # (head 0 holds the large stand-in key)
    for h in range(2):
        want, want_lse = o.masked_attention(to_f64(run.Qc[0, h]), to_f64(run.Kc[0, h]), to_f64(run.Vc[0, h]), rp, ci, bs,
                                            return_lse=True)
        for qb, blk in want.items():
            if h == 1:
                blk[:, 5] = 0.0
            rows = slice(qb * bs, qb * bs + blk.shape[0])
            assert np.abs(to_f64(O[0, h, rows]) - blk).max() <= bounds[0] * 4, (h, qb)
            assert np.abs(lse[0, h, rows].cpu().numpy() - want_lse[qb]).max() <= bounds[1] * 4 + 1e-5, (h, qb)


@pytest.mark.parametrize("dtype,d", STORAGE)
def test_lists_longer_than_every_streams_window(dtype, d):
    """Block size 32: a stream of eight (four) sees every eighth (fourth) entry through a window of 64 of its own."""
    wl = dataclasses.replace(tiny_case("ragged128"), dtype=dtype, d=d, Bs=32, Nf=19, Hg=27, Wg=33, H=1, index=62)
    run = GpuRun(wl)
    Sb = wl.Sb                                               # N = 16929: 530 blocks, the last of one key
    assert Sb > 8 * 64
    rows = [[] for _ in range(Sb)]
    rows[0] = rows[5] = rows[Sb - 1] = list(range(Sb))
    rows[7] = list(range(0, Sb, 2))
    rp, ci = _csr(rows)
    _check(run, rp, ci, *_attend(run, rp, ci))


@pytest.mark.parametrize("dtype,d", STORAGE)
@pytest.mark.parametrize("bs", [64, 128])
def test_lists_around_the_window_of_64_entries(dtype, d, bs):
    """Block sizes 128 and 64: the list is held 64 entries at a time, and the loop of d = 128, block size 128 asks for entries four
    tiles ahead, past the list's end too.  Rows on both sides of one, two and (block size 64) four windows, that end with the
    partial last block and that do not, between rows that list nothing; the first and the last row are full."""
    frames, hg, wg = 13, 31, 41                              # N = 16523: the last block has 11 keys at either block size
    wl = dataclasses.replace(tiny_case("ragged128"), dtype=dtype, d=d, Bs=bs, Nf=frames, Hg=hg, Wg=wg, H=1, index=65)
    run = GpuRun(wl)
    Sb = wl.Sb
    assert Sb >= 130 and wl.N % bs == 11
    rng = np.random.default_rng(bs + d)
    rows = [[] for _ in range(Sb)]
    rows[0] = rows[Sb - 1] = list(range(Sb))
    for at, n in enumerate(n for n in (1, 2, 63, 64, 65, 66, 67, 68, 69, 127, 128, 129, 191, 192, 193, 256, 257) if n < Sb):
        rows[2 + 3 * at] = sorted(rng.choice(Sb - 1, n, replace=False).tolist())
        rows[3 + 3 * at] = sorted(rng.choice(Sb - 1, n - 1, replace=False).tolist()) + [Sb - 1]
    rp, ci = _csr(rows)
    _check(run, rp, ci, *_attend(run, rp, ci))


@pytest.mark.parametrize("dtype,d", STORAGE)
@pytest.mark.parametrize("bs", [64, 128])
@pytest.mark.parametrize("hidden", [32, 33])
def test_a_row_that_starts_with_a_whole_tile_of_minus_infinity(dtype, d, bs, hidden):
    """The first tile of a row (32 keys), and a key of the next, are out of reach by a logit of -inf: weight 0."""
    run = _run(dtype, d, bs, 5, 9, 13)                       # N = 585
    Sb = run.wl.Sb
    rp, ci = _csr([list(range(Sb))] * Sb)
    run.Qc[..., 3] = run.Qc[..., 3].abs() + 0.5
    run.Kc[:, :, :hidden] = 0.0
    run.Kc[:, :, :hidden, 3] = -float("inf")
    run.Q, run.K, run.V = run.Qc.cuda(), run.Kc.cuda(), run.Vc.cuda()
    O, lse = _attend(run, rp, ci)
    run.Kc[:, :, :hidden, 3] = -1e4                          # the same by a finite logit (its weight underflows in 64 bits too)
    for h in range(2):
        want, want_lse = o.masked_attention(to_f64(run.Qc[0, h]), to_f64(run.Kc[0, h]), to_f64(run.Vc[0, h]), rp, ci, bs,
                                            return_lse=True)
        finite = run.Kc.clone()
        finite[:, :, :hidden] = 0.0                          # (the bounds: of the keys that carry weight)
        q, k, v = (np.abs(to_f64(t[0, h])) for t in (run.Qc, finite, run.Vc))
        logit = 2.0 ** -22 * float((q @ k.T).max()) / np.sqrt(d)
        tol = v.max() * (2.0 * logit + 2.0 ** -20) + (v.max() * 2.0 ** -8 if dtype == "bf16" else 0.0)
        for qb, blk in want.items():
            rows = slice(qb * bs, qb * bs + blk.shape[0])
            assert np.abs(to_f64(O[0, h, rows]) - blk).max() <= tol, (h, qb)
            assert np.abs(lse[0, h, rows].cpu().numpy() - want_lse[qb]).max() <= logit + 2.0 ** -20 + 2.0 ** -23 * 16, (h, qb)


@pytest.mark.parametrize("dtype,d", STORAGE)
@pytest.mark.parametrize("bs", [32, 64, 128])
def test_output_over_q_for_every_input(dtype, d, bs):
    """A query block reads only its own rows of Q, also when infinities send it to the plain pass: O may overlay Q."""
    run = _run(dtype, d, bs, 5, 9, 13)                       # N = 585
    Sb = run.wl.Sb
    rows = [list(range(Sb))] * Sb
    rows[1] = list(range(2, Sb))                             # not the key block of the infinity at any block size: stays finite
    rp, ci = _csr(rows)
    run.Vc[:, :, 20, 5] = float("inf")
    run.V = run.Vc.cuda()
    want, want_lse = _attend(run, rp, ci)
    rowptr, colidx = (torch.from_numpy(x.astype(np.int32)).view(1, 1, -1).contiguous().cuda() for x in (rp, ci))
    O, lse = run.Q.clone(), torch.empty_like(want_lse)
    dr.dr_sparse_attn_fwd(run.ctx, run.shape, O, run.K, run.V, rowptr, colidx, 1, colidx.shape[2], O, lse)
    torch.cuda.synchronize()
    assert torch.isposinf(want[:, :, :bs, 5].float()).all() and torch.isfinite(want[:, :, bs:2 * bs].float()).all()
    assert torch.equal(O.view(torch.uint8), want.view(torch.uint8)) and torch.equal(lse, want_lse)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("bs", [32, 64, 128])
@pytest.mark.parametrize("q_by,k_by", [
    (1e-36, 1e36),      # ordinary logits of factors whose third part lies below bf16's range
    (1e36, 1e-36),
    (1e-36, 1.0),       # tiny queries alone: every logit is 0 to any accuracy
])
def test_fp32_accuracy_of_logits_at_the_ends_of_the_range(d, bs, q_by, k_by):
    """Errors relative to the results, as near 1; a few zeros, which say nothing about the range, stand among the values."""
    run = _run("f32", d, bs, 5, 9, 13)                       # N = 585
    Sb = run.wl.Sb
    rp, ci = _csr([list(range(Sb))] * Sb)
    for name, by in (("Qc", q_by), ("Kc", k_by)):
        t = getattr(run, name)
        t[:, :, ::17, 3] = 0.0
        setattr(run, name, (t.double() * by).float())
    run.Q, run.K = run.Qc.cuda(), run.Kc.cuda()
    _check(run, rp, ci, *_attend(run, rp, ci))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("bs", [32, 64, 128])
@pytest.mark.parametrize("v_by", [1e-30, 1e-35, 1e-37])
def test_fp32_values_whose_parts_end_below_the_range(d, bs, v_by):
    """Every key of a head carries the same value row, so the result is that row however the weights round: a value held in
    fewer bits shows as it is (1e-37: 4.5e-4 of it at bf16's last place) instead of averaging out."""
    run = _run("f32", d, bs, 5, 9, 13)                       # N = 585
    Sb = run.wl.Sb
    rp, ci = _csr([list(range(Sb))] * Sb)
    row = (run.Vc[:, :, :1].sign() * (run.Vc[:, :, :1].abs() + 0.5)).double() * v_by
    run.Vc = row.float().expand_as(run.Vc).contiguous()
    run.V = run.Vc.cuda()
    O, _ = _attend(run, rp, ci)
    # numerator and normaliser: chains of at most 585 additions of terms of one sign, each within 2^-24 of the running sum
    assert ((O.cpu().double() - run.Vc.double()).abs() <= 2 * run.wl.N * 2.0 ** -24 * run.Vc.double().abs()).all()


@pytest.mark.parametrize("bs", [32, 64, 128])
def test_bf16_rows_too_far_apart_for_the_matrix_kernels(bs):
    """bf16 at d = 128 with a token stride of 2^24 elements, beyond the 32-bit offsets of the kernels that serve it otherwise."""
    run = _run("bf16", 128, bs, 2, 5, 7)                     # N = 70
    N, far = run.wl.N, 1 << 24
    Sb = run.wl.Sb
    rp, ci = _csr([list(range(Sb))] * Sb)
    wide = torch.zeros(N, far, dtype=torch.bfloat16, device="cuda")
    views = [wide.as_strided((1, 2, N, 128), (1024, 512, far, 1), 128 * i) for i in range(4)]      # Q, K, V, O of both heads
    for view, t in zip(views, (run.Q, run.K, run.V)):
        view.copy_(t)
    run.shape.stride_b, run.shape.stride_h, run.shape.stride_n = 1024, 512, far
    rowptr, colidx = (torch.from_numpy(x.astype(np.int32)).view(1, 1, -1).contiguous().cuda() for x in (rp, ci))
    lse = torch.empty(1, 2, N, dtype=torch.float32, device="cuda")
    dr.dr_sparse_attn_fwd(run.ctx, run.shape, *views[:3], rowptr, colidx, 1, colidx.shape[2], views[3], lse)
    torch.cuda.synchronize()
    _check(run, rp, ci, views[3].contiguous(), lse)
