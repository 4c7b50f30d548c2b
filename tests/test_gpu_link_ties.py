"""The safeguard of a set in which nothing passes, where many columns share the highest score: the first in row-major order is kept,
and the call takes no longer for it than without ties (a program that sweeps thresholds reaches it with features that are
alike, such as a static background)."""
import numpy as np
import pytest
import torch

import paper_2604_20470_amd as dr

pytestmark = pytest.mark.gpu


def _scores(kind, N, Nt, g):
    u = torch.arange(N, device="cuda") % Nt
    if kind == "rows":                          # equal keys: a score depends on its row alone
        return torch.randn(N, 1, generator=g, device="cuda").expand(N, N)
    if kind == "late":                          # and the highest is the last row that a column sees
        return u.float()[:, None].expand(N, N)
    if kind == "columns":
        return torch.randn(1, N, generator=g, device="cuda").expand(N, N)
    if kind == "constant":
        return torch.zeros(N, N, device="cuda")
    if kind == "zeros":                         # of both signs
        return torch.where(torch.rand(N, N, generator=g, device="cuda") < 0.5, -0.0, 0.0)
    if kind == "few":
        return (torch.rand(N, N, generator=g, device="cuda") < 0.002).float()
    if kind == "mixed":                         # -inf and NaN alone, beside sets of numbers
        s = torch.randn(N, N, generator=g, device="cuda")
        s[:Nt] = torch.where(torch.rand(Nt, N, generator=g, device="cuda") < 0.5, float("nan"), -float("inf"))
        return s
    return torch.randn(N, N, generator=g, device="cuda")


def _call(frames, hg, wg, kind):
    Nt, N, bs = hg * wg, frames * hg * wg, 32
    s = _scores(kind, N, Nt, torch.Generator(device="cuda").manual_seed(N)).contiguous().view(1, 1, N, N)
    ctx, params = dr.Context(0), dr.MaskParams(gamma=1.0, head_fuse=1)
    shape = dr.Shape(1, 1, N, 64, frames, hg, wg, bs, 0, 0, N * 64, N * 64, 64)
    Sb = -(-N // bs)
    cap, _ = dr.dr_mask_capacity(ctx, shape, 1.0, params)
    rowptr = torch.zeros((1, 1, Sb + 1), dtype=torch.int32, device="cuda")
    colidx = torch.zeros((1, 1, cap), dtype=torch.int32, device="cuda")
    nnz = torch.zeros((1, 1), dtype=torch.int64, device="cuda")
    links = torch.full((1, 1, N, N), 9, dtype=torch.uint8, device="cuda")
    return s, links, lambda: dr.dr_build_mask_tokens(ctx, shape, float("inf"), 1.0, params, s, rowptr, colidx, cap, nnz, links)


@pytest.mark.parametrize("frames,hg,wg", [(4, 3, 43), (5, 16, 16), (4, 23, 31), (4, 32, 32)])
@pytest.mark.parametrize("kind", ["rows", "late", "columns", "constant", "zeros", "few", "mixed", "random"])
def test_first_of_the_best_is_kept(frames, hg, wg, kind):
    from oracle import dynamicrad_oracle as o
    Nt = hg * wg
    s, links, call = _call(frames, hg, wg, kind)
    call()
    tab = o.frame_table(frames, Nt, 32, 1.0, 1.0)
    u = torch.arange(Nt, device="cuda")
    for i in range(frames):
        for j in range(frames):
            t = abs(i - j)
            got = links[0, 0, i * Nt:(i + 1) * Nt, j * Nt:(j + 1) * Nt]
            if t <= 1 or not tab["retained"][t]:
                assert bool((got == (1 if t <= 1 else 0)).all())
                continue
            inside = (u[:, None] - u[None, :]).abs() <= int(tab["w"][t])
            tile = s[0, 0, i * Nt:(i + 1) * Nt, j * Nt:(j + 1) * Nt]
            ranked = tile[inside & ~tile.isnan()]
            first = int(((tile == ranked.max()) & inside).flatten().int().argmax())
            assert got.nonzero().tolist() == [list(divmod(first, Nt))], (i, j)


@pytest.mark.parametrize("frames,hg,wg", [(8, 32, 32), (4, 64, 64)])
def test_ties_cost_nothing(frames, hg, wg):
    def time(kind):
        _, _, call = _call(frames, hg, wg, kind)
        call()
        out = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(4):
                call()
            b.record()
            b.synchronize()
            out.append(a.elapsed_time(b))
        return float(np.median(out))
    base = time("random")
    for kind in ("rows", "late", "constant"):
        assert time(kind) <= 1.5 * base, kind
