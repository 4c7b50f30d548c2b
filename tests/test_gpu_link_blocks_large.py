"""Link bytes that go past the caches (from 140 million of them on) against the rule in fp64, and the masks against the density rule over those
bytes: columns that end inside a step, links that are and are not aligned to words, and rows that are no multiple of four (both of which
keep to the caches); sets of which nothing passes, whose highest score is kept."""
import pytest
import torch

import paper_2604_20470_amd as dr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("frames,hg,wg,masks,offset,tau", [
    (8, 37, 40, 1, 0, 0.4),       # 11 840: 140.2 million
    (8, 37, 40, 1, 1, 0.4),       # ... from an odd address
    (7, 1, 1693, 1, 0, 0.4),      # 11 851
    (4, 34, 50, 4, 0, 0.4),       # 6800 x 4 masks
    (4, 34, 50, 4, 0, -0.6),      # ... whose blocks are dense
    (8, 37, 40, 1, 0, 30.0),      # nothing passes
])
def test_links_past_the_caches_follow_the_rule(frames, hg, wg, masks, offset, tau):
    N, bs = frames * hg * wg, 128
    Sb = -(-N // bs)
    assert masks * N * N >= 140000000
    far = 0.9 if tau < 30.0 else 30.0
    params = dr.MaskParams(head_fuse=0, tau_far=far)
    g = torch.Generator(device="cuda").manual_seed(N)
    scores = torch.randn(1, masks, N, N, generator=g, device="cuda")
    shape = dr.Shape(1, masks, N, 64, frames, hg, wg, bs, 0, 0, N * 64 * masks, N * 64, 64)
    ctx = dr.Context(0)
    cap, _ = dr.dr_mask_capacity(ctx, shape, 1.0, params)
    rowptr = torch.zeros(1, masks, Sb + 1, dtype=torch.int32, device="cuda")
    colidx = torch.zeros(1, masks, cap, dtype=torch.int32, device="cuda")
    nnz = torch.zeros(1, masks, dtype=torch.int64, device="cuda")
    links = torch.full((masks * N * N + 8,), 9, dtype=torch.uint8, device="cuda")[offset:offset + masks * N * N].view(1, masks, N, N)
    dr.dr_build_mask_tokens(ctx, shape, tau, 1.0, params, scores, rowptr, colidx, cap, nnz, links)

    # frame pairs one by one, in fp64
    Nt = hg * wg
    u = torch.arange(Nt, device="cuda")
    L0 = 1 << (Nt - 1).bit_length()
    for m in range(masks):
        for i in range(frames):
            for j in range(frames):
                got = links[0, m, i * Nt:(i + 1) * Nt, j * Nt:(j + 1) * Nt]
                t = abs(i - j)
                if t <= 1:
                    assert bool((got == 1).all())
                    continue
                base = L0 / (1 << t.bit_length())
                w = max(int(base + 0.5), bs)
                sf = max(int(bs / (base + 1e-6)), 1)
                if t % sf:
                    assert not bool(got.any())
                    continue
                inside = (u[:, None] - u[None, :]).abs() <= w
                s = scores[0, m, i * Nt:(i + 1) * Nt, j * Nt:(j + 1) * Nt].double()
                n = int(inside.sum())
                mu = s[inside].sum() / n
                dev = ((s - mu) ** 2)[inside].sum() / n
                z = (s - mu) / (dev.sqrt() + 1e-6)
                own = tau if base >= bs else far
                want = inside & (z >= own)
                if not bool(want.any()):
                    want.view(-1)[s.masked_fill(~inside, -torch.inf).argmax()] = True
                sure = inside & ((z - own).abs() > 1e-9)          # (the sums' order may decide the others)
                assert torch.equal(got[sure].bool(), want[sure]) and not bool(got[~inside].any())

    # the density rule over the bytes: columns of which more than 15 % of a block's rows are links, and more than 60 % of its columns
    first = torch.arange(Sb, device="cuda") * bs
    last = (first + bs).clamp(max=N) - 1
    forced = torch.maximum(first[None, :] // Nt - last[:, None] // Nt, first[:, None] // Nt - last[None, :] // Nt) <= 1
    size = (last - first + 1).double()
    fill = (0, Sb * bs - N)
    for m in range(masks):
        keep = torch.zeros(Sb, Sb, dtype=torch.bool, device="cuda")
        for qb in range(Sb):
            column = links[0, m, first[qb]:last[qb] + 1].sum(0, dtype=torch.int32).double() / size[qb] > 0.15
            keep[qb] = torch.nn.functional.pad(column, fill).view(Sb, bs).sum(-1).double() / size > 0.60
        keep |= forced
        total = int(nnz[0, m])
        assert total == int(keep.sum()) and bool((tau != -0.6) | (total > int(forced.sum())))
        assert torch.equal(rowptr[0, m, 1:], keep.sum(-1).cumsum(0).int()) and int(rowptr[0, m, 0]) == 0
        assert torch.equal(colidx[0, m, :total], keep.nonzero()[:, 1].int())
