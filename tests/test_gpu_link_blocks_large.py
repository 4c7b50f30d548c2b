"""Link bytes that go past the caches (from 140 million of them on) against the rule in fp64: columns that end inside a step, links that are and
are not aligned to words, and rows that are no multiple of four (both of which keep to the caches)."""
import pytest
import torch

import paper_2604_20470_amd as dr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("frames,hg,wg,masks,offset", [
    (8, 37, 40, 1, 0),       # 11 840: 140.2 million
    (8, 37, 40, 1, 1),       # ... from an odd address
    (7, 1, 1693, 1, 0),      # 11 851
    (4, 34, 50, 4, 0),       # 6800 x 4 masks
])
def test_links_past_the_caches_follow_the_rule(frames, hg, wg, masks, offset):
    N, bs = frames * hg * wg, 128
    Sb = -(-N // bs)
    assert masks * N * N >= 140000000
    params = dr.MaskParams(head_fuse=0, tau_far=0.9)
    g = torch.Generator(device="cuda").manual_seed(N)
    scores = torch.randn(1, masks, N, N, generator=g, device="cuda")
    shape = dr.Shape(1, masks, N, 64, frames, hg, wg, bs, 0, 0, N * 64 * masks, N * 64, 64)
    ctx = dr.Context(0)
    cap, _ = dr.dr_mask_capacity(ctx, shape, 1.0, params)
    rowptr = torch.zeros(1, masks, Sb + 1, dtype=torch.int32, device="cuda")
    colidx = torch.zeros(1, masks, cap, dtype=torch.int32, device="cuda")
    nnz = torch.zeros(1, masks, dtype=torch.int64, device="cuda")
    links = torch.full((masks * N * N + 8,), 9, dtype=torch.uint8, device="cuda")[offset:offset + masks * N * N].view(1, masks, N, N)
    dr.dr_build_mask_tokens(ctx, shape, 0.4, 1.0, params, scores, rowptr, colidx, cap, nnz, links)

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
                tau = 0.4 if base >= bs else 0.9
                sure = inside & ((z - tau).abs() > 1e-9)          # (the sums' order may decide the others)
                assert torch.equal(got[sure].bool(), z[sure] >= tau) and not bool(got[~inside].any())
    total = int(nnz[0, 0])
    assert total == int(rowptr[0, 0, -1]) and total > 0
