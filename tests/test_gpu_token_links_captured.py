"""dr_build_mask_tokens of many small frames, first made under capture by a context whose bitmaps an earlier call has sized: the links go
the way that needs no other scratch, with the same bits."""
import pytest
import torch

import paper_2604_20470_amd as dr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("frames,hg,wg,masks", [(200, 1, 18, 1), (45, 5, 16, 1), (33, 11, 11, 1), (16, 8, 15, 4)])      # more than 12 * 2^20 pairs
def test_first_token_mask_of_a_context_may_be_captured(frames, hg, wg, masks):
    N, bs = frames * hg * wg, 32
    shape, params = dr.Shape(1, masks, N, 64, frames, hg, wg, bs, 0, 0, N * 64 * masks, N * 64, 64), dr.MaskParams(head_fuse=0)
    assert masks * N * N > 12 << 20
    Sb = -(-N // bs)
    g = torch.Generator(device="cuda").manual_seed(N)
    scores = torch.randn(1, masks, N, N, generator=g, device="cuda")

    def outputs(cap):
        return [torch.zeros(*s, dtype=t, device="cuda") for s, t in (((1, masks, Sb + 1), torch.int32), ((1, masks, cap), torch.int32),
                                                                      ((1, masks), torch.int64), ((1, masks, N, N), torch.uint8))]

    def tokens(ctx, cap, out):
        dr.dr_build_mask_tokens(ctx, shape, 0.4, 1.0, params, scores, out[0], out[1], cap, out[2], out[3])

    ctx = dr.Context(0)
    cap, _ = dr.dr_mask_capacity(ctx, shape, 1.0, params)
    want, got = outputs(cap), outputs(cap)
    tokens(ctx, cap, want)
    ctx = dr.Context(0)
    dr.dr_build_mask(ctx, shape, dr.MODE_STATIC, 0.5, 1.0, params, torch.zeros(1, masks, Sb, Sb, device="cuda"), got[0], got[1], cap, got[2])
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        tokens(ctx, cap, got)
    for _ in range(3):
        for t in got:
            t.fill_(7)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        n = int(want[2].max())
        assert torch.equal(got[0], want[0]) and torch.equal(got[2], want[2]) and torch.equal(got[3], want[3])
        for m in range(masks):
            assert torch.equal(got[1][0, m, :int(want[2][0, m])], want[1][0, m, :int(want[2][0, m])])
    tokens(ctx, cap, got)                       # and eagerly, with the scratch
    assert torch.equal(got[3], want[3]) and n > 0
