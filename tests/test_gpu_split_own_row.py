"""fp32-accuracy attention (fp32 storage, bf16 at d = 64): a query block's result is its own list's alone, to the last bit, and a
call keeps nothing outside its inputs and outputs, so that calls of one context may overlap and the first may be captured."""
import numpy as np
import pytest
import torch

import paper_2604_20470_amd as dr

pytestmark = pytest.mark.gpu

KINDS = [("f32", 64, 128), ("f32", 64, 64), ("f32", 128, 128), ("f32", 128, 64), ("bf16", 64, 128), ("bf16", 64, 64)]
GEO = (8, 24, 32)                               # N = 6144: two heads leave most of the chip idle


def _inputs(dtype, d, bs, heads, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    N = GEO[0] * GEO[1] * GEO[2]
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    q, k, v = (torch.randn(1, heads, N, d, generator=g, device="cuda").to(dt) for _ in range(3))
    keep = np.random.default_rng(seed).random((N // bs, N // bs)) < 0.5
    rowptr = torch.from_numpy(np.concatenate([[0], keep.sum(1).cumsum()]).astype(np.int32)).view(1, 1, -1).cuda()
    colidx = torch.from_numpy(np.nonzero(keep)[1].astype(np.int32)).view(1, 1, -1).cuda()
    return q, k, v, rowptr, colidx


def _attend(ctx, bs, q, k, v, rowptr, colidx, O=None, stream=None, fn=dr.dr_sparse_attn_fwd):
    O = torch.empty_like(q) if O is None else O
    lse = torch.empty(q.shape[:3], dtype=torch.float32, device="cuda")
    fn(ctx, dr.shape_of(q, *GEO, bs), q, k, v, rowptr, colidx, 1, colidx.shape[2], O, lse, stream)
    return O, lse


@pytest.mark.parametrize("dtype,d,bs", KINDS)
def test_bits_depend_on_the_row_alone(dtype, d, bs):
    ctx = dr.Context(0)
    q, k, v, rowptr, colidx = _inputs(dtype, d, bs, 5, 1)
    O, lse = _attend(ctx, bs, q, k, v, rowptr, colidx)
    wide = torch.zeros(1, 1, 8 * colidx.shape[2], dtype=torch.int32, device="cuda")
    wide[..., :colidx.shape[2]] = colidx
    assert all(torch.equal(x, y) for x, y in zip(_attend(ctx, bs, q, k, v, rowptr, wide), (O, lse)))      # a larger capacity
    few = _attend(ctx, bs, *(t[:, :2].contiguous() for t in (q, k, v)), rowptr, colidx)                   # fewer heads
    assert torch.equal(few[0], O[:, :2]) and torch.equal(few[1], lse[:, :2])


@pytest.mark.parametrize("dtype,d,bs", KINDS)
def test_first_call_of_a_context_may_be_captured(dtype, d, bs):
    q, k, v, rowptr, colidx = _inputs(dtype, d, bs, 2, 2)
    want, _ = _attend(dr.Context(0), bs, q, k, v, rowptr, colidx)
    torch.cuda.synchronize()
    ctx, O, graph = dr.Context(0), torch.empty_like(q), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        _attend(ctx, bs, q, k, v, rowptr, colidx, O)
    for _ in range(3):
        O.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(O, want)


@pytest.mark.parametrize("fn", [dr.dr_sparse_attn_fwd, dr.dr_sparse_attn_fwd_static], ids=["context", "static"])
@pytest.mark.parametrize("dtype,d,bs", KINDS)
def test_calls_on_two_streams_may_overlap(dtype, d, bs, fn):
    ctx = dr.Context(0)
    sides = []
    for seed in (3, 4):
        x = _inputs(dtype, d, bs, 2, seed)
        want, _ = _attend(ctx, bs, *x)
        torch.cuda.synchronize()
        sides.append((torch.cuda.Stream(), x, want))
    for _ in range(10):
        outs = [_attend(ctx, bs, *x, stream=s, fn=fn) for s, x, _ in sides]
        torch.cuda.synchronize()
        assert all(torch.equal(O, want) for (O, _), (_, _, want) in zip(outs, sides))
