"""bf16 attention at d = 64, whose rows go straight from memory to LDS (stages of 64, at block size 32 a tile of 32 per wavefront): sequences that end anywhere in a stage, tensors of
any row and head stride (rows 2^31 bytes apart among them), lists in any order and with entries that name no block."""
import math

import pytest
import torch

import paper_2604_20470_amd as dr

pytestmark = pytest.mark.gpu


def reference(Q, K, V, keep, bs):
    """fp64 softmax over the keys of the kept blocks; keep: [Sb, Sb] bool."""
    N = Q.shape[2]
    allowed = keep.repeat_interleave(bs, 0).repeat_interleave(bs, 1)[:N, :N]
    s = (Q.double() @ K.double().transpose(-1, -2) / 8.0).masked_fill(~allowed, -math.inf)
    return torch.softmax(s, -1) @ V.double(), torch.logsumexp(s, -1)


def attend(Q, K, V, rowptr, colidx, bs):
    B, H, N, _ = Q.shape
    shape = dr.shape_of(Q, 1, 1, N, bs)
    O, lse = torch.empty_strided(Q.shape, Q.stride(), dtype=Q.dtype, device="cuda"), torch.empty(B, H, N, device="cuda")
    dr.dr_sparse_attn_fwd(dr.Context(0), shape, Q, K, V, rowptr, colidx, 1, colidx.shape[2], O, lse)
    return O, lse


def check(O, lse, want, want_lse):
    # O is rounded once to bf16: eight significant bits, half a unit in the last place is at most 2^-8 of the value; all before is 32-bit
    assert ((O.double() - want).abs() <= 2 ** -8 * want.abs() + 1e-5).all()
    assert (lse.double() - want_lse).abs().max() < 1e-5


@pytest.mark.parametrize("bs", [32, 64, 128])
@pytest.mark.parametrize("N", [1, 31, 32, 33, 63, 64, 65, 95, 97, 127, 128, 129, 191, 193, 257, 700])
@pytest.mark.parametrize("layout", ["plain", "strided"])
def test_every_end_of_the_sequence(bs, N, layout):
    B, H = 2, 3
    g = torch.Generator(device="cuda").manual_seed(N)
    if layout == "plain":
        Q, K, V = (torch.randn(B, H, N, 64, generator=g, device="cuda").bfloat16() for _ in range(3))
    else:                                                        # [B, N, H, 192] with q, k, v side by side
        x = torch.randn(B, N, H, 192, generator=g, device="cuda").bfloat16()
        Q, K, V = (x[..., i * 64:i * 64 + 64].transpose(1, 2) for i in range(3))
    Sb = -(-N // bs)
    keep = torch.rand(Sb, Sb, generator=g, device="cuda") < 0.6
    keep.fill_diagonal_(True)
    rowptr, cols = torch.zeros(Sb + 1, dtype=torch.int32, device="cuda"), []
    for r in range(Sb):
        own = keep[r].nonzero().flatten().int()
        cols.append(own.flip(0) if r % 2 else own)               # any order
        rowptr[r + 1] = rowptr[r] + own.numel()
    colidx = torch.cat(cols).repeat(B, 1, 1)
    O, lse = attend(Q, K, V, rowptr.repeat(B, 1, 1), colidx, bs)
    check(O, lse, *reference(Q, K, V, keep, bs))


@pytest.mark.parametrize("bs", [32, 64, 128])
def test_rows_two_gigabytes_apart(bs):
    N, stride = 5, 1 << 30
    g = torch.Generator(device="cuda").manual_seed(1)
    x = torch.empty(N * stride, dtype=torch.bfloat16, device="cuda")
    Q, K, V = (x.as_strided((1, 1, N, 64), (N * stride, N * stride, stride, 1), 64 * i) for i in range(3))
    for t in (Q, K, V):
        t.copy_(torch.randn(1, 1, N, 64, generator=g, device="cuda"))
    shape = dr.shape_of(Q, 1, 1, N, bs)
    O = x.as_strided((1, 1, N, 64), (N * stride, N * stride, stride, 1), 192)
    lse = torch.empty(1, 1, N, device="cuda")
    rowptr, colidx = torch.tensor([[[0, 1]]], dtype=torch.int32, device="cuda"), torch.zeros(1, 1, 1, dtype=torch.int32, device="cuda")
    dr.dr_sparse_attn_fwd(dr.Context(0), shape, Q, K, V, rowptr, colidx, 1, 1, O, lse)
    check(O, lse, *reference(Q, K, V, torch.ones(1, 1, dtype=torch.bool, device="cuda"), bs))


@pytest.mark.parametrize("bs", [32, 64, 128])
def test_entries_that_name_no_block_are_clamped(bs):
    N = 3 * bs - 5
    g = torch.Generator(device="cuda").manual_seed(2)
    Q, K, V = (torch.randn(1, 1, N, 64, generator=g, device="cuda").bfloat16() for _ in range(3))
    rowptr = torch.tensor([[[0, 1, 2, 3]]], dtype=torch.int32, device="cuda")
    colidx = torch.tensor([[[-7, 1, 99]]], dtype=torch.int32, device="cuda")
    O, lse = attend(Q, K, V, rowptr, colidx, bs)
    check(O, lse, *reference(Q, K, V, torch.eye(3, dtype=torch.bool, device="cuda"), bs))


@pytest.mark.parametrize("H", [8, 9, 16])                        # 32 blocks each: 256 workgroups, 288, 512
def test_few_and_many_workgroups_give_the_same_bits(H):
    N, bs = 1000, 32
    g = torch.Generator(device="cuda").manual_seed(3)
    Q, K, V = (torch.randn(1, H, N, 64, generator=g, device="cuda").bfloat16() for _ in range(3))
    Sb = -(-N // bs)
    rowptr = (torch.arange(Sb + 1, dtype=torch.int32) * Sb).view(1, 1, -1).cuda()
    colidx = torch.arange(Sb, dtype=torch.int32).repeat(Sb).view(1, 1, -1).cuda()
    O, lse = attend(Q, K, V, rowptr, colidx, bs)
    check(O, lse, *reference(Q, K, V, torch.ones(Sb, Sb, dtype=torch.bool, device="cuda"), bs))
    for h in range(H):
        own_O, own_lse = attend(*(t[:, h:h + 1].contiguous() for t in (Q, K, V)), rowptr, colidx, bs)
        assert torch.equal(own_O[0, 0], O[0, h]) and torch.equal(own_lse[0, 0], lse[0, h])
