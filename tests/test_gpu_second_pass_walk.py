"""The second pass over flagged query blocks: one walk of a block's list in its order, whose bits follow from the list alone, and O and
log-sum-exp against 64 bits for lists of every length and order that the walk treats differently."""
import math

import pytest
import torch

import paper_2604_20470_amd as dr

pytestmark = pytest.mark.gpu


def csr(lists):
    """rowptr, colidx [1, 1, ..] of one list of key blocks per query block."""
    rowptr = torch.tensor([0] + [len(l) for l in lists]).cumsum(0).int().view(1, 1, -1).cuda()
    return rowptr, torch.tensor([kb for l in lists for kb in l], dtype=torch.int32).view(1, 1, -1).cuda()


def attend(Q, K, V, lists, bs, ctx=None):
    B, H, N, _ = Q.shape
    O, lse = torch.full_like(Q, 7.0), torch.zeros(B, H, N, device="cuda")
    rowptr, colidx = csr(lists)
    rowptr, colidx = rowptr.repeat(B, 1, 1), colidx.repeat(B, 1, 1)
    dr.dr_sparse_attn_fwd(ctx or dr.Context(0), dr.shape_of(Q, 1, 1, N, bs), Q, K, V, rowptr, colidx, 1, colidx.shape[2], O, lse)
    return O, lse


def check_rows(O, lse, Q, K, V, rows, keys, scaled_q=False):
    """Rows `rows` of one head against fp64 over the keys `keys`.  The probabilities are rounded to bf16 (2^-8 each, in the sum of O and in the
    normaliser alike) and so is O; what is left, logits summed in 32 bits, is 128 products of 2^-24 of the largest of weight.
    scaled_q: the fast pass, whose scaled Q is rounded to bf16 again, 2^-8 of every product."""
    q, k = Q[rows].double(), K[keys].double()
    s = q @ k.T / math.sqrt(Q.shape[-1])
    p, v = torch.softmax(s, -1), V[keys].double()
    want, want_lse = p @ v, torch.logsumexp(s, -1)
    weight = p > 2.0 ** -60
    slack = 128 * 2.0 ** -24 * torch.where(weight, s.abs(), 0.0).amax(-1)
    if scaled_q:
        slack = slack + 2.0 ** -8 * torch.where(weight, q.abs() @ k.abs().T / math.sqrt(Q.shape[-1]), 0.0).amax(-1)
    spread = torch.stack([(p * (v[:, c] - want[:, c:c + 1]).abs()).sum(-1) for c in range(v.shape[1])], -1)
    assert ((O[rows].double() - want).abs() <= 2.0 ** -8 * (1.02 * spread + 1.02 * want.abs()) + 2 * slack[:, None] * spread + 1e-6).all()
    assert ((lse[rows].double() - want_lse).abs() <= 2.0 ** -8 + slack + 2.0 ** -22 * want_lse.abs()).all()
    return want_lse


@pytest.mark.parametrize("N", [128 * 9, 128 * 9 - 37, 128 * 8 + 35])          # last blocks of 128, 91 and 35 tokens
def test_flagged_blocks_have_the_bits_of_one_walk_in_order(N):
    """The second pass of block size 64 walks the same keys in the same steps of 64 where every block is given as its two halves."""
    H, Sb, Sb64 = 3, -(-N // 128), -(-N // 64)
    g = torch.Generator(device="cuda").manual_seed(N)
    Q, K, V = (torch.randn(1, H, N, 128, generator=g, device="cuda").bfloat16() for _ in range(3))
    Q = (Q.float() * 14).bfloat16()
    keep = torch.rand(Sb, Sb, generator=torch.Generator().manual_seed(N)) < 0.7
    lists = [[kb for kb in range(Sb) if keep[qb, kb] or kb == qb] for qb in range(Sb)]
    halves = [[k for kb in lists[qb64 // 2] for k in (2 * kb, 2 * kb + 1) if k < Sb64] for qb64 in range(Sb64)]
    O, lse = attend(Q, K, V, lists, 128)
    want_O, want_lse = attend(Q, K, V, halves, 64)
    flagged = torch.nn.functional.pad(lse.abs() > 46.0, (0, Sb * 128 - N)).view(H, Sb, 128).any(-1).repeat_interleave(128, 1)[:, :N]
    assert flagged.float().mean() > 0.8
    assert torch.equal(O[0][flagged], want_O[0][flagged]) and torch.equal(lse[0][flagged], want_lse[0][flagged])


@pytest.mark.parametrize("order", ["ascending", "descending", "one_chunk_block_second"])
def test_lists_of_every_length_against_64_bits(order):
    bs, Sb = 128, 131
    N = Sb * bs - 70                                     # the last block is one step of 64 keys
    g = torch.Generator(device="cuda").manual_seed(5)
    Q, K, V = (torch.randn(1, 1, N, 128, generator=g, device="cuda").bfloat16() for _ in range(3))
    lists = [[qb] for qb in range(Sb)]
    lengths = {0: 1, 7: 2, 20: 3, 21: 64, 50: 65, 51: 128, 90: 129, 91: 130, 130: 131}
    for qb, n in lengths.items():
        own = torch.randperm(Sb - 1, generator=torch.Generator().manual_seed(qb))[:n - 1].tolist() + [Sb - 1]
        own.sort(reverse=order == "descending")
        if order == "one_chunk_block_second" and n > 1:
            own = [own[0], Sb - 1] + own[1:-1]
        lists[qb] = own
        Q[0, 0, qb * bs:qb * bs + bs] *= 20
    O, lse = attend(Q, K, V, lists, bs)
    for qb in lengths:
        rows = torch.arange(qb * bs, min(qb * bs + bs, N), device="cuda")
        keys = torch.cat([torch.arange(kb * bs, min(kb * bs + bs, N), device="cuda") for kb in lists[qb]])
        assert check_rows(O[0, 0], lse[0, 0], Q[0, 0], K[0, 0], V[0, 0], rows, keys).abs().max() > 46.0


@pytest.mark.parametrize("heads", [(0, 10), (13, 17), (30, 40), (0, 40)])     # of the first batch: 120 blocks of one queue; some of two; ..
def test_clusters_of_flagged_blocks_are_drawn_from_any_xcd(monkeypatch, heads):
    """More flagged blocks in one queue than its own workgroups, 64 on 256 compute units: the others' take part, call after call."""
    B, H, Sb = 2, 40, 12
    N = Sb * 128 - 9
    g = torch.Generator(device="cuda").manual_seed(heads[1])
    Q, K, V = (torch.randn(B, H, N, 128, generator=g, device="cuda").bfloat16() for _ in range(3))
    Q[0, heads[0]:heads[1]] *= 20
    lists = [list(range(Sb))] * Sb
    ctx = dr.Context(0)
    monkeypatch.setenv("DR_ATTN_PAIRS", "0")
    want_O, want_lse = attend(Q, K, V, lists, 128)
    flagged = torch.nn.functional.pad(want_lse.abs() > 46.0, (0, 9)).view(B, H, Sb, 128).any(-1)
    assert int(flagged.sum()) >= 11 * (heads[1] - heads[0])
    rows = flagged.repeat_interleave(128, 2)[:, :, :N]
    for _ in range(3):
        O, lse = attend(Q, K, V, lists, 128, ctx)
        assert torch.equal(O[rows], want_O[rows]) and torch.equal(lse[rows], want_lse[rows])
        assert (O.float() - want_O.float()).abs().max() < 4e-2
