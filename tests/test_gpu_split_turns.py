"""fp32 attention at d = 64, block size 128, on both sides of the number of query blocks from which a workgroup takes its two streams of keys in
turn: the same bits, for sequences that end anywhere, lists of any length and order, and values that send a block to the plain pass."""
import math

import pytest
import torch

import paper_2604_20470_amd as dr

pytestmark = pytest.mark.gpu


def attend(q, k, v, rowptr, colidx):
    O, lse = torch.full_like(q, 7.0), torch.full(q.shape[:3], 7.0, device="cuda")
    dr.dr_sparse_attn_fwd(dr.Context(0), dr.shape_of(q, 1, 1, q.shape[2], 128), q, k, v, rowptr, colidx, 1, colidx.shape[2], O, lse)
    return O, lse


@pytest.mark.parametrize("N,heads", [(128 * 70 - 37, 33), (128 * 70 - 100, 33), (128 * 30 - 64, 66), (128 * 15 - 1, 88), (700, 66), (128, 550), (31, 550), (97, 550)])
@pytest.mark.parametrize("kind", ["plain", "infinite"])
def test_many_blocks_have_the_bits_of_few(N, heads, kind):
    Sb, few = -(-N // 128), max(1, heads // 11)
    line = 256 * (1 if Sb <= 8 else 4 if Sb <= 16 else 7 if Sb <= 32 else 8)      # on 256 compute units
    assert Sb * heads > line >= Sb * few
    g = torch.Generator(device="cuda").manual_seed(N)
    q, k, v = (torch.randn(1, heads, N, 64, generator=g, device="cuda") for _ in range(3))
    if kind == "infinite":
        k[:, 1::7, N // 2, 5] = -math.inf
        v[:, ::5, N // 3] = math.inf
    lists = []
    for qb in range(Sb):
        own = torch.randperm(Sb, generator=torch.Generator().manual_seed(qb))[:qb % (Sb + 1) if Sb > 1 else 1].tolist()
        lists.append(own if qb % 3 else sorted(own))
    rowptr = torch.tensor([0] + [len(l) for l in lists]).cumsum(0).int().view(1, 1, -1).cuda()
    colidx = torch.tensor([kb for l in lists for kb in l], dtype=torch.int32).view(1, 1, -1).cuda()
    O, lse = attend(q, k, v, rowptr, colidx)
    for h in range(0, heads, 3 * few):
        part = attend(*(t[:, h:h + few].contiguous() for t in (q, k, v)), rowptr, colidx)
        want = O[:, h:h + few], lse[:, h:h + few]
        assert all(torch.equal(x.view(torch.int32), y.contiguous().view(torch.int32)) for x, y in zip(part, want)), h
    if kind == "plain":                                     # one head against 64 bits
        h = heads - 1
        allowed = torch.zeros(Sb, Sb, dtype=torch.bool, device="cuda")
        for qb, l in enumerate(lists):
            allowed[qb, l] = True
        allowed = allowed.repeat_interleave(128, 0).repeat_interleave(128, 1)[:N, :N]
        s = (q[0, h].double() @ k[0, h].double().T / 8.0).masked_fill(~allowed, -math.inf)
        want = torch.softmax(s, -1).nan_to_num(0.0) @ v[0, h].double()
        # 32-bit probabilities and sums: 2^-24 of each of up to 8960 terms, of size |v| in the mean
        assert (O[0, h].double() - want).abs().max() < 2e-5
        some = allowed.any(-1)
        assert (lse[0, h].double() - torch.logsumexp(s, -1))[some].abs().max() < 1e-5 and bool(torch.isneginf(lse[0, h][~some]).all())
