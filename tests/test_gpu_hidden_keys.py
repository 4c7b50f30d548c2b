"""bf16 attention at d = 128 over keys that a query cannot see, or hardly: a channel that puts their logits at -100, -50 000, the lowest value or
-infinity, in the first 64 keys of a row's list, of its second block, or of both, in rows of the second pass and of the fast one."""
import pytest
import torch

from test_gpu_second_pass_walk import attend, check_rows

pytestmark = pytest.mark.gpu

LOWEST = torch.finfo(torch.bfloat16).min


def inputs(N, H, level, hidden, hot):
    g = torch.Generator(device="cuda").manual_seed(N + len(hidden))
    Q, K, V = (torch.randn(1, H, N, 128, generator=g, device="cuda").bfloat16() for _ in range(3))
    if hot:
        Q[:, :, ::8] *= 24                                   # in every group of 128 rows: all are taken by the second pass
    Q[..., 127], K[..., 127] = 1.0, 0.0
    for lo, hi in hidden:
        K[:, :, lo:hi, 127] = level if level in (LOWEST, -float("inf")) else level * 128 ** 0.5
    return Q, K, V


@pytest.mark.parametrize("bs", [128, 64, 32])
@pytest.mark.parametrize("pairs", ["1", "0"])
@pytest.mark.parametrize("hot", [True, False])
@pytest.mark.parametrize("level", [-100.0, -2000.0, -50000.0, LOWEST, -float("inf")])
@pytest.mark.parametrize("hidden", [[(0, 64)], [(128, 192)], [(0, 64), (128, 192)], [(0, 256)], [(64, 700)]])
def test_rows_with_keys_out_of_sight(monkeypatch, bs, pairs, hot, level, hidden):
    monkeypatch.setenv("DR_ATTN_PAIRS", pairs)
    N, H = 700, 2
    Q, K, V = inputs(N, H, level, hidden, hot)
    Sb = -(-N // bs)
    lists = [[kb for kb in range(Sb) if kb != qb * 5 % Sb or kb * bs < 64] for qb in range(Sb)]
    O, lse = attend(Q, K, V, lists, bs)
    assert bool(torch.isfinite(O).all()) and bool(torch.isfinite(lse).all())
    for qb in range(Sb):
        rows = torch.arange(qb * bs, min(qb * bs + bs, N), device="cuda")
        keys = torch.cat([torch.arange(kb * bs, min(kb * bs + bs, N), device="cuda") for kb in lists[qb]])
        for h in range(H):
            check_rows(O[0, h], lse[0, h], Q[0, h], K[0, h], V[0, h], rows, keys, scaled_q=not hot)


@pytest.mark.parametrize("bs", [128, 64, 32])
@pytest.mark.parametrize("N", [40, 64, 200])                 # 40: too short for the kernels of 256 queries
@pytest.mark.parametrize("level", [-100.0, -400.0, LOWEST])
def test_rows_whose_keys_are_all_far_away(bs, N, level):
    """Every exponential of the fast pass underflows: the rows are taken again, whose weights are those of the logits' differences."""
    Q, K, V = inputs(N, 1, level, [(0, N)], False)
    Sb = -(-N // bs)
    O, lse = attend(Q, K, V, [list(range(Sb))] * Sb, bs)
    every = torch.arange(N, device="cuda")
    check_rows(O[0, 0], lse[0, 0], Q[0, 0], K[0, 0], V[0, 0], every, every)


@pytest.mark.parametrize("bs", [128, 64, 32])
@pytest.mark.parametrize("pairs", ["1", "0"])
def test_rows_without_keys_beside_rows_of_the_second_pass(monkeypatch, bs, pairs):
    monkeypatch.setenv("DR_ATTN_PAIRS", pairs)
    N = 512
    Q, K, V = inputs(N, 1, 0.0, [], True)
    Sb = N // bs
    empty = {1, Sb - 1}
    O, lse = attend(Q, K, V, [[] if qb in empty else list(range(Sb)) for qb in range(Sb)], bs)
    for qb in range(Sb):
        rows = torch.arange(qb * bs, qb * bs + bs, device="cuda")
        if qb in empty:
            assert bool((O[0, 0, rows] == 0).all()) and bool(torch.isneginf(lse[0, 0, rows]).all())
        else:
            check_rows(O[0, 0], lse[0, 0], Q[0, 0], K[0, 0], V[0, 0], rows, torch.arange(N, device="cuda"))


@pytest.mark.parametrize("bs", [128, 64, 32])
@pytest.mark.parametrize("more", [0.0, -60.0, -90.0, -108.0, -130.0])
def test_rows_at_the_edge_of_what_the_first_walk_sums(bs, more):
    """All exponents between 100 and 140 (units of log2) below the least reference of the second pass, where powers of 2 end."""
    N = 200
    Q, K, V = inputs(N, 1, 0.0, [], False)
    K[..., 127], Q[..., 126], K[..., 126] = -33024.0, 1.0, more
    Sb = -(-N // bs)
    O, lse = attend(Q, K, V, [list(range(Sb))] * Sb, bs)
    q, k = Q[0, 0].double(), K[0, 0].double()
    s = q @ k.T / 128 ** 0.5
    want, want_lse = torch.softmax(s, -1) @ V[0, 0].double(), torch.logsumexp(s, -1)
    # logits of size 33 000 in 32 bits, four roundings of 2^-24 each in their sum: 2^-7 of the unscaled logit, and as much of the exponent
    assert (O[0, 0].double() - want).abs().max() < 3e-2 and (lse[0, 0].double() - want_lse).abs().max() < 8e-3
