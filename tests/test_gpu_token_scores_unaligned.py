"""dr_token_scores reads sixteen (bf16: eight) bytes at a time and takes any element-aligned base: the same bits as from an aligned one."""
import pytest
import torch

import paper_2604_20470_amd as dr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("shift", [1, 2, 3, 5])
def test_base_aligned_to_an_element(dtype, d, shift):
    H, N = 2, 77
    g = torch.Generator(device="cuda").manual_seed(d + shift)
    Q, K = (torch.randn(1, H, N, d, generator=g, device="cuda").to(dtype) for _ in range(2))
    room = torch.zeros(2, H * N * d + 8, dtype=dtype, device="cuda")
    moved = [room[i, shift:shift + H * N * d].view(1, H, N, d).copy_(t) for i, t in enumerate((Q, K))]
    ctx, shape = dr.Context(0), dr.shape_of(Q, 1, 7, 11, 32)
    out = [torch.full((1, 1, N, N), float("nan"), device="cuda") for _ in range(2)]
    dr.dr_token_scores(ctx, shape, Q, K, H, out[0])
    dr.dr_token_scores(ctx, shape, *moved, H, out[1])
    assert torch.isfinite(out[0]).all() and torch.equal(out[0], out[1])
