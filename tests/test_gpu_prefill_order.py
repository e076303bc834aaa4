"""The order in which a prefill launch deals its query tiles: every (strip, tile) once, whatever the number of strips."""
import math

import pytest
import torch

from paper_2412_20105_amd import binding as st3

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# strips below, at and above multiples of the 32 lanes, one to ten to a lane; two, three and five tiles
@pytest.mark.parametrize("B,H", [(1, 1), (1, 31), (1, 32), (3, 11), (1, 63), (2, 32), (5, 13), (4, 32), (7, 20), (5, 32), (9, 20),
                                 (8, 40)])
@pytest.mark.parametrize("n,D", [(129, 128), (330, 64), (333, 128), (642, 64)])
def test_every_tile_once(B, H, n, D):
    g = torch.Generator(device=DEV).manual_seed(B * 1000 + H * 10 + n)
    q, k, v = [torch.randn((B, H, n, D), generator=g, device=DEV).to(torch.bfloat16) for _ in range(3)]
    out = torch.full_like(q, float("nan"))
    mass = torch.full((B, n - 20), float("nan"), device=DEV)
    shape = st3.make_shape(B, H, D, st3.ST3_BF16)
    ws = torch.empty((st3.st3_workspace_bytes(shape, n, n - 20, 1),), dtype=torch.uint8, device=DEV)
    st3.st3_prefill_attention(shape, q, k, v, n, 10, n - 20, 1, out, mass, ws)
    causal = torch.ones((n, n), dtype=torch.bool, device=DEV).tril()
    for b in range(B):
        p = torch.matmul(q[b].float(), k[b].float().transpose(1, 2).contiguous()) / math.sqrt(D)
        p = torch.softmax(p.masked_fill_(~causal, float("-inf")), dim=-1)
        want = torch.matmul(p, v[b].float())
        # outputs are rounded to bf16 (2^-9 of the value); sums in float32 and P in 16 bits of mantissa leave less than 1e-4
        assert bool(((out[b].float() - want).abs() <= want.abs() / 256 + 2e-4).all()), b
        m = p[:, -1, 10:n - 10].mean(dim=0)
        assert bool(((mass[b] - m).abs() <= 1e-4 * m + 1e-9).all()), b


# prompts around the length from which a strip's tiles come one after the other: 4096 rows of 128, 8192 of 64; strips left over or not
@pytest.mark.parametrize("B,H,n,D", [(1, 33, 4096, 128), (1, 33, 4097, 128), (2, 32, 4200, 128), (3, 32, 8192, 64), (3, 33, 8193, 64)])
def test_order_of_long_prompts(B, H, n, D):
    g = torch.Generator(device=DEV).manual_seed(n)
    q, k, v = [torch.randn((B, H, n, D), generator=g, device=DEV).to(torch.bfloat16) for _ in range(3)]
    out = torch.full_like(q, float("nan"))
    st3.st3_prefill_attention(st3.make_shape(B, H, D, st3.ST3_BF16), q, k, v, n, 0, 0, 1, out, None, None)
    assert not bool(out.isnan().any())          # every row has been written
    rows = torch.tensor(sorted({0, n - 1, *range(37, n, 128), *range(127, n, 128)}), device=DEV)    # two of every tile
    causal = torch.arange(n, device=DEV)[None] <= rows[:, None]
    for b in range(B):
        p = torch.matmul(q[b][:, rows].float(), k[b].float().transpose(1, 2).contiguous()) / math.sqrt(D)
        want = torch.matmul(torch.softmax(p.masked_fill_(~causal, float("-inf")), dim=-1), v[b].float())
        assert bool(((out[b][:, rows].float() - want).abs() <= want.abs() / 256 + 2e-4).all()), b      # (as above)
