"""bf16 prefill attention at the edges of the rule that picks how many groups of waves share a query block's keys, of its
tiles and of the score window, against the same attention in 64 bits."""
import math

import pytest
import torch

from paper_2412_20105_amd import binding as st3

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _run(B, H, d, n, sys_len, vis, window, extra_rows=0, dead=()):
    g = torch.Generator(device=DEV).manual_seed(n * 13 + H + d)
    q, k, v = (torch.randn((B, H, n + (extra_rows if i else 0), d), generator=g, device=DEV).to(torch.bfloat16) for i in range(3))
    q[..., 0] = 1.0
    for j in dead:
        k[:, :, j, 0] = -math.inf       # keys of logit -inf for every query
    shape = st3.make_shape(B, H, d, st3.ST3_BF16)
    ws = torch.empty((st3.st3_workspace_bytes(shape, n, vis, window),), dtype=torch.uint8, device=DEV)
    ws.fill_(0xFF)                      # logits that no row has left are NaN
    out, mass = torch.full_like(q, math.nan), torch.zeros((B, max(vis, 1)), device=DEV)
    st3.st3_prefill_attention(shape, q, k[:, :, :n], v[:, :, :n], n, sys_len, vis, window, out, mass if vis else None, ws)
    above = torch.ones((n, n), dtype=torch.bool, device=DEV).triu(1)
    for b in range(B):
        x = torch.matmul(q[b].double(), k[b, :, :n].double().transpose(1, 2).contiguous()) / math.sqrt(d)
        p = torch.softmax(x.masked_fill(above, -math.inf), dim=-1)
        want = torch.matmul(p, v[b, :, :n].double())
        # one rounding to bf16 (2^-9 of the value) and, for values far below their row's largest, P's 16 bits: 2^-16 of that
        err = (out[b].double() - want).abs()
        assert bool((err <= 2.0 ** -8 * want.abs() + 2.0 ** -13 * want.abs().amax(dim=-1, keepdim=True)).all()), (n, float(err.max()))
        if vis:
            m = p[:, n - window:, sys_len:sys_len + vis].sum(dim=1).mean(dim=0)
            assert torch.allclose(mass[b].double(), m, rtol=5e-5, atol=1e-9), n


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 63, 64, 65, 95, 127, 128, 129, 161, 255, 256, 257, 300])
def test_four_groups(n, d):
    _run(1, 3, d, n, 0, max(0, n - 1), 1, extra_rows=5)


@pytest.mark.parametrize("B,H,d,n", [
    (1, 32, 128, 257), (1, 32, 128, 739), (2, 32, 128, 448), (1, 16, 128, 543), (1, 8, 128, 1057), (1, 33, 128, 300),
    (1, 64, 64, 600), (3, 11, 64, 545), (1, 64, 64, 257)])
def test_two_groups(B, H, d, n):
    _run(B, H, d, n, 7, n - 40, 1)


@pytest.mark.parametrize("n", [193, 202, 211, 220, 229, 238, 247, 256, 257, 266, 275, 284, 293, 302, 311, 320])
def test_one_group_every_offset_of_the_query_tiles(n):
    _run(3, 33, 128, n, 3, n - 30, 1)


@pytest.mark.parametrize("B,H,d,n", [(1, 2, 128, 100), (1, 32, 128, 400), (3, 33, 128, 200), (1, 2, 64, 333), (5, 33, 64, 200)])
@pytest.mark.parametrize("window,sys_len,short", [(16, 0, 0), (16, 33, 3), (5, 64, 30), (1, 1, 17)])
def test_window_rows_and_visual_edges(B, H, d, n, window, sys_len, short):
    """Visual segments that start and end inside tiles, up to the last key; window rows that do not see them all."""
    _run(B, H, d, n, sys_len, n - sys_len - short, window)


@pytest.mark.parametrize("B,H,d,n", [(1, 2, 128, 250), (1, 32, 128, 300), (3, 33, 128, 200), (1, 2, 64, 250)])
@pytest.mark.parametrize("tile", [1, 2])
def test_a_tile_of_keys_that_weigh_nothing(B, H, d, n, tile):
    """The first keys that a group of waves meets have logit -inf: they add nothing, and nothing turns into NaN."""
    _run(B, H, d, n, 4, n - 20, 1, dead=range(64 * tile, 64 * tile + 64))
