"""The head reductions of the visual mass and the cuts of a stand-alone decode attention, at the edges of the groups that
heads, window rows, keys and chunks are dealt to, against the same sums in 64 bits."""
import math

import pytest
import torch

from paper_2412_20105_amd import binding as st3

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _close(got, want):
    # float32 exponents of logits good to 1e-6, a normaliser, a sum over heads: 5e-5, as for every mass
    assert torch.allclose(got.double(), want, rtol=5e-5, atol=1e-9), float((got.double() - want).abs().max())


@pytest.mark.parametrize("B,H,n,sys_len,vis,window", [
    (1, 1, 1, 0, 1, 1),             # fewer (head, row) pairs than waves
    (2, 3, 70, 5, 63, 1),
    (1, 16, 70, 2, 64, 1),          # one pair per wave
    (1, 17, 90, 3, 65, 1),
    (2, 40, 200, 7, 193, 16),       # window rows that cannot see the last keys
    (1, 5, 130, 0, 129, 7),
])
def test_prefill_mass(B, H, n, sys_len, vis, window):
    g = torch.Generator(device=DEV).manual_seed(n * 7 + H)
    q, k, v = (torch.randn((B, H, n, 64), generator=g, device=DEV) for _ in range(3))
    shape = st3.make_shape(B, H, 64, st3.ST3_F32)
    ws = torch.empty((st3.st3_workspace_bytes(shape, n, vis, window),), dtype=torch.uint8, device=DEV)
    ws.fill_(0xFF)                  # logits that no row has left are NaN
    out, mass = torch.empty_like(q), torch.zeros((B, vis), device=DEV)
    st3.st3_prefill_attention(shape, q, k, v, n, sys_len, vis, window, out, mass, ws)
    x = torch.matmul(q.double(), k.double().transpose(2, 3).contiguous()) / 8.0
    p = torch.softmax(x.masked_fill(torch.ones((n, n), dtype=torch.bool, device=DEV).triu(1), -math.inf), dim=-1)
    _close(mass, p[:, :, n - window:, sys_len:sys_len + vis].sum(dim=2).mean(dim=1))


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("B,H,lens", [
    (1, 1, [1]),
    (1, 3, [4096]),                 # 63 chunks, the most that this call cuts
    (1, 16, [256]), (1, 16, [257]), (1, 47, [700]), (1, 48, [700]),        # few strips: finer cuts for short ones only
    (2, 64, [700, 31]), (3, 43, [700, 64, 1]), (8, 40, [600, 1, 65, 300, 64, 128, 599, 2]), (3, 107, [600, 33, 257]),
    (3, 1, [64, 65, 700]),
    (5, 40, [173, 1111, 600, 64, 999]),
    (2, 65, [513, 300]),
    (4, 128, [130, 129, 128, 1]),   # enough strips: none is cut
])
def test_decode_attention_and_mass_in_chunks(B, H, lens, noalloc):
    g = torch.Generator(device=DEV).manual_seed(B * 100 + H)
    cap, sys_len = max(lens) + 3, 1
    nvis = [max(0, min(x - sys_len, (x * 2) // 3)) for x in lens]
    q = torch.randn((B, H, 64), generator=g, device=DEV)
    k, v = (torch.randn((B, H, cap, 64), generator=g, device=DEV) for _ in range(2))
    shape = st3.make_shape(B, H, 64, st3.ST3_F32)
    seg = st3.segments(sys_len, max(nvis), max(lens), torch.tensor(nvis, dtype=torch.int32, device=DEV),
                       torch.tensor(lens, dtype=torch.int32, device=DEV))
    out, mass = torch.empty_like(q), torch.zeros((B, max(1, max(nvis))), device=DEV)
    kv = st3.kv_layer(k, v)
    if noalloc:
        st3.st3_decode_attention_noalloc(shape, q, kv, seg, out, mass)
    else:
        ws = torch.empty((st3.st3_workspace_bytes(shape, cap, max(nvis), 1),), dtype=torch.uint8, device=DEV)
        st3.st3_workspace_init(shape, cap, ws)
        st3.st3_decode_attention(shape, q, kv, seg, out, mass, ws)
    for b in range(B):
        p = torch.softmax(torch.matmul(k[b, :, :lens[b]].double(), q[b].double()[..., None])[..., 0] / 8.0, dim=-1)
        want = torch.matmul(p[:, None], v[b, :, :lens[b]].double())[:, 0]
        assert float((out[b].double() - want).abs().max()) < 1e-4
        if nvis[b]:
            _close(mass[b, :nvis[b]], p[:, sys_len:sys_len + nvis[b]].mean(dim=0))
        assert not mass[b, nvis[b]:].any()
