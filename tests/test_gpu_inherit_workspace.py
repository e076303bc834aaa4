"""A lazy layer's stand-alone attention whose scratch is its source's workspace: it reads what the source left there and leaves it
as it was, for the lazy layers that follow."""
import pytest
import torch

from paper_2412_20105_amd import binding as st3

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("B,H,lens", [
    (2, 3, [700, 31]),                          # strips cut into chunks
    (4, 70, [90, 5, 64, 1]),                    # whole strips, many workgroups a sequence
    (1, 1, [0]),                                # nothing to inherit
], ids=["cut", "whole", "empty"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_source_and_scratch_in_one_workspace(B, H, lens, dtype):
    g = torch.Generator(device=DEV).manual_seed(B * 100 + H)
    d, ns, cap = 64, 1, max(lens) + 3
    shape = st3.make_shape(B, H, d, st3.ST3_F32 if dtype == torch.float32 else st3.ST3_BF16)
    q = torch.randn((B, H, d), generator=g, device=DEV).to(dtype)
    k, v, *lazy = (torch.randn((B, H, cap, d), generator=g, device=DEV).to(dtype) for _ in range(5))
    kv_len = torch.tensor(lens, dtype=torch.int32, device=DEV)
    vis = (kv_len - ns).clamp(min=0)
    seg = st3.segments(ns, int(vis.max()), max(lens), vis, kv_len)
    ws = torch.empty((st3.st3_workspace_bytes(shape, cap, int(vis.max()), 1),), dtype=torch.uint8, device=DEV)
    st3.st3_workspace_init(shape, cap, ws)
    src_out, outs = torch.zeros_like(q), [torch.full_like(q, 7.0) for _ in lazy]
    st3.st3_decode_attention(shape, q, st3.kv_layer(k, v), seg, src_out, None, ws)
    for vl, out in zip(lazy, outs):             # one after the other, each of the same source
        st3.st3_decode_attention_inherit(shape, st3.kv_layer(None, vl), seg, ws, cap, out, ws)
    torch.cuda.synchronize()
    # float32 sums of up to 700 products of weights that add to 1 with values of at most about 6: 1e-5; a bf16 output rounds once more
    step = 2.0 ** -8 if dtype == torch.bfloat16 else 0.0
    for b, n in enumerate(lens):
        p = torch.softmax((k[b, :, :n].double() * q[b, :, None].double()).sum(-1) / d ** 0.5, dim=-1)
        for values, got in [(v, src_out), *zip(lazy, outs)]:
            want = (p[:, :, None] * values[b, :, :n].double()).sum(1)
            assert bool(((got[b].double() - want).abs() <= 1e-5 + step * want.abs()).all()), (b, float((got[b].double() - want).abs().max()))
