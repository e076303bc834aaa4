"""Keys whose logit is -inf (a cached key of -inf, or one whose product with the query falls below the float32 range) weigh
nothing, wherever the rows of a tile, of a wave or of a chunk hold no other: outputs and masses are those of the softmax in 64
bits, never NaN."""
import math

import pytest
import torch

from paper_2412_20105_amd import binding as st3

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BF, F32 = torch.bfloat16, torch.float32
SYS = 3


class Layer:
    """One layer's cache of `rows` rows per sequence, rows `dead` of every strip with logit -inf."""

    def __init__(self, B, H, d, dtype, rows, dead, lowest=False, with_new=False, new_dead=False, seed=0):
        g = torch.Generator(device=DEV).manual_seed(seed + rows * 7 + B * H + d)
        rnd = lambda *s: torch.randn(s, generator=g, device=DEV).to(dtype)  # noqa: E731
        self.B, self.H, self.d, self.rows, self.n = B, H, d, rows, rows - SYS - 5
        self.q, self.k_new, self.v_new = rnd(B, H, d), rnd(B, H, d), rnd(B, H, d)
        self.k, self.v = rnd(B, H, rows + 4, d), rnd(B, H, rows + 4, d)
        # q[0] = 8: times -inf, or times the lowest finite value of the type (the product overflows)
        self.q[..., 0] = 8.0
        value = torch.finfo(dtype).min if lowest else -math.inf
        for x, n in ((self.k[:, :, :, 0], dead), (self.k_new[:, :, 0], None)):
            if n is not None:
                x[:, :, list(n)] = value
            elif new_dead:
                x[:] = value
        self.out = torch.full((B, H, d), math.nan, dtype=dtype, device=DEV)
        self.mass = torch.zeros((B, self.n), device=DEV)
        self.vis = torch.full((B,), self.n, dtype=torch.int32, device=DEV)
        self.len = torch.full((B,), rows, dtype=torch.int32, device=DEV)
        self.shape = st3.make_shape(B, H, d, st3.ST3_F32 if dtype == F32 else st3.ST3_BF16)
        self.ws = torch.empty((st3.st3_workspace_bytes(self.shape, rows + 4, self.n, 1),), dtype=torch.uint8, device=DEV)
        st3.st3_workspace_init(self.shape, rows + 4, self.ws)
        self.kv = st3.kv_layer(self.k, self.v)
        self.seg = st3.segments(SYS, self.n, rows, self.vis, self.len)
        self.keys, self.values = self.k[:, :, :rows].double(), self.v[:, :, :rows].double()
        if with_new:
            self.keys = torch.cat([self.keys, self.k_new[:, :, None].double()], dim=2)
            self.values = torch.cat([self.values, self.v_new[:, :, None].double()], dim=2)

    def probabilities(self):
        x = torch.matmul(self.keys, self.q.double()[..., None])[..., 0] / math.sqrt(self.d)
        # (in 64 bits the product of the lowest value is finite, and as far below the other logits)
        return torch.softmax(x, dim=-1)

    def check(self, out=None, mass=True, values=None):
        p = self.probabilities()
        assert bool((p.sum(dim=-1) - 1).abs().max() < 1e-9)
        out = self.out if out is None else out
        want = torch.matmul(p[:, :, None], self.values if values is None else values)[:, :, 0]
        # float32 sums of terms below 8 in all, and one rounding to the output's type
        step = 2.0 ** -8 if out.dtype == BF else 0.0
        err = (out.double() - want).abs()
        assert bool((err <= 1e-4 + step * want.abs()).all()), float(err.max())
        if mass:
            # a float32 exponent of a logit good to a few 1e-6, normaliser, sum over heads (as for every mass)
            assert torch.allclose(self.mass.double(), p[:, :, SYS:SYS + self.n].mean(dim=1), rtol=5e-5, atol=1e-9)


# rows that begin a wave's share of a chunk, a whole chunk, the front of the strip, all rows but one
DEAD = {"tile": range(224, 240), "half_tile": range(224, 232), "wave": range(224, 288), "chunks": range(64, 640), "front": range(0, 64),
        "long_front": range(0, 700), "scattered": range(1, 1100, 2), "all_but_one": [x for x in range(1111) if x != 777]}


@pytest.mark.parametrize("lowest", [False, True])
@pytest.mark.parametrize("dead", list(DEAD))
@pytest.mark.parametrize("B,H,d,dtype", [(5, 40, 128, BF), (1, 4, 128, BF), (1, 4, 64, BF), (2, 3, 64, F32), (1, 5, 128, F32), (13, 40, 64, BF)])
def test_decode_attention(B, H, d, dtype, dead, lowest):
    x = Layer(B, H, d, dtype, 1111, DEAD[dead], lowest)
    st3.st3_decode_attention(x.shape, x.q, x.kv, x.seg, x.out, x.mass, x.ws)
    x.check()
    alone = torch.full_like(x.out, math.nan)
    st3.st3_decode_attention(x.shape, x.q, x.kv, x.seg, alone, None, x.ws)
    x.check(alone, mass=False)
    x.mass.zero_()
    x.out.fill_(math.nan)
    st3.st3_decode_attention_noalloc(x.shape, x.q, x.kv, x.seg, x.out, x.mass)
    x.check()


@pytest.mark.parametrize("B,H,d,dtype", [(1, 4, 128, BF), (2, 3, 64, F32)])
@pytest.mark.parametrize("dead", ["tile", "chunks", "front"])
def test_a_lazy_layer_inherits_them(B, H, d, dtype, dead):
    src, lazy = (Layer(B, H, d, dtype, 1111, DEAD[dead], seed=s) for s in (0, 1))
    st3.st3_decode_attention(src.shape, src.q, src.kv, src.seg, src.out, src.mass, src.ws)
    st3.st3_decode_attention_inherit(lazy.shape, st3.kv_layer(None, lazy.v), lazy.seg, src.ws, 1111 + 4, lazy.out, lazy.ws)
    src.check(lazy.out, mass=False, values=lazy.values)


# 64 * 5 rows and the appended one: the new row can be the only one of its chunk
@pytest.mark.parametrize("rows,dead,new_dead", [(320, range(0), True), (320, range(256, 320), True), (320, range(128, 192), False),
                                               (321, range(320, 321), True), (1111, range(224, 240), True), (70, range(0, 16), False)])
@pytest.mark.parametrize("B,H,d,dtype", [(1, 4, 128, BF), (1, 3, 64, F32), (12, 40, 64, BF)])
def test_steps(B, H, d, dtype, rows, dead, new_dead):
    one = Layer(B, H, d, dtype, rows, dead, with_new=True, new_dead=new_dead)
    st3.st3_decode_layer_step(one.shape, one.kv, one.seg, None, None, -1, st3.ST3_HOLE_FILL, one.q, one.k_new, one.v_new, one.out,
                              one.mass, one.ws)
    one.check()
    layers = [Layer(B, H, d, dtype, rows, dead, with_new=True, new_dead=new_dead, seed=s) for s in range(3)]
    arr = (st3.LayerStep * 3)()
    for e, x in zip(arr, layers):
        e.kv, e.seg, e.keep_after, e.inherit_from = x.kv, x.seg, -1, -1
        e.q, e.k_new, e.v_new, e.out = x.q.data_ptr(), x.k_new.data_ptr(), x.v_new.data_ptr(), x.out.data_ptr()
        e.vis_mass, e.mass_stride = x.mass.data_ptr(), x.mass.stride(0)
        e.workspace, e.workspace_bytes = x.ws.data_ptr(), x.ws.numel()
    arr[2].inherit_from = 1
    st3.st3_decode_step(layers[0].shape, arr, 3, st3.ST3_HOLE_FILL)
    for x in layers[:2]:
        x.check()
    layers[1].check(layers[2].out, mass=False, values=layers[2].values)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n,dead", [(100, 40), (300, 64), (300, 200)])
def test_float32_prefill_behind_a_dead_front(d, n, dead):
    """Queries whose first tiles hold dead keys only (a query that sees no other key has no softmax and is left out)."""
    g = torch.Generator(device=DEV).manual_seed(n + d)
    q, k, v = (torch.randn((2, 3, n, d), generator=g, device=DEV) for _ in range(3))
    q[..., 0] = 8.0
    k[:, :, :dead, 0] = -math.inf
    vis = n - 5
    shape = st3.make_shape(2, 3, d, st3.ST3_F32)
    ws = torch.empty((st3.st3_workspace_bytes(shape, n, vis, 4),), dtype=torch.uint8, device=DEV)
    out, mass = torch.empty_like(q), torch.zeros((2, vis), device=DEV)
    st3.st3_prefill_attention(shape, q, k, v, n, 2, vis, 4, out, mass, ws)
    x = torch.matmul(q.double(), k.double().transpose(2, 3).contiguous()) / math.sqrt(d)
    p = torch.softmax(x.masked_fill(torch.ones((n, n), dtype=torch.bool, device=DEV).triu(1), -math.inf), dim=-1)
    want = torch.matmul(p[:, :, dead:], v.double())
    assert float((out[:, :, dead:].double() - want).abs().max()) < 1e-4
    assert torch.allclose(mass.double(), p[:, :, n - 4:, 2:2 + vis].sum(dim=2).mean(dim=1), rtol=5e-5, atol=1e-9)
