"""Whole steps over caches whose rows lie more than a megabyte apart (token-major, all layers of a token side by side) or whose
system prompt is longer than 65535 rows: their layers share launches like any others', with the results of the layers one by one."""
import pytest
import torch

from paper_2412_20105_amd import binding as st3
from test_gpu_step_fallbacks import launches
from test_gpu_step_launches import BF, DEV, F32, Step, _same

pytestmark = pytest.mark.gpu


def token_major(step, row_bytes):
    """The step's caches moved into one buffer of rows of that many bytes, every layer's K and V side by side."""
    s0 = step.state[0]["v"]
    B, H, _, d = s0.shape
    cap = max(s["v"].shape[2] for s in step.state)
    offset, views = 0, []
    for s in step.state:
        for name in ("k", "v"):
            if s[name] is not None:
                views.append((s, name, offset))
                offset += B * H * d * s[name].element_size()
    assert offset <= row_bytes
    big = torch.zeros((cap * row_bytes,), dtype=torch.uint8, device=DEV)
    for s, name, at in views:
        x = s[name]
        t = big.view(x.dtype)
        eb = x.element_size()
        view = torch.as_strided(t, x.shape, (H * d, d, row_bytes // eb, 1), at // eb)
        view.copy_(x)
        s[name] = view
    for l, s in enumerate(step.state):
        scale = step.refs[3 * l + 2]
        step.arr[l].kv = st3.kv_layer(s["k"], s["v"], None if s["k"] is None else scale, scale)
    step.refs.append(big)
    return step


@pytest.mark.parametrize("args", [
    dict(L=4, B=2, H=5, d=128, dtype=BF, vis=[60, 33], tail=9, lazy={1: 0}),
    dict(L=3, B=1, H=3, d=64, dtype=F32, vis=[70], tail=5, drop=60),
    dict(L=3, B=2, H=4, d=128, dtype=BF, vis=[80], tail=3, e4m3={0, 2}, fixed_tail=False),
    dict(L=35, B=1, H=2, d=64, dtype=BF, vis=[20], tail=2),             # more layers than a wide table holds
], ids=["lazy", "f32", "mixed", "many"])
@pytest.mark.parametrize("more", [0, 16])
def test_rows_far_apart(args, more):
    wide = lambda: token_major(Step(**args), (1 << 20) + more)  # noqa: E731
    _same(wide().whole(), wide().layer_by_layer())
    # ordinary layers of one format, lazy ones and a format of their own: one attention launch each, and one behind them all
    # (evictions included); 35 layers of wide entries take two attention launches where others take one
    extra = 1 if args["L"] == 35 else 0
    assert launches(wide()) <= launches(Step(**args)) + extra


def test_columns_that_take_the_mass_with_rows_far_apart():
    args = dict(L=3, B=2, H=5, d=64, dtype=F32, vis=[60, 7], tail=3, drop=3)
    a, b = token_major(Step(**args), 1 << 20), Step(**args)
    for s in (a, b):
        for l, st in enumerate(s.state):
            s.arr[l].vis_mass, s.arr[l].mass_stride = st["score"].data_ptr(), st["score"].stride(0)
    _same(a.whole(), b.whole())         # (cut alike: the same sums in the same order)


def test_a_system_prompt_of_more_than_65535_rows():
    """The rows in front of the visual ones are shared by all layers here (nothing moves or writes them)."""
    def build():
        s = Step(L=2, B=1, H=1, d=64, dtype=F32, vis=[40], tail=9)
        head = 70_000
        g = torch.Generator(device=DEV).manual_seed(5)
        for l, st in enumerate(s.state):
            cap = head + st["v"].shape[2]
            for name in ("k", "v"):
                st[name] = torch.cat([torch.randn((1, 1, head, 64), generator=g, device=DEV), st[name]], dim=2)
            for name in ("kv_len", "tail"):
                st[name] += head
            st["ws"] = torch.empty((st3.st3_workspace_bytes(s.shape, cap, 40, 1),), dtype=torch.uint8, device=DEV)
            st3.st3_workspace_init(s.shape, cap, st["ws"])
            e = s.arr[l]
            e.kv = st3.kv_layer(st["k"], st["v"])
            e.seg = st3.segments(3 + head, 40, 3 + head + 49, st["vis_len"], st["kv_len"], st["tail"], 40, 3 + head + 40)
            e.workspace, e.workspace_bytes = st["ws"].data_ptr(), st["ws"].numel()
        return s

    _same(build().whole(), build().layer_by_layer())
    assert launches(build()) == 2
