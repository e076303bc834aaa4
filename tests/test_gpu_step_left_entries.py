"""Whole steps of more layers than one ranking table holds, whose columns take the step's mass: the plans are launched once, from the
entries that the attention leaves in the workspaces, with the results of the same layers in two calls."""
import ctypes as C

import pytest
import torch

from paper_2412_20105_amd import binding as st3
from test_gpu_step_fallbacks import launches
from test_gpu_step_launches import BF, F32, MODE, Step
from test_gpu_step_wide_rows import token_major

pytestmark = pytest.mark.gpu


def _current(args, make=lambda s: s):
    s = make(Step(**args))
    for l, st in enumerate(s.state):
        s.arr[l].vis_mass, s.arr[l].mass_stride = st["score"].data_ptr(), st["score"].stride(0)
    return s


def _in_two_calls(s, first):
    """Layers [0, first), then the rest (strips are cut alike: 64 rows a chunk, the shortest)."""
    size = C.sizeof(st3.LayerStep)
    for at, n in ((0, first), (first, s.L - first)):
        part = (st3.LayerStep * n).from_buffer(s.arr, at * size)
        st3.st3_decode_step(s.shape, part, n, MODE)
    torch.cuda.synchronize()
    return s


def _equal(a, b):
    assert torch.equal(a.out, b.out)
    for l, (x, y) in enumerate(zip(a.state, b.state)):
        for name in ("ids", "score", "kv_len", "vis_len", "k", "v"):
            if x[name] is not None:
                assert torch.equal(x[name], y[name]), (l, name)


CASES = [
    dict(L=35, B=1, H=2, d=64, dtype=F32, vis=[60, 7], tail=3, drop=3),             # one table holds them
    dict(L=36, B=1, H=2, d=64, dtype=F32, vis=[60, 7], tail=3, drop=3),
    dict(L=40, B=2, H=3, d=128, dtype=BF, vis=[150, 20], tail=9, drop=5),           # strips cut in chunks
    dict(L=41, B=3, H=2, d=64, dtype=BF, vis=[90], tail=4, drop=60, fixed_tail=False),      # rows moved by launches of their own
    dict(L=40, B=2, H=2, d=128, dtype=BF, vis=[40], tail=9, drop=5, e4m3={1, 5, 39}, lazy={2: 0, 3: 0, 6: 5}),
    dict(L=80, B=1, H=1, d=64, dtype=F32, vis=[33], tail=2, drop=2),
]


@pytest.mark.parametrize("args", CASES, ids=["35", "36", "cut", "moved", "mixed", "80"])
def test_many_layers_whose_columns_take_the_mass(args):
    _equal(_in_two_calls(_current(args), 20), _current(args).whole())


def test_wide_entries():
    args = dict(CASES[2], L=33)          # (32 to a table)
    far = lambda s: token_major(s, 1 << 20)  # noqa: E731
    _equal(_in_two_calls(_current(args, far), 16), _current(args, far).whole())
    assert launches(_current(args, far)) <= 3


def test_workspaces_without_room_behind():
    """Workspaces of just what the decode calls take: the entries travel in two launches."""
    def tight(s):
        for l, e in enumerate(s.arr):
            e.workspace_bytes = st3.st3_workspace_bytes(s.shape, e.kv.capacity, 0, 1) - 256     # (less the prefill's part)
        return s
    args = CASES[1]
    _equal(_in_two_calls(_current(args), 20), tight(_current(args)).whole())
    assert launches(tight(_current(args))) == launches(_current(args)) + 1


@pytest.mark.parametrize("L,most", [(35, 2), (36, 3), (40, 3), (70, 3), (80, 4)])
def test_launches(L, most):
    """35 layers to an attention launch, one launch behind them all."""
    assert launches(_current(dict(L=L, B=1, H=1, d=64, dtype=F32, vis=[20], tail=2))) == most
