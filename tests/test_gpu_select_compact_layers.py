"""Evictions of several layers in one call where entries share what the call writes: the result is that of the single calls in order."""
import pytest
import torch

from paper_2412_20105_amd import binding as st3
from test_gpu_step_launches import BF, F32, Step

pytestmark = pytest.mark.gpu


def _pair(share, drop, mode, fixed_tail):
    """Two equal sets of layers; share(entries, state): what they have in common."""
    out = []
    for _ in range(2):
        s = Step(L=3, B=2, H=4, d=64, dtype=F32, vis=[90, 150, 40], tail=9, fixed_tail=fixed_tail, drop=drop)
        share(s)
        out.append(s)
    a, b = out
    st3.st3_select_compact_layers(a.shape, a.arr, a.L, mode)
    for l in range(b.L):
        e, st = b.arr[l], b.state[l]
        ws = b.state[1]["ws"] if e.workspace == b.state[1]["ws"].data_ptr() else st["ws"]
        st3.st3_select_compact_layer(b.shape, e.kv, e.seg, st["score"], st["ids"], e.keep_after, mode, ws)
    torch.cuda.synchronize()
    for l, (x, y) in enumerate(zip(a.state, b.state)):
        for name in ("ids", "score", "kv_len", "vis_len", "k", "v"):
            assert torch.equal(x[name], y[name]), (l, name)


@pytest.mark.parametrize("drop", [7, 30])               # moved by the plan; by a launch of their own (STABLE always)
@pytest.mark.parametrize("mode", [st3.ST3_HOLE_FILL, st3.ST3_STABLE])
@pytest.mark.parametrize("fixed_tail", [True, False])
def test_one_workspace_for_all_layers(drop, mode, fixed_tail):
    def share(s):       # the largest one
        for e in s.arr:
            e.workspace, e.workspace_bytes = s.state[1]["ws"].data_ptr(), s.state[1]["ws"].numel()
    _pair(share, drop, mode, fixed_tail)


def test_one_layer_twice():
    """The second entry finds the lengths and the columns as the first one left them."""
    s, t = (Step(L=2, B=2, H=4, d=64, dtype=BF, vis=[90], tail=9, drop=20) for _ in range(2))
    s.arr[1] = s.arr[0]
    s.arr[1].keep_after = 50
    st3.st3_select_compact_layers(s.shape, s.arr, 2, st3.ST3_HOLE_FILL)
    e, st = t.arr[0], t.state[0]
    for keep in (70, 50):
        st3.st3_select_compact_layer(t.shape, e.kv, e.seg, st["score"], st["ids"], keep, st3.ST3_HOLE_FILL, st["ws"])
    torch.cuda.synchronize()
    for name in ("ids", "score", "kv_len", "vis_len", "k", "v"):
        assert torch.equal(s.state[0][name], st[name]), name
    assert st["vis_len"].tolist() == [50, 50]
