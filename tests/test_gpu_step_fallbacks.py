"""Whole steps whose layers cannot all share a launch - caches of two formats, output or token rows that layers share, strides
that a launch's table cannot hold: the results are those of the layers one by one, in as few launches as the layers allow."""
import ctypes as C

import pytest
import torch

from paper_2412_20105_amd import binding as st3
from test_gpu_step_launches import BF, DEV, F32, MODE, Step, _same

pytestmark = pytest.mark.gpu


def launches(step, mode=MODE):
    """How many kernels the whole-step call enqueues (nothing runs: the call is captured and the graph's nodes are counted)."""
    hip = st3.lib()             # (the runtime that the library itself is linked to)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph, count = C.c_void_p(), C.c_size_t()
    assert hip.hipStreamBeginCapture(C.c_void_p(side.cuda_stream), 2) == 0      # relaxed
    try:
        st3.st3_decode_step(step.shape, step.arr, step.L, mode, side)
    finally:
        assert hip.hipStreamEndCapture(C.c_void_p(side.cuda_stream), C.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, C.byref(count)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return count.value


MIXED = [
    dict(L=8, B=1, H=4, d=128, dtype=BF, vis=[300, 90], tail=9, e4m3={1, 4, 5}),                            # cut strips
    dict(L=6, B=20, H=30, d=64, dtype=BF, vis=[40], tail=5, e4m3={0}),                                      # whole strips
    dict(L=7, B=2, H=5, d=128, dtype=BF, vis=[260], tail=9, e4m3={1, 2, 5}, lazy={1: 0, 2: 0, 5: 4, 6: 4}, fixed_tail=False),
    dict(L=4, B=2, H=4, d=128, dtype=BF, vis=[300], tail=9, e4m3={0, 3}, drop=80),                          # more moves than a plan's list holds
]


@pytest.mark.parametrize("args", MIXED)
def test_caches_of_two_formats(args):
    _same(Step(**args).whole(), Step(**args).layer_by_layer())


@pytest.mark.parametrize("args,most", [
    (MIXED[0], 3),              # one attention launch per format, one plan launch
    (MIXED[1], 3),
    (MIXED[2], 4),              # ordinary layers of one format, lazy ones of two
    (MIXED[3], 3),
])
def test_launches_of_a_step_with_two_formats(args, most):
    assert launches(Step(**args)) <= most


@pytest.mark.parametrize("L,e4m3,attention,behind", [
    (35, False, 1, 1), (36, False, 2, 1), (32, True, 1, 1), (33, True, 2, 1), (41, False, 2, 1), (42, False, 2, 2), (70, False, 2, 2),
    (71, False, 3, 2), (83, False, 3, 3),
])
def test_launches_of_many_layers(L, e4m3, attention, behind):
    """35 layers to an attention launch (32 with E4M3 caches), 41 to the launch behind it."""
    assert launches(Step(L=L, B=1, H=1, d=64, dtype=BF, vis=[20], tail=2, e4m3=e4m3)) == attention + behind


@pytest.mark.parametrize("mode", [MODE, st3.ST3_STABLE])
def test_evictions_by_launches_of_their_own(mode):
    """Many rows of a tail that closes up, or moves whose order matters: a launch for each layer that evicts."""
    args = dict(L=3, B=2, H=4, d=128, dtype=BF, vis=[300, 20], tail=9, drop=80, fixed_tail=mode != MODE)
    a, b = Step(**args), Step(**args)
    st3.st3_decode_step(a.shape, a.arr, a.L, mode)
    for l in range(b.L):
        st3.st3_decode_layer_attend(b.shape, b.arr, b.L, l, mode)
    st3.st3_decode_plans(b.shape, b.arr, b.L, mode)
    torch.cuda.synchronize()
    _same(a, b)
    assert launches(Step(**args), mode) == 2 + 2


@pytest.mark.parametrize("field", ["q", "k_new", "v_new", "out"])
@pytest.mark.parametrize("lazy", [{}, {1: 0, 3: 2}])
def test_rows_shared_by_layers_with_cut_strips(field, lazy):
    """Layer 2 reads (or overwrites) what layer 0 has put out; every output is whole before the next layer runs."""
    args = dict(L=4, B=1, H=4, d=128, dtype=F32, vis=[500, 500, 300, 300], tail=9, lazy=lazy)
    a, b = Step(**args), Step(**args)
    for s in (a, b):
        setattr(s.arr[2], field, s.out[0].data_ptr())
    _same(a.whole(), b.layer_by_layer())


@pytest.mark.parametrize("field", ["col_stride", "mass_stride"])
def test_strides_beyond_the_table(field):
    """A stride of 2^33 floats (one sequence: never multiplied by more than 0) does not fit a table entry."""
    args = dict(L=18, B=1, H=4, d=128, dtype=BF, vis=[300, 90], tail=9, lazy={5: 4})
    a, b = Step(**args), Step(**args)
    for s in (a, b):
        setattr(s.arr[3], field, 1 << 33)
    _same(a.whole(), b.layer_by_layer())
