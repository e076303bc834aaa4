"""Whole steps of batches whose sequences differ in length, with and without the caller's word that most are as long as the bounds:
strips are cut differently, with the results of the layers one by one."""
import pytest
import torch

from test_gpu_step_launches import BF, F32, Step, _same

pytestmark = pytest.mark.gpu


def _build(args, part, hint):
    s = Step(**args)
    for l, st in enumerate(s.state):
        n, B = st["n"], st["vis_len"].numel()
        if n == 0:
            continue
        st["vis_len"].copy_(torch.tensor([n if b == 0 else max(1, int(n * part)) for b in range(B)], dtype=torch.int32))
        if hint != "all":
            s.arr[l].seg.vis_len_hint = n - 1 if hint == "shorter" else 0 if hint == "none" or l == 0 else n
    return s


@pytest.mark.parametrize("hint", ["all", "shorter", "none", "one_layer"])
@pytest.mark.parametrize("args", [
    dict(L=3, B=4, H=40, d=64, dtype=BF, vis=[900, 0], tail=9),                         # a chunk of 512ths is longer than 384 rows, of 2048ths not
    dict(L=2, B=8, H=70, d=64, dtype=F32, vis=[760], tail=20, drop=6),                  # both are
    dict(L=2, B=3, H=4, d=128, dtype=BF, vis=[300], tail=9, drop=6, lazy={1: 0}),       # neither is
], ids=["384", "2048ths", "512ths"])
@pytest.mark.parametrize("part", [1.0, 0.1])
def test_cuts_of_a_ragged_batch(args, hint, part):
    _same(_build(args, part, hint).whole(), _build(args, part, hint).layer_by_layer())
