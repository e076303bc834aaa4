"""Whole steps whose attention takes several heads per workgroup and leaves sums of probabilities in the place of logits, against the
same layers one by one: heads that are no multiple of a group, layers in and behind the groups, layers that keep their logits among them."""
import pytest
import torch

from test_gpu_step_launches import BF, Step, _same

pytestmark = pytest.mark.gpu


# A workgroup takes 8, 4 or 2 heads while that many rows are at most a 384th of what the launch has behind the layer: of `strips` equal strips a
# layer and L layers, layer l takes 8 while (L - 1 - l) * strips >= 8 * 384, and so on.
@pytest.mark.parametrize("args", [
    dict(L=20, B=16, H=12, d=128, dtype=BF, vis=[70], tail=5),                  # 8, 4, 2 and one head; 12 = 8 + 4
    dict(L=20, B=24, H=13, d=64, dtype=BF, vis=[61, 33], tail=5),               # one head left over of every group
    dict(L=9, B=64, H=3, d=128, dtype=BF, vis=[40, 300, 7], tail=3),            # pairs of three heads, long layers behind short ones
    dict(L=4, B=400, H=1, d=64, dtype=BF, vis=[20], tail=3),                    # a single head: no groups
    dict(L=12, B=32, H=8, d=128, dtype=BF, vis=[65], tail=4, e4m3=True),
    dict(L=12, B=32, H=9, d=64, dtype=BF, vis=[130, 64], tail=4, e4m3={1, 4, 5, 6, 7, 8}),      # launches of either format
    dict(L=14, B=32, H=8, d=128, dtype=BF, vis=[80], tail=4, lazy={2: 1, 3: 1, 13: 12}),        # layers with heirs keep their logits
    dict(L=40, B=10, H=16, d=64, dtype=BF, vis=[50, 0, 33], tail=2),            # two launches; layers without visual rows
    dict(L=12, B=32, H=8, d=128, dtype=BF, vis=[90], tail=4, drop=30),
    dict(L=12, B=32, H=8, d=128, dtype=BF, vis=[90], tail=4, drop=100),         # nothing is evicted
    dict(L=12, B=32, H=8, d=128, dtype=BF, vis=[90], tail=4, fixed_tail=False),
])
def test_groups_of_heads(args):
    _same(Step(**args).whole(), Step(**args).layer_by_layer())


@pytest.mark.parametrize("e4m3", [False, True])
def test_sequences_that_differ_and_layers_without_a_mass(e4m3):
    args = dict(L=12, B=32, H=9, d=128, dtype=BF, vis=[90, 50], tail=6, e4m3=e4m3, drop=12)
    a, b = Step(**args), Step(**args)
    for s in (a, b):
        for l, st in enumerate(s.state):
            st["vis_len"][1::3] = st["n"] - 11          # fewer visual rows than the hint says, and than most
            st["vis_len"][2::5] = 0
            st["kv_len"][3::4] -= 2                     # (still behind the tail's start)
            if l % 5 == 2:
                s.arr[l].vis_mass = None
    _same(a.whole(), b.layer_by_layer())


def test_repeated_steps_are_bit_equal():
    args = dict(L=16, B=24, H=11, d=128, dtype=BF, vis=[77], tail=5)
    a, b = Step(**args).whole(), Step(**args).whole()
    assert torch.equal(a.out, b.out)
    assert all(torch.equal(s["mass"], t["mass"]) for s, t in zip(a.state, b.state))
