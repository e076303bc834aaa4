"""Rows ranked by the first workgroups of a step's attention launch, one for each layer and sequence: where they fill their part of the
grid (heads x chunks a slice), where one is left over, and beside layers that evict nothing."""
import pytest
import torch

from test_gpu_step_launches import BF, F32, Step, _same
from test_gpu_step_launches import test_plan_keeps_the_best_rows_and_finishes_the_mass as plans_of_a_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,B,H,n,drop", [
    (2, 2, 4, 30, 3),                   # a slice of four, four rankings
    (2, 2, 3, 30, 3),                   # a slice of three, four rankings
    (5, 7, 1, 40, 9),                   # slices of one
    (3, 2, 2, 700, 11),                 # slices of heads x chunks
    (35, 3, 2, 20, 2), (36, 3, 2, 20, 2),       # the most layers of a launch, and one more
])
def test_rankings_of_a_launch(L, B, H, n, drop):
    plans_of_a_step(L, B, H, n, drop, ties=True, fixed_tail=True)


@pytest.mark.parametrize("evicting", [{0}, {3}, {1, 4}])
@pytest.mark.parametrize("lazy", [{}, {2: 1, 5: 4}])
def test_some_layers_evict(evicting, lazy):
    evicting = evicting | {l for l, src in lazy.items() if src in evicting}
    args = dict(L=6, B=3, H=5, d=128, dtype=BF, vis=[90, 60], tail=9, drop=7, lazy=lazy)
    a, b = Step(**args), Step(**args)
    for s in (a, b):
        for l in range(6):
            src = lazy.get(l, l)
            if l not in evicting:
                s.arr[l].keep_after = -1
            elif src != l:
                s.arr[l].keep_after = s.arr[src].keep_after
    _same(a.whole(), b.layer_by_layer())
    assert [bool((st["vis_len"] < st["n"]).all()) for st in a.state] == [l in evicting for l in range(6)]


def test_no_layer_evicts():
    args = dict(L=3, B=2, H=3, d=64, dtype=F32, vis=[70], tail=4, drop=100)
    _same(Step(**args).whole(), Step(**args).layer_by_layer())


@pytest.mark.parametrize("L,B,H,n,drop", [
    (1, 1, 2, 1024, 6), (1, 1, 2, 1700, 6), (1, 1, 2, 1900, 6),         # beside the attention: 1024 rows and fewer; the line at 1636
    (2, 1, 2, 2000, 60), (1, 1, 2, 2000, 60),                           # two layers, or one, that evict more than a plan moves
    (1, 1, 16, 8192, 9), (1, 1, 15, 8192, 9), (1, 1, 14, 8192, 8190),   # the most rows: 16 heads beside, 14 behind
])
@pytest.mark.parametrize("fixed_tail", [True, False])
def test_ranked_beside_the_attention_or_behind_it(L, B, H, n, drop, fixed_tail):
    plans_of_a_step(L, B, H, n, drop, ties=n % 100 == 0, fixed_tail=fixed_tail)


def test_steps_ranked_behind_the_attention():
    for args in (dict(L=2, B=2, H=3, d=128, dtype=BF, vis=[2900, 40], tail=9, drop=30, lazy={1: 0}),
                 dict(L=2, B=1, H=4, d=64, dtype=F32, vis=[3000, 900], tail=3, drop=500),
                 dict(L=3, B=1, H=2, d=128, dtype=BF, vis=[2500], tail=9, drop=20, e4m3={1}, fixed_tail=False)):
        _same(Step(**args).whole(), Step(**args).layer_by_layer())
