"""Eviction plans in parts (ranking beside the attention; masses, row moves and lengths behind it) and whole, where the columns
that are ranked take the step's mass: the edges of both and of the rule between them."""
import pytest
import torch

from test_gpu_step_launches import BF, F32, Step, _same
from test_gpu_step_launches import test_plan_keeps_the_best_rows_and_finishes_the_mass as plans_of_a_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,B,H,n,drop", [
    (1, 1, 3, 3, 1), (2, 2, 5, 255, 4), (2, 1, 33, 256, 48), (1, 3, 31, 257, 48), (1, 1, 7, 1027, 6),      # mass: four keys a lane
    (1, 1, 4, 60, 60),                                                                                      # nothing is kept
    (40, 60, 2, 30, 7),                                                                                     # one workgroup moves all strips
])
@pytest.mark.parametrize("fixed_tail", [True, False])
def test_parts(L, B, H, n, drop, fixed_tail):
    plans_of_a_step(L, B, H, n, drop, ties=n % 2 == 0, fixed_tail=fixed_tail)


@pytest.mark.parametrize("args", [
    dict(L=5, B=2, H=9, d=128, dtype=BF, vis=[200, 33], tail=9, e4m3={0, 3, 4}, lazy={1: 0, 4: 3}, drop=11),
    dict(L=4, B=3, H=5, d=64, dtype=BF, vis=[90], tail=2, e4m3=True, lazy={1: 0}, drop=48, fixed_tail=False),
    dict(L=3, B=2, H=3, d=128, dtype=F32, vis=[400], tail=30, drop=48, fixed_tail=False),
], ids=["mixed", "e4m3", "f32"])
def test_row_moves_of_every_format(args):
    _same(Step(**args).whole(), Step(**args).layer_by_layer())


@pytest.mark.parametrize("args", [
    dict(L=3, B=2, H=5, d=64, dtype=F32, vis=[60, 7], tail=3, drop=3),
    dict(L=2, B=3, H=33, d=128, dtype=BF, vis=[300], tail=9, drop=30, fixed_tail=False),
    dict(L=2, B=1, H=16, d=64, dtype=F32, vis=[1100], tail=5, drop=20),
], ids=["256", "512", "1024"])
@pytest.mark.parametrize("layer", [None, 1])
def test_columns_that_take_the_mass(args, layer):
    """Mass written into the score column (of all layers or of one): the rows that stay are those this step's attention gives
    most, so the ranking waits for the mass."""
    a, b = Step(**args), Step(**args)
    for s in (a, b):
        for l, st in enumerate(s.state):
            if layer in (None, l):
                s.arr[l].vis_mass, s.arr[l].mass_stride = st["score"].data_ptr(), st["score"].stride(0)
    was = [{x: st[x].clone() for x in ("k", "ids")} for st in a.state]
    a.whole()
    b.layer_by_layer()
    d, H = args["d"], args["H"]
    for l, (s, t, w) in enumerate(zip(a.state, b.state, was)):
        n, rows = s["n"], 3 + s["n"] + args["tail"]
        k = n - args["drop"]
        if layer not in (None, l):
            continue
        q, kn, _ = a.qkv[l].double()
        p = torch.softmax(torch.matmul(torch.cat([w["k"][:, :, :rows].double(), kn[:, :, None]], 2), q[..., None])[..., 0] / d ** 0.5, -1)
        mass = p[:, :, 3:3 + n].mean(1)
        for i in range(args["B"]):
            by_id = dict(zip(w["ids"][i].tolist(), mass[i].tolist()))
            kth = sorted(by_id.values())[n - k]
            for st in (s, t):
                kept = st["ids"][i, :k].tolist()
                assert len(set(kept)) == k
                # float32 probabilities: relative error 5e-5 (as for every mass)
                assert all(by_id[x] >= kth * (1 - 1e-4) for x in kept)
                got = torch.tensor([by_id[x] for x in kept], device=st["score"].device)
                assert torch.allclose(st["score"][i, :k], got.float(), rtol=5e-5, atol=1e-9)
        assert torch.equal(s["kv_len"], t["kv_len"]) and torch.equal(s["vis_len"], t["vis_len"])


@pytest.mark.parametrize("args", [
    dict(L=3, B=2, H=5, d=128, dtype=BF, vis=[700, 120], tail=9, drop=90, lazy={1: 0}),
    dict(L=2, B=1, H=3, d=64, dtype=F32, vis=[1500], tail=3, drop=900),
    dict(L=30, B=40, H=4, d=64, dtype=BF, vis=[90], tail=2, drop=60),               # fewer workgroups than a sequence's moves fill
    dict(L=3, B=2, H=5, d=128, dtype=BF, vis=[300], tail=9, drop=60, e4m3={1}),
    dict(L=3, B=2, H=5, d=128, dtype=BF, vis=[300], tail=200, drop=60, fixed_tail=False),       # by launches of their own
], ids=["bf16", "f32", "many_plans", "mixed", "closing_tail"])
def test_large_evictions(args):
    _same(Step(**args).whole(), Step(**args).layer_by_layer())
