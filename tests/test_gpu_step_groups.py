"""Whole steps whose attention takes several heads per workgroup and leaves sums of probabilities in the place of logits, against the
same layers one by one: heads that are no multiple of a group, layers in and behind the groups, layers that keep their logits among them."""
import pytest
import torch

from paper_2412_20105_amd import binding as st3
from test_gpu_step_launches import BF, Step, _same

pytestmark = pytest.mark.gpu


# A workgroup takes 8, 4 or 2 heads while that many rows are at most a 384th of what the launch has behind the layer: of `strips` equal strips a
# layer and L layers, layer l takes 8 while (L - 1 - l) * strips >= 8 * 384, and so on.
@pytest.mark.parametrize("args", [
    dict(L=20, B=16, H=12, d=128, dtype=BF, vis=[70], tail=5),                  # 8, 4, 2 and one head; 12 = 8 + 4
    dict(L=20, B=24, H=13, d=64, dtype=BF, vis=[61, 33], tail=5),               # one head left over of every group
    dict(L=9, B=64, H=3, d=128, dtype=BF, vis=[40, 300, 7], tail=3),            # pairs of three heads in the first layer, longer layers head by head behind it
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


# ---- which layers are grouped, read from what the step has left in the workspaces -----------------------------------------------------
UNTOUCHED = 0x7f7f7f7f


def _mark(step):
    """Workspaces of words that no call writes (the descriptors cleared as a program has them)."""
    for s in step.state:
        s["ws"].fill_(0x7f)
        st3.st3_workspace_init(step.shape, s["v"].shape[2], s["ws"])
    return step


def _groups(step, drop):
    """Heads whose probabilities each layer's attention has added up (1: it has left logits, None: of every key, or no mass).  A sum takes the
    place of the logits of its heads and needs no norms; the descriptor takes four words a sequence, a list of moves three for each and one."""
    out = []
    for l, s in enumerate(step.state):
        n, (B, H) = s["n"], step.out.shape[1:3]
        if n == 0 or step.arr[l].vis_mass is None or l in step.lazy or l in step.lazy.values():
            out.append(None)
            continue
        words = int((s["ws"].view(torch.int32) != UNTOUCHED).sum())
        fits = [g for g in (8, 4, 2, 1) if 0 <= words - 4 * B - B * n * -(-H // g) - (B * H * 2 if g == 1 else 0) <= B * (3 * drop + 1)]
        assert len(fits) == 1, (l, words, fits)
        out += fits
    return out


def _rule(step):
    """The same by the rule: at most a 384th of the rows behind the layer."""
    B, H = step.out.shape[1:3]
    rows, out, g = [s["kv_len"][0].item() + 1 for s in step.state], [], 8
    own = [l for l in range(step.L) if l not in step.lazy]
    for l in range(step.L):
        behind = B * H * sum(rows[j] for j in own if j > l)
        while g > 1 and (g > H or g * rows[l] * 384 > behind):
            g //= 2
        out.append(g)
    return out


def _ragged(step):
    for s in step.state:
        s["vis_len"][1::3] = s["n"] - 11
        s["vis_len"][2::5] = 0
        s["vis_len"][3::7] = s["n"] // 2 + 1
        s["kv_len"][4::9] -= 1


@pytest.mark.parametrize("ragged", [False, True])
@pytest.mark.parametrize("args,drop", [
    (dict(L=20, B=32, H=8, d=128, dtype=BF, vis=[300], tail=6, e4m3=True), 2),          # a second round of the threads that add, and of keys
    (dict(L=20, B=32, H=9, d=64, dtype=BF, vis=[257, 256], tail=4, e4m3=True), 12),     # one head left over; either side of a round
    (dict(L=17, B=32, H=12, d=128, dtype=BF, vis=[520, 513], tail=3), 30),              # three rounds; eight heads and four
    (dict(L=16, B=32, H=16, d=64, dtype=BF, vis=[300], tail=5, fixed_tail=False), 40),
    (dict(L=20, B=32, H=8, d=128, dtype=BF, vis=[270], tail=4, e4m3=True, lazy={3: 2, 4: 2, 19: 18}), 7),
    (dict(L=20, B=32, H=8, d=64, dtype=BF, vis=[300], tail=4, lazy={1: 0, 7: 6}), 7),
])
def test_the_groups_that_the_rule_names(args, drop, ragged):
    a, b = _mark(Step(**args, drop=drop)), Step(**args, drop=drop)
    if ragged:
        _ragged(a); _ragged(b)
    rule = _rule(a)
    a.whole()
    assert rule[0] == 8 and rule[-1] == 1 and {4, 2} <= set(rule)
    if not ragged:                      # (else fewer words than the bounds say are written)
        assert all(got in (None, want) for got, want in zip(_groups(a, drop), rule))
        assert _groups(a, drop).count(None) == len({*a.lazy, *a.lazy.values()})
    _same(a, b.layer_by_layer())


@pytest.mark.parametrize("dtype,e4m3", [(BF, False), (BF, True)])
def test_keys_without_weight_and_not_numbers(dtype, e4m3):
    """Logits of -inf and NaN in grouped layers: rows of a wave's tile, all rows but one, every row of a strip."""
    args = dict(L=20, B=32, H=8, d=64, dtype=dtype, vis=[300], tail=5, e4m3=e4m3, drop=0)
    a, b = _mark(Step(**args)), Step(**args)
    for s in (a, b):
        q, k_new = s.qkv[:, 0], s.qkv[:, 1]
        q[..., 0] = 8.0
        for st in s.state:
            k, nan = (st["k"], 0x7f) if e4m3 else (st["k"][..., 0], float("nan"))
            k[3, 2, 77] = nan                                   # one key of one head: the sequence has no mass
            k[4, 7] = nan
            if not e4m3:                                        # (E4M3 has no infinity)
                low = float("-inf")
                k[0, :, 16:48] = low
                k[1, ::2, :250] = low
                k[2, 1, :290] = low
                k[5, 3] = low
        if not e4m3:
            k_new[:, 5, 3, 0] = float("-inf")                   # every key of this strip: no softmax
            k_new[:, 6, :, 0] = float("-inf")
    a.whole()
    assert _groups(a, 0)[0] == 8 and set(_groups(a, 0)) == {8, 4, 2, 1}
    b.layer_by_layer()
    lost = (3, 4) if e4m3 else (3, 4, 5)
    for l in range(a.L):
        bad = torch.zeros((32, 8), dtype=torch.bool, device=a.out.device)
        bad[3, 2] = bad[4, 7] = True
        bad[5, 3] = not e4m3
        for s in (a, b):
            assert torch.equal(s.out[l].isnan().any(dim=-1), bad) and torch.equal(s.out[l].isnan().all(dim=-1), bad), l
            mass = s.state[l]["mass"]
            assert all(bool(mass[i].isnan().all() if i in lost else mass[i].isfinite().all()) for i in range(32)), l
    ok = ~a.out.isnan()
    x, y = a.out[ok].double(), b.out[ok].double()
    assert bool(((x - y).abs() <= 1e-5 + 2.0 ** -7 * y.abs()).all())        # as _same
    for s, t in zip(a.state, b.state):
        assert torch.allclose(s["mass"], t["mass"], rtol=5e-5, atol=1e-9, equal_nan=True)
