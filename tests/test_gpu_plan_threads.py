"""Top-k selection and eviction plans at the edges of the rules that pick how many threads a workgroup has."""
import pytest
import torch

from paper_2412_20105_amd import binding as st3
from test_gpu_step_launches import BF, DEV, F32, MODE, Step, _same
from test_gpu_step_launches import test_plan_keeps_the_best_rows_and_finishes_the_mass as plans_of_a_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("rows,n", [(1, 1), (3, 256), (3, 257), (2, 512), (2, 513), (5, 1024), (512, 1025), (513, 1025), (1, 8192), (2, 8193),
                                    (513, 16384), (4000, 16)])
def test_select_topk(rows, n, ties):
    g = torch.Generator(device=DEV).manual_seed(rows * 31 + n)
    score = torch.rand((rows, n), generator=g, device=DEV)
    if ties:
        score = (score * 8).floor()
    ids = torch.rand((rows, n), generator=g, device=DEV).argsort(dim=1).to(torch.int32)
    k = max(1, (n * 3) // 7)
    idx = torch.full((rows, k), -7, dtype=torch.int32, device=DEV)
    mask = torch.full((rows, n), 9, dtype=torch.uint8, device=DEV)
    st3.st3_select_topk(score, ids, None, n, k, mask, idx)
    by_id = ids.long().argsort(dim=1)           # (score descending, id ascending)
    order = by_id.gather(1, score.gather(1, by_id).argsort(dim=1, descending=True, stable=True))[:, :k]
    want = torch.zeros((rows, n), dtype=torch.uint8, device=DEV).scatter_(1, order, 1)
    assert torch.equal(mask, want)
    assert torch.equal(idx.long(), order.sort(dim=1)[0])


@pytest.mark.parametrize("L,B,H,n,drop", [
    (1, 1, 8, 256, 9), (1, 1, 12, 256, 9), (1, 1, 11, 257, 9),          # 256 and 512 threads
    (1, 3, 5, 60, 3), (1, 3, 9, 64, 3), (1, 2, 33, 65, 3), (1, 2, 48, 64, 3),      # groups of keys in 256 and 512 threads
    (1, 1, 32, 257, 40), (1, 1, 16, 512, 40), (2, 1, 17, 512, 40),     # 512 and 1024 by the mass
    (1, 1, 1, 513, 40), (1, 257, 1, 513, 5),                            # 1024 by the rows, unless there are many plans
    (4, 128, 5, 1700, 5), (4, 129, 5, 1700, 5),                         # ... and by the mass
    (8, 80, 2, 50, 8),
])
def test_plans_of_a_whole_step(L, B, H, n, drop):
    plans_of_a_step(L, B, H, n, drop, ties=L == 1, fixed_tail=True)


@pytest.mark.parametrize("B,H,n,drop", [(1, 2, 16, 8), (3, 9, 64, 5), (1, 33, 128, 40), (1, 32, 300, 3), (1, 3, 600, 40), (300, 2, 520, 3),
                                        (700, 2, 30, 2), (2, 8, 256, 100)])
@pytest.mark.parametrize("dtype", [BF, F32])
def test_one_layer_calls(B, H, n, drop, dtype):
    """st3_decode_layer_step and st3_select_compact_layer against the whole-step call over that layer.  (Whole strips or not, rows
    that a plan moves itself or not: what stays behind the kept rows may differ, what is kept may not.)"""
    args = dict(L=1, B=B, H=H, d=64, dtype=dtype, vis=[n], tail=5, drop=drop)
    a, b, c = Step(**args).whole(), Step(**args), Step(**args)
    s, e = b.state[0], b.arr[0]
    q, kn, vn = b.qkv[0]
    st3.st3_decode_layer_step(b.shape, e.kv, e.seg, s["score"], s["ids"], n - drop, MODE, q, kn, vn, b.out[0], s["mass"], s["ws"])
    c.arr[0].keep_after = -1                    # attend only, then the eviction as a call of its own
    c.whole()
    t = c.state[0]
    seg = st3.segments(3, n, 3 + n + 5 + 1, t["vis_len"], t["kv_len"], t["tail"])
    st3.st3_select_compact_layer(c.shape, c.arr[0].kv, seg, t["score"], t["ids"], n - drop, MODE, t["ws"])
    torch.cuda.synchronize()
    k = n - drop
    for x in (b, c):
        for st in (x.state[0], a.state[0]):
            st["score"][:, k:], st["ids"][:, k:] = 0, 0
            st["k"][:, :, 3 + k:3 + n], st["v"][:, :, 3 + k:3 + n] = 0, 0
        x.out.copy_(a.out)                      # (the attention's, cut into other chunks: not what this is about)
        _same(a, x)
