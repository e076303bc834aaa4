"""The two calls that serve a prune event and the start of decoding in one launch: kept columns, and the evictions of many layers."""
import pytest
import torch

from paper_2412_20105_amd import binding as st3
from test_gpu_step_launches import BF, DEV, F32, MODE, Step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,n,k,ties", [(1, 1, 1, False), (3, 300, 300, False), (3, 300, 1, True), (5, 257, 100, True),
                                           (2, 1025, 1000, False), (2, 8193, 4000, True)])
def test_select_columns(rows, n, k, ties):
    g = torch.Generator(device=DEV).manual_seed(rows + n)
    score = torch.rand((rows, n + 3), generator=g, device=DEV)
    if ties:
        score = (score * 8).floor()
    ids = torch.rand((rows, n + 5), generator=g, device=DEV).argsort(dim=1).to(torch.int32)
    out_s = torch.full((rows, k + 2), -1.0, device=DEV)
    out_i = torch.full((rows, k + 4), -1, dtype=torch.int32, device=DEV)
    st3.st3_select_columns(score, ids, n, k, out_s, out_i)
    s, i = score[:, :n], ids[:, :n]
    by_id = i.long().argsort(dim=1)             # (score descending, id ascending)
    pos = by_id.gather(1, s.gather(1, by_id).argsort(dim=1, descending=True, stable=True))[:, :k].sort(dim=1)[0]
    assert torch.equal(out_s[:, :k], s.gather(1, pos)) and torch.equal(out_i[:, :k], i.gather(1, pos))
    assert bool((out_s[:, k:] == -1).all()) and bool((out_i[:, k:] == -1).all())
    with pytest.raises(st3.St3Error):
        st3.st3_select_columns(score, ids, n, k, score, out_i)


@pytest.mark.parametrize("layout", ["outputs", "all"])
def test_rows_of_one_buffer_alternate(layout):
    """Scores and ids of a row side by side: rows of outputs lie between rows of outputs, or of inputs, without touching them."""
    rows, n, k = 5, 70, 40
    g = torch.Generator(device=DEV).manual_seed(9)
    score, ids = torch.rand((rows, n), generator=g, device=DEV), torch.rand((rows, n), generator=g, device=DEV).argsort(dim=1).to(torch.int32)
    want_s, want_i = torch.empty((rows, k), device=DEV), torch.empty((rows, k), dtype=torch.int32, device=DEV)
    st3.st3_select_columns(score, ids, n, k, want_s, want_i)
    buf = torch.zeros((rows, 2 * n + 2 * k), device=DEV)
    out_s, out_i = buf[:, 2 * n:2 * n + k], buf[:, 2 * n + k:].view(torch.int32)
    if layout == "all":
        buf[:, :n], buf[:, n:2 * n].view(torch.int32)[:] = score, ids
        score, ids = buf[:, :n], buf[:, n:2 * n].view(torch.int32)
    st3.st3_select_columns(score, ids, n, k, out_s, out_i)
    assert torch.equal(out_s, want_s) and torch.equal(out_i, want_i)


@pytest.mark.parametrize("mode", [st3.ST3_STABLE, MODE])
@pytest.mark.parametrize("args", [
    dict(L=35, B=2, H=3, d=64, dtype=BF, vis=[60, 9], tail=4, drop=5),                      # three launches
    dict(L=3, B=1, H=5, d=128, dtype=F32, vis=[400], tail=4, drop=120, lazy={1: 0}),
    dict(L=2, B=3, H=2, d=64, dtype=BF, vis=[130], tail=40, drop=48, fixed_tail=False, e4m3={0}),
], ids=["many", "large", "closing_tail"])
def test_evictions_of_many_layers(args, mode):
    a, b = Step(**args), Step(**args)
    for l in range(0, a.L, 3):
        a.arr[l].keep_after = -1
    st3.st3_select_compact_layers(a.shape, a.arr, a.L, mode)
    for l, (st, e) in enumerate(zip(b.state, b.arr)):
        if l % 3:
            st3.st3_select_compact_layer(b.shape, e.kv, e.seg, st["score"], st["ids"], e.keep_after, mode, st["ws"])
    torch.cuda.synchronize()
    for l, (s, t) in enumerate(zip(a.state, b.state)):
        n = s["n"]
        k = n if l % 3 == 0 else n - args["drop"]
        assert torch.equal(s["vis_len"], t["vis_len"]) and torch.equal(s["kv_len"], t["kv_len"])
        assert s["vis_len"].tolist() == [k] * args["B"]
        end = int(s["kv_len"][0])
        for x in ("score", "ids"):
            assert torch.equal(s[x][:, :k], t[x][:, :k]), (l, x)
        for x in ("k", "v"):
            if s[x] is not None:
                assert torch.equal(s[x][:, :, :3 + k], t[x][:, :, :3 + k]), (l, x)
                assert torch.equal(s[x][:, :, 3 + n if args.get("fixed_tail", True) else 3 + k:end], t[x][:, :, 3 + n if args.get("fixed_tail", True) else 3 + k:end]), (l, x)
