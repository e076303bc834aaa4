"""The whole-step call serves many layers per launch: it must do what the same layers do one call at a time
(st3_decode_layer_attend for each, then st3_decode_plans), at the edges of what a launch holds and of the rules that
choose chunks and stores, and fall back to one launch per layer where layers share rows."""
import pytest
import torch

from paper_2412_20105_amd import binding as st3

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
MODE = st3.ST3_HOLE_FILL


class Step:
    """One step's buffers; two objects of equal arguments hold equal values.  e4m3: True, or the layers whose caches are E4M3."""

    def __init__(self, L, B, H, d, dtype, vis, tail, lazy=None, fixed_tail=True, e4m3=False, drop=2):
        g = torch.Generator(device=DEV).manual_seed(L * 1009 + B * 31 + H)
        rnd = lambda *s: torch.randn(s, generator=g, device=DEV)  # noqa: E731
        self.shape = st3.make_shape(B, H, d, st3.ST3_F32 if dtype == torch.float32 else st3.ST3_BF16)
        self.L, self.lazy = L, dict(lazy or {})
        self.out = torch.zeros((L, B, H, d), dtype=dtype, device=DEV)
        self.qkv = rnd(L, 3, B, H, d).to(dtype)
        self.arr = (st3.LayerStep * L)()
        self.state, self.refs = [], []
        one = B * H * d * self.out.element_size()
        for l in range(L):
            src = self.lazy.get(l)
            n = vis[l % len(vis)] if src is None else self.state[src]["n"]
            rows = 3 + n + tail
            cap = rows + 5 + l % 3
            coded = e4m3 if isinstance(e4m3, bool) else l in e4m3
            scale = torch.full((B, H), 0.01, dtype=torch.float32, device=DEV) if coded else None

            def cache():
                x = rnd(B, H, cap, d)
                return (x * 50).to(torch.float8_e4m3fn).view(torch.uint8) if coded else x.to(dtype)

            k, v = None if src is not None else cache(), cache()
            s = {"n": n, "k": k, "v": v, "kv_len": torch.full((B,), rows, dtype=torch.int32, device=DEV),
                 "vis_len": torch.full((B,), n, dtype=torch.int32, device=DEV),
                 "tail": torch.full((B,), 3 + n, dtype=torch.int32, device=DEV) if fixed_tail else None,
                 "mass": torch.zeros((B, max(n, 1)), dtype=torch.float32, device=DEV)}
            if src is None:
                s["score"] = torch.rand((B, max(n, 1)), generator=g, device=DEV)
                s["ids"] = torch.rand((B, max(n, 1)), generator=g, device=DEV).argsort(dim=1).to(torch.int32)
            else:
                s["score"], s["ids"] = self.state[src]["score"].clone(), self.state[src]["ids"].clone()
            s["ws"] = torch.empty((st3.st3_workspace_bytes(self.shape, cap, n, 1),), dtype=torch.uint8, device=DEV)
            st3.st3_workspace_init(self.shape, cap, s["ws"])
            kv = st3.kv_layer(k, v, None if k is None else scale, scale)
            seg = st3.segments(3, n, rows, s["vis_len"], s["kv_len"], s["tail"], n, 3 + n if fixed_tail else 0)
            self.refs += [kv, seg, scale]
            e = self.arr[l]
            e.kv, e.seg = kv, seg
            e.score_col, e.id_col, e.col_stride = s["score"].data_ptr(), s["ids"].data_ptr(), s["score"].stride(0)
            e.keep_after = n - drop if n > drop else -1
            e.inherit_from = -1 if src is None else src
            e.q, e.k_new, e.v_new = (self.qkv.data_ptr() + (3 * l + i) * one for i in range(3))
            e.out, e.vis_mass, e.mass_stride = self.out[l].data_ptr(), s["mass"].data_ptr(), s["mass"].stride(0)
            e.workspace, e.workspace_bytes = s["ws"].data_ptr(), s["ws"].numel()
            self.state.append(s)

    def whole(self):
        st3.st3_decode_step(self.shape, self.arr, self.L, MODE)
        torch.cuda.synchronize()
        return self

    def layer_by_layer(self):
        for l in range(self.L):
            st3.st3_decode_layer_attend(self.shape, self.arr, self.L, l, MODE)
        st3.st3_decode_plans(self.shape, self.arr, self.L, MODE)
        torch.cuda.synchronize()
        return self


def _same(a, b):
    # Both add the same float32 products, cut into other chunks: an output differs by a few roundings of a sum whose
    # terms are at most max|v| <= 6 in all (weights add to 1), i.e. 1e-5; a bf16 output then by one step more, to the next
    # number of 8 significant bits: at most 2^-7 of the value (two sums on either side of a rounding boundary).
    x, y = a.out.double(), b.out.double()
    step = 2.0 ** -7 if a.out.dtype == torch.bfloat16 else 0.0
    assert bool(((x - y).abs() <= 1e-5 + step * y.abs()).all()), float((x - y).abs().max())
    for l, (s, t) in enumerate(zip(a.state, b.state)):
        # masses: probabilities, relative error of a float32 exponent and normaliser
        assert torch.allclose(s["mass"], t["mass"], rtol=5e-5, atol=1e-9), l
        for name in ("ids", "score", "kv_len", "vis_len", "k", "v"):
            if s[name] is not None:
                assert torch.equal(s[name], t[name]), (l, name)


BF, F32 = torch.bfloat16, torch.float32


@pytest.mark.parametrize("args", [
    dict(L=1, B=1, H=1, d=64, dtype=F32, vis=[5], tail=0),
    dict(L=2, B=3, H=5, d=64, dtype=BF, vis=[0, 300], tail=1),                  # a layer without visual rows
    dict(L=21, B=1, H=3, d=128, dtype=BF, vis=[130, 65, 64], tail=33),
    dict(L=22, B=2, H=2, d=128, dtype=BF, vis=[700, 31, 1], tail=7),            # strips cut unevenly
    dict(L=65, B=1, H=2, d=64, dtype=F32, vis=[40, 39], tail=2),                # two launches of either kind
    dict(L=9, B=16, H=40, d=128, dtype=F32, vis=[20], tail=3),                  # rows written past the caches (8.8 MB)
    dict(L=24, B=1, H=4, d=128, dtype=BF, vis=[500], tail=40, lazy={5: 4, 6: 4, 7: 4, 23: 22}),     # lazy strips cut too
    dict(L=4, B=2, H=4, d=128, dtype=BF, vis=[260, 90], tail=40, lazy={1: 0}, fixed_tail=False),
    dict(L=5, B=2, H=6, d=128, dtype=BF, vis=[200, 33], tail=9, e4m3=True, lazy={3: 2}),
    dict(L=3, B=2, H=4, d=128, dtype=BF, vis=[300], tail=9, drop=80),           # more moves than a plan's list holds
    dict(L=3, B=2, H=4, d=128, dtype=BF, vis=[300], tail=9, drop=80, fixed_tail=False),         # evictions by launches of their own
    dict(L=2, B=1, H=2, d=64, dtype=F32, vis=[8190], tail=3000),                # long strips: 59 chunks
    dict(L=35, B=1, H=3, d=128, dtype=BF, vis=[130, 65, 64], tail=33),          # one full attention launch, and two
    dict(L=36, B=1, H=3, d=128, dtype=BF, vis=[130, 65, 64], tail=33),
    dict(L=32, B=2, H=2, d=64, dtype=BF, vis=[70], tail=3, e4m3=True),          # the same with E4M3 caches
    dict(L=33, B=2, H=2, d=64, dtype=BF, vis=[70], tail=3, e4m3=True),
    dict(L=41, B=1, H=2, d=64, dtype=F32, vis=[40], tail=2),                    # one full launch behind the attention, and two
    dict(L=42, B=1, H=2, d=64, dtype=F32, vis=[40], tail=2),
], ids=lambda a: "-".join(f"{k}{v}" for k, v in a.items() if k in ("L", "B", "H", "d", "drop", "e4m3")))
def test_whole_step_is_the_layers_one_by_one(args):
    _same(Step(**args).whole(), Step(**args).layer_by_layer())


@pytest.mark.parametrize("args", [
    dict(L=1, B=1, H=1, d=64, dtype=F32, vis=[4000], tail=92),                  # 64 chunks, a lane of the wave for each
    dict(L=1, B=42, H=50, d=64, dtype=F32, vis=[4150], tail=20),                # cut for the logit staging area alone
], ids=["64_chunks", "staging"])
def test_cuts_of_long_strips(args):
    _same(Step(**args).whole(), Step(**args).layer_by_layer())


@pytest.mark.parametrize("field", ["q", "k_new", "v_new"])
def test_layers_that_read_an_earlier_layers_output(field):
    """Layer 2's token comes from layer 0's output buffer: in order, it is what layer 0 has just written (B * H = 600: no
    strip is cut in either form, so layer by layer the output is there)."""
    args = dict(L=3, B=20, H=30, d=64, dtype=BF, vis=[40], tail=5)
    a, b = Step(**args), Step(**args)
    for s in (a, b):
        setattr(s.arr[2], field, s.out[0].data_ptr())
    _same(a.whole(), b.layer_by_layer())


def test_layers_that_share_an_output_buffer():
    args = dict(L=3, B=20, H=30, d=64, dtype=BF, vis=[40], tail=5)
    a, b = Step(**args), Step(**args)
    for s in (a, b):
        s.arr[2].out = s.arr[0].out
    _same(a.whole(), b.layer_by_layer())


@pytest.mark.parametrize("L,B,H,n,drop,ties,fixed_tail", [
    (1, 1, 1, 1, 1, False, True),               # the last visual row goes
    (2, 2, 5, 128, 3, True, True),              # the smaller workgroup's bound, heads that fill no group
    (2, 2, 33, 129, 48, False, True),
    (3, 1, 4, 256, 40, True, False),            # thread groups of the mass: 256, 257, 512, 513, 1024, 1025 rows
    (3, 1, 3, 257, 2, False, True),
    (2, 1, 7, 512, 49, False, True),            # one row more than the plan moves by itself
    (2, 3, 6, 513, 5, True, True),
    (2, 1, 9, 1024, 30, False, False),
    (2, 1, 2, 1025, 1024, True, True),
    (1, 2, 2, 8192, 20, False, True),           # the most rows a plan ranks
    (8, 65, 2, 40, 7, True, True),              # more plans than 512
])
def test_plan_keeps_the_best_rows_and_finishes_the_mass(L, B, H, n, drop, ties, fixed_tail):
    s = Step(L=L, B=B, H=H, d=64, dtype=F32, vis=[n], tail=6, fixed_tail=fixed_tail, drop=0)
    k = n - drop
    before = []
    for l, st in enumerate(s.state):
        s.arr[l].keep_after = k
        if ties:        # a few values only: the k-th score is shared
            st["score"].copy_((st["score"] * 4).floor() / 4)
        before.append({x: st[x].clone() for x in ("k", "v", "score", "ids")})
    s.whole()
    for l, (st, was) in enumerate(zip(s.state, before)):
        rows = 3 + n + 6
        q, kn, _ = s.qkv[l].double()
        keys = torch.cat([was["k"][:, :, :rows].double(), kn[:, :, None]], dim=2)
        p = torch.softmax(torch.matmul(keys, q[..., None])[..., 0] / 8.0, dim=-1)
        # float32 exponent of a logit good to 1e-6, normaliser and a sum over heads (as for every mass)
        assert torch.allclose(st["mass"].double(), p[:, :, 3:3 + n].mean(dim=1), rtol=5e-5, atol=1e-9), l
        assert st["vis_len"].tolist() == [k] * B and st["kv_len"].tolist() == [rows + 1 - (0 if fixed_tail else drop)] * B
        for b in range(B):
            sc, ids = was["score"][b].tolist(), was["ids"][b].tolist()
            best = sorted(range(n), key=lambda i: (-sc[i], ids[i]))[:k]
            got = st["ids"][b, :k].tolist()
            assert sorted(got) == sorted(ids[i] for i in best), (l, b)
            at = {ids[i]: i for i in range(n)}
            src = torch.tensor([at[i] for i in got], dtype=torch.long, device=DEV)
            assert torch.equal(st["score"][b, :k], was["score"][b][src]), (l, b)
            for x in ("k", "v"):
                assert torch.equal(st[x][b, :, 3:3 + k], was[x][b][:, 3 + src]), (l, b, x)
