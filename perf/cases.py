"""What this library's users have it do, as cases that can be timed and compared.

The library is the attention and visual-token-trimming path of a LLaVA-style decoder: a prompt of
[system | visual | instruction] tokens is prefilled layer by layer while visual tokens are pruned from layer to
layer, then tokens are decoded against caches whose visual segment keeps shrinking.  A serving program
therefore spends its time in five places, and each is a kind of case here:

  step     one decode step over all layers (st3_decode_step): append, attend, mass, evict
  layers   the same step called layer by layer (st3_decode_layer_attend, st3_decode_plans), the form a
           decoder whose layers depend on each other uses
  attend   one stand-alone decode attention over a ragged batch (st3_decode_attention[_noalloc])
  prefill  the causal attention of one layer's prompt with the visual mass of its last rows
  prune    a prune event at prefill: top-k by mass, compaction of the columns, gather of Q, K and V
  job      a whole generation through pipeline.Generation: prefill of all layers, then decode steps

Sizes are the repository's own shapes (workloads/configs.py): 4 heads of 64 in float32 with 64 visual tokens,
7B (32 layers, 32 heads of 128), 13B (40 layers, 40 heads of 128), 576 visual tokens for one image and 2880 for
a high-resolution one.  Values are what those workloads draw: N(0, sigma^2), sigma = 0.02 sqrt(heads * dim).
"""
from __future__ import annotations

import math

import torch

DEV = "cuda:0"


# ---------------------------------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------------------------------
def _model(layers, heads, dim, dtype="bf16", sys=35, vis=576, txt=64):
    return {"layers": layers, "heads": heads, "dim": dim, "dtype": dtype, "sys": sys, "vis": vis, "txt": txt}


_TINY = _model(2, 4, 64, "f32", 8, 64, 16)
_7B = _model(32, 32, 128, txt=64)
_13B = _model(40, 40, 128, txt=128)
_HR = _model(32, 32, 128, sys=0, vis=2880, txt=256)


def _step(name, model, batch, steps, at, tau, end=0.1, cache="plain", lazy=False, kind="step"):
    return {"name": name, "kind": kind, **model, "batch": batch, "steps": steps, "at": at, "tau": tau, "end": end,
            "cache": cache, "lazy": lazy}


def listed():
    return [
        # the smallest thing there is: two layers in float32, a few kilobytes; all latency
        _step("step_tiny_f32_b1", _TINY, 1, 8, 3, 8, end=0.5),
        # one user, one image, interactive: the latency of a token, half way through the answer
        _step("step_7b_b1", _7B, 1, 256, 128, 256),
        # a small batch under the paper's fast annealing (tau = 50: many rows evicted per step), the last layers in
        # groups that inherit their source layer's attention
        _step("step_13b_b8_lazy_evict", _13B, 8, 512, 12, 50, lazy=True),
        # the serving batch this repository's benchmark runs, half way through the answer
        _step("step_13b_b32", _13B, 32, 512, 256, 512),
        # a high-resolution image with 8-bit caches
        _step("step_hr_b8_e4m3", _HR, 8, 256, 64, 256, end=0.05, cache="e4m3"),
        # a decoder that needs a layer's output before it can form the next layer's query
        _step("layers_7b_b16", _7B, 16, 256, 100, 256, kind="layers"),
        # one layer's attention for a ragged batch (requests of different age and image size), contiguous caches
        {"name": "attend_13b_ragged_b5", "kind": "attend", "heads": 40, "dim": 128, "dtype": "bf16", "cache": "plain",
         "batch": 5, "sys": 35, "vis": 576, "shortest": 173, "longest": 1111, "entry": "workspace"},
        # first layer of the benchmark's batch: 739 prompt tokens, no multiple of any tile
        {"name": "prefill_13b_b32", "kind": "prefill", "heads": 40, "dim": 128, "dtype": "bf16", "batch": 32, "sys": 35,
         "vis": 576, "txt": 128, "window": 1},
        # the largest prompt: a tiled high-resolution image, batch 8
        {"name": "prefill_hr_b8", "kind": "prefill", "heads": 32, "dim": 128, "dtype": "bf16", "batch": 8, "sys": 0,
         "vis": 2880, "txt": 256, "window": 1},
        # a late, well pruned layer for a single user: little work, few workgroups
        {"name": "prefill_7b_b1_pruned", "kind": "prefill", "heads": 32, "dim": 128, "dtype": "bf16", "batch": 1, "sys": 35,
         "vis": 211, "txt": 64, "window": 1},
        # a prune event in the middle of a prefill
        {"name": "prune_13b_b8", "kind": "prune", "heads": 40, "dim": 128, "dtype": "bf16", "batch": 8, "sys": 35, "vis": 576,
         "txt": 128, "alive": 365, "keep": 350},
        # a whole short answer for four users: prefill of every layer and 16 decode steps under fast annealing
        {"name": "job_7b_b4", "kind": "job", **_7B, "batch": 4, "steps": 16, "tau": 50, "end": 0.1},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "layers", "attend", "prefill", "prefill", "prune"])
    f32 = rng.random() < 0.15
    dim = 64 if f32 and rng.random() < 0.5 else rng.choice([128, 128, 128, 64])
    heads = _log(rng, 4, 16) if f32 else rng.choice([8, 12, 16, 20, 32, 32, 40, 40])
    dtype = "f32" if f32 else "bf16"
    if kind in ("step", "layers"):
        hr = rng.random() < 0.2
        vis = _log(rng, 1500, 2880) if hr else _log(rng, 48, 640)
        batch = _log(rng, 1, 8 if hr else 32)
        steps = _log(rng, 16, 512)
        model = _model(_log(rng, 2, 32 if hr else 40), heads, dim, dtype, rng.randint(0, 48), vis, _log(rng, 5, 256))
        c = _step("", model, batch, steps, rng.randint(1, max(1, steps - 1)), rng.choice([50, 128, steps + 1, 2 * steps]),
                  end=rng.choice([0.05, 0.1, 0.5, 1.0]), cache="e4m3" if not f32 and rng.random() < 0.3 else "plain",
                  lazy=kind == "step" and model["layers"] >= 8 and rng.random() < 0.3, kind=kind)
        del c["name"]
        return c
    if kind == "attend":
        longest = _log(rng, 64, 3300)
        vis = rng.randint(0, longest // 2)
        return {"kind": kind, "heads": heads, "dim": dim, "dtype": dtype, "cache": "e4m3" if not f32 and rng.random() < 0.3 else "plain",
                "batch": _log(rng, 1, 24), "sys": rng.randint(0, min(48, longest // 4)), "vis": vis,
                "shortest": rng.randint(1, longest), "longest": longest, "entry": rng.choice(["workspace", "noalloc"])}
    if kind == "prefill":
        if f32:     # the small float32 models that checks are run with
            return {"kind": kind, "heads": heads, "dim": dim, "dtype": dtype, "batch": rng.randint(1, 4), "sys": rng.randint(0, 16),
                    "vis": _log(rng, 16, 200), "txt": _log(rng, 1, 40), "window": rng.choice([1, 1, 4])}
        vis = _log(rng, 30, 2880)
        most = max(1, min(32, int(8 * (3136 / (vis + 100)) ** 2)))
        return {"kind": kind, "heads": heads, "dim": dim, "dtype": dtype, "batch": _log(rng, 1, most), "sys": rng.randint(0, 48),
                "vis": vis, "txt": _log(rng, 5, 250), "window": rng.choice([1, 1, 1, 4, 16])}
    vis = _log(rng, 64, 2880)
    alive = rng.randint(max(2, vis // 8), vis)
    return {"kind": kind, "heads": heads, "dim": dim, "dtype": dtype, "batch": _log(rng, 1, 4 if vis > 700 else 16),
            "sys": rng.randint(0, 48), "vis": vis, "txt": _log(rng, 5, 250), "alive": alive,
            "keep": rng.randint(1, alive - 1)}


# ---------------------------------------------------------------------------------------------------
# inputs (plain torch, from the seed alone)
# ---------------------------------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 17)


def _dt(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


def _eb(c):
    return 4 if c["dtype"] == "f32" else 2


def _sigma(c):
    return 1.0 if c["dtype"] == "f32" else 0.02 * math.sqrt(c["heads"] * c["dim"])


def _randn(g, c, *shape, into=None):
    t = torch.empty(shape, dtype=_dt(c), device=DEV) if into is None else into
    return t.normal_(0.0, _sigma(c), generator=g)


def _cache_rows(g, c, *shape):
    """Cached rows in the cache's own format."""
    if c["cache"] == "plain":
        return _randn(g, c, *shape)
    out = torch.empty(shape, dtype=torch.uint8, device=DEV)
    for i in range(shape[0]):       # codes of N(0, sigma^2) at 6 sigma / 448 per unit
        x = torch.empty(shape[1:], dtype=torch.float32, device=DEV).normal_(0.0, 448.0 / 6.0, generator=g)
        out[i] = x.clamp_(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)
    return out


def _unit(c):
    return 6.0 * _sigma(c) / 448.0


def _masses(g, B, n):
    """Scores as attention leaves them: positive, a few large, most small."""
    x = torch.empty((B, n), dtype=torch.float32, device=DEV).normal_(0.0, 1.5, generator=g)
    return torch.softmax(x, dim=-1) * 0.8


def _ids(g, B, n_all, n):
    """n distinct original token ids per sequence, in the order evictions have left them."""
    return torch.rand((B, n_all), generator=g, device=DEV).argsort(dim=-1)[:, :n].to(torch.int32)


def _keep0(c):
    """Visual tokens per layer after the prefill: all of them in the first three layers, then fewer, linearly."""
    L, vis = c["layers"], c["vis"]
    first = 2 if L > 3 else 0
    keep = [vis if l <= first else int(vis * (1.0 - (1.0 - c["end"]) * (l - first) / max(1, L - 1 - first))) for l in range(L)]
    src = _sources(c)
    return [keep[s] if s >= 0 else k for k, s in zip(keep, src)]


def _sources(c):
    """Source layer of each lazy layer (-1: an ordinary layer): the last layers in groups of four."""
    L = c["layers"]
    src = [-1] * L
    if c.get("lazy"):
        for first in range(L - 4 * max(1, int(0.3 * L) // 4), L, 4):
            for l in range(first + 1, first + 4):
                src[l] = first
    return src


def _keep_at(c, t):
    """Visual rows per layer during decode step t (cosine annealing)."""
    beta = 0.5 * (1.0 + math.cos(math.pi * min(t, c["tau"]) / c["tau"]))
    return [int(k * beta + 1e-9) for k in _keep0(c)]


class _StepInputs:
    pass


def _step_inputs(c, seed):
    """The state of a batch right before decode step `at`: per layer a cache in the fixed-tail layout (visual rows
    shrink in place, instruction and generated rows stay where the prefill put them), its ranking columns and lengths."""
    g = _gen(seed)
    s = _StepInputs()
    L, B, H, d, vis, t = c["layers"], c["batch"], c["heads"], c["dim"], c["vis"], c["at"]
    s.src, s.keep0, s.now, s.next = _sources(c), _keep0(c), _keep_at(c, t), _keep_at(c, t + 1)
    s.cap = [max(c["sys"] + k0 + c["txt"] + c["steps"], c["sys"] + vis + c["txt"]) for k0 in s.keep0]
    s.tail = [c["sys"] + k0 for k0 in s.keep0]
    s.rows = [ts + c["txt"] + t - 1 for ts in s.tail]           # rows stored before this step's token
    # lengths and columns of all layers side by side in one buffer
    s.saved = torch.zeros((L * (2 * B + 2 * B * vis),), dtype=torch.int32, device=DEV)
    kv_len, vis_len, score, ids = _live_views(s.saved, L, B, vis)
    s.k, s.v = [], []
    per_unit = 1 if c["cache"] == "e4m3" else _eb(c)
    for l in range(L):
        n, k = s.now[l], s.next[l]
        kv_len[l], vis_len[l] = s.rows[l], n
        if s.src[l] >= 0:           # a lazy layer ranks by copies of its source's columns and caches values only
            score[l], ids[l] = score[s.src[l]], ids[s.src[l]]
        elif n > 0:
            score[l, :, :n], ids[l, :, :n] = _masses(g, B, n), _ids(g, B, vis, n)
        s.k.append(None if s.src[l] >= 0 else _cache_rows(g, c, B, H, s.cap[l], d))
        s.v.append(_cache_rows(g, c, B, H, s.cap[l], d))
        if 0 < k < n:
            # A pass starts from the same lengths and columns each time, while the rows that the eviction moves
            # inside the caches stay moved: the holes hold the rows that fill them from the start, so that every
            # pass (the first included) meets the same caches and moves the same rows.
            dst, srcp = _fills(score[l, :, :n], ids[l, :, :n], k, c["sys"], s.cap[l] - 1)
            for x in (s.k[l], s.v[l]):
                if x is not None:
                    at = lambda i: i[:, None, :, None].expand(B, H, i.shape[1], d)  # noqa: E731
                    x.scatter_(2, at(dst), x.gather(2, at(srcp)))
    s.qkv = _randn(g, c, L, 3, B, H, d)
    s.per_unit = per_unit
    return s


def _live_views(buf, L, B, vis):
    kv_len = buf[:L * B].view(L, B)
    vis_len = buf[L * B:2 * L * B].view(L, B)
    cols = buf[2 * L * B:].view(2, L, B, vis)
    return kv_len, vis_len, cols[0].view(torch.float32), cols[1]


def _fills(score, ids, k, first_row, spare_row):
    """Rows (dst, src) [B, n - k] of an eviction to k: the i-th hole among the first k positions is filled from the
    i-th survivor behind them; pairs that do not exist name a row nobody uses."""
    B, n = score.shape
    by_id = ids.argsort(dim=-1)
    order = by_id.gather(1, score.gather(1, by_id).argsort(dim=-1, descending=True, stable=True))
    kept = torch.zeros((B, n), dtype=torch.bool, device=DEV).scatter_(1, order[:, :k], True)
    pos = torch.arange(n, device=DEV).expand(B, n)
    none = torch.full_like(pos, n)
    dst = torch.where((pos < k) & ~kept, pos, none).sort(dim=-1)[0][:, :n - k]
    src = torch.where((pos >= k) & kept, pos, none).sort(dim=-1)[0][:, :n - k]
    real = dst < n
    spare = torch.full_like(dst, spare_row)
    return torch.where(real, dst + first_row, spare), torch.where(real, src + first_row, spare)


def _attend_inputs(c, seed):
    g = _gen(seed)
    s = _StepInputs()
    B, H, d = c["batch"], c["heads"], c["dim"]
    r = torch.Generator().manual_seed(int(seed) * 31 + 5)
    lens = torch.randint(c["shortest"], c["longest"] + 1, (B,), generator=r)
    lens[-1] = c["longest"]
    room = (lens - c["sys"]).clamp(min=0)
    s.nvis = torch.minimum((torch.rand((B,), generator=r) * (c["vis"] + 1)).long(), room)
    s.nvis[-1] = min(c["vis"], int(room[-1]))
    s.lens = lens
    s.cap = c["longest"] + 64
    s.k, s.v = _cache_rows(g, c, B, H, s.cap, d), _cache_rows(g, c, B, H, s.cap, d)
    s.q = _randn(g, c, B, H, d)
    return s


def _prefill_inputs(c, seed):
    """Queries in a buffer of their own; keys and values already in the layer's cache, as a prefill leaves them."""
    g = _gen(seed)
    s = _StepInputs()
    B, H, d = c["batch"], c["heads"], c["dim"]
    s.n = c["sys"] + c["vis"] + c["txt"]
    s.cap = s.n + 96
    s.q = _randn(g, c, B, H, s.n, d)
    s.k, s.v = _randn(g, c, B, H, s.cap, d), _randn(g, c, B, H, s.cap, d)
    return s


def _prune_inputs(c, seed):
    """The layer's input rows by original token id, the previous layer's mass, and which tokens are alive."""
    g = _gen(seed)
    s = _StepInputs()
    B, H, d, alive = c["batch"], c["heads"], c["dim"], c["alive"]
    n0 = c["sys"] + c["vis"] + c["txt"]
    s.qkv = [_randn(g, c, B, H, n0, d) for _ in range(3)]
    s.mass = torch.zeros((B, c["vis"]), dtype=torch.float32, device=DEV)
    s.mass[:, :alive] = _masses(g, B, alive)
    s.ids = torch.zeros((B, c["vis"]), dtype=torch.int32, device=DEV)
    s.ids[:, :alive] = _ids(g, B, c["vis"], alive).sort(dim=-1)[0]
    return s


# ---------------------------------------------------------------------------------------------------
# what a program holds before the call
# ---------------------------------------------------------------------------------------------------
def prepare(case, seed):
    from paper_2412_20105_amd import binding as st3
    c = case
    kind = c["kind"]
    if kind == "job":
        return _prepare_job(c, seed)
    B, H, d = c["batch"], c["heads"], c["dim"]
    shape = st3.make_shape(B, H, d, st3.ST3_F32 if c["dtype"] == "f32" else st3.ST3_BF16)

    def scale():
        return torch.full((B, H), _unit(c), dtype=torch.float32, device=DEV) if c.get("cache") == "e4m3" else None

    if kind in ("step", "layers"):
        s = _step_inputs(c, seed)
        L, vis = c["layers"], c["vis"]
        s.live = s.saved.clone()
        s.kv_len, s.vis_len, s.score, s.ids = _live_views(s.live, L, B, vis)
        s.out = torch.zeros((L, B, H, d), dtype=_dt(c), device=DEV)
        s.mass = torch.zeros((L, B, vis), dtype=torch.float32, device=DEV)
        s.tail_dev = torch.tensor(s.tail, dtype=torch.int32, device=DEV)[:, None].expand(L, B).contiguous()
        s.scale = scale()
        s.ws, s.refs = [], []
        arr = (st3.LayerStep * L)()
        one = B * H * d * _eb(c)
        for l in range(L):
            e = arr[l]
            ws = torch.empty((st3.st3_workspace_bytes(shape, s.cap[l], vis, 1),), dtype=torch.uint8, device=DEV)
            st3.st3_workspace_init(shape, s.cap[l], ws)
            s.ws.append(ws)
            kv = st3.kv_layer(s.k[l], s.v[l], None if s.k[l] is None else s.scale, s.scale)
            seg = st3.segments(c["sys"], s.now[l], s.rows[l], s.vis_len[l], s.kv_len[l], s.tail_dev[l], s.now[l], s.tail[l])
            s.refs += [kv, seg]
            e.kv, e.seg = kv, seg
            e.score_col, e.id_col, e.col_stride = s.score[l].data_ptr(), s.ids[l].data_ptr(), vis
            e.keep_after = s.next[l] if s.next[l] < s.now[l] else -1
            e.inherit_from = s.src[l]
            base = s.qkv.data_ptr() + 3 * l * one
            e.q, e.k_new, e.v_new = base, base + one, base + 2 * one
            e.out, e.vis_mass, e.mass_stride = s.out[l].data_ptr(), s.mass[l].data_ptr(), vis
            e.workspace, e.workspace_bytes = ws.data_ptr(), ws.numel()
        s.arr, s.L, s.layerwise = arr, L, kind == "layers"
        held = [x for x in s.k + s.v if x is not None]
        s.caches = held if len(held) <= 48 and sum(x.numel() for x in held) < 1 << 26 else []
    elif kind == "attend":
        s = _attend_inputs(c, seed)
        s.kv_len, s.vis_len = s.lens.to(torch.int32).to(DEV), s.nvis.to(torch.int32).to(DEV)
        s.scale = scale()
        s.kv = st3.kv_layer(s.k, s.v, s.scale, s.scale)
        s.seg = st3.segments(c["sys"], int(s.nvis.max()), c["longest"], s.vis_len, s.kv_len)
        s.out = torch.zeros((B, H, d), dtype=_dt(c), device=DEV)
        s.mass = torch.zeros((B, max(1, c["vis"])), dtype=torch.float32, device=DEV)
        s.ws = None
        if c["entry"] == "workspace":
            s.ws = torch.empty((st3.st3_workspace_bytes(shape, s.cap, c["vis"], 1),), dtype=torch.uint8, device=DEV)
            st3.st3_workspace_init(shape, s.cap, s.ws)
    elif kind == "prefill":
        s = _prefill_inputs(c, seed)
        s.out = torch.empty_like(s.q)
        s.mass = torch.zeros((B, c["vis"]), dtype=torch.float32, device=DEV)
        s.ws = torch.empty((st3.st3_workspace_bytes(shape, s.cap, c["vis"], c["window"]),), dtype=torch.uint8, device=DEV)
        s.kn, s.vn = s.k[:, :, :s.n], s.v[:, :, :s.n]
    else:
        s = _prune_inputs(c, seed)
        rows = c["sys"] + c["keep"] + c["txt"]
        s.keep_idx = torch.empty((B, c["vis"]), dtype=torch.int32, device=DEV)
        s.new_ids, s.new_score = torch.zeros_like(s.ids), torch.zeros_like(s.mass)
        s.dst = [torch.empty((B, H, rows, d), dtype=_dt(c), device=DEV) for _ in range(3)]
        s.pairs = list(zip(s.qkv, s.dst))
    s.c, s.shape, s.st3 = c, shape, st3
    return s


def _prepare_job(c, seed):
    from paper_2412_20105_amd import pipeline
    g = _gen(seed)
    s = _StepInputs()
    L, B, H, d = c["layers"], c["batch"], c["heads"], c["dim"]
    n0 = c["sys"] + c["vis"] + c["txt"]
    table = [_keep_at(c, t) for t in range(c["steps"] + 1)]
    keep = [[table[t][l] for t in range(c["steps"] + 1)] for l in range(L)]
    s.gen = pipeline.Generation(L, H, d, _dt(c), B, c["sys"], c["vis"], c["txt"], c["steps"], keep, device=DEV)
    s.prompt = [[_randn(g, c, B, H, n0, d) for _ in range(3)] for _ in range(L)]
    s.tokens = [_randn(g, c, L, 3, B, H, d) for _ in range(c["steps"])]
    s.c = c
    return s


# ---------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------
def run(state):
    s, c = state, state.c
    kind = c["kind"]
    if kind == "job":
        for l, (q, k, v) in enumerate(s.prompt):
            s.gen.prefill_layer(l, q, k, v)
        for t, qkv in enumerate(s.tokens):
            out = s.gen.decode_step(t + 1, qkv)
        return {"out": out}
    st3 = s.st3
    if kind in ("step", "layers"):
        s.live.copy_(s.saved)           # lengths and columns as the previous step left them
        if s.layerwise:
            for l in range(s.L):
                st3.st3_decode_layer_attend(s.shape, s.arr, s.L, l, st3.ST3_HOLE_FILL)
            st3.st3_decode_plans(s.shape, s.arr, s.L, st3.ST3_HOLE_FILL)
        else:
            st3.st3_decode_step(s.shape, s.arr, s.L, st3.ST3_HOLE_FILL)
        return {"out": s.out, "mass": s.mass, "kv_len": s.kv_len, "vis_len": s.vis_len, "score": s.score, "ids": s.ids,
                "caches": s.caches}
    if kind == "attend":
        if s.ws is None:
            st3.st3_decode_attention_noalloc(s.shape, s.q, s.kv, s.seg, s.out, s.mass)
        else:
            st3.st3_decode_attention(s.shape, s.q, s.kv, s.seg, s.out, s.mass, s.ws)
        return {"out": s.out, "mass": s.mass}
    if kind == "prefill":
        st3.st3_prefill_attention(s.shape, s.q, s.kn, s.vn, s.n, c["sys"], c["vis"], c["window"], s.out, s.mass, s.ws)
        return {"out": s.out, "mass": s.mass}
    # prune: the launches of a prefill layer whose input loses visual tokens
    B, alive, keep = c["batch"], c["alive"], c["keep"]
    st3.st3_select_topk(s.mass, s.ids, None, alive, keep, None, s.keep_idx)
    for col, src in ((s.new_ids, s.ids), (s.new_score, s.mass)):
        col.copy_(src)
        st3.st3_compact_rows(col.data_ptr(), B, 1, col.stride(0) * 4, 0, 4, 4, s.keep_idx, keep, alive, 0)
    st3.st3_gather_rows(s.pairs, c["sys"], s.new_ids, keep, c["vis"], c["txt"])
    return {"ids": s.new_ids, "score": s.new_score, "q": s.dst[0], "k": s.dst[1], "v": s.dst[2]}


# ---------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------------
def _step_work(c, t, last=False):
    B, H, d, eb = c["batch"], c["heads"], c["dim"], _eb(c)
    cb = 1 if c.get("cache") == "e4m3" else eb
    now, nxt, src = _keep_at(c, t), _keep_at(c, t if last else t + 1), _sources(c)
    by = fl = 0
    for l in range(c["layers"]):
        rows = c["sys"] + now[l] + c["txt"] + t - 1         # cached rows attended
        halves = 1 if src[l] >= 0 else 2                    # K and V, or V alone
        by += B * H * d * (halves * rows * cb + halves * (eb + cb) + (3 - (src[l] >= 0)) * eb)
        by += 4 * B * now[l]                                # the mass
        fl += 2 * halves * B * H * d * (rows + 1)
        if 0 <= nxt[l] < now[l]:                            # ranking, and the rows that fill the holes
            gone = now[l] - nxt[l]
            by += 8 * B * now[l] + int(gone * nxt[l] / now[l]) * B * 2 * halves * H * d * cb
    return by, fl


def work(case):
    c = case
    B, H, d, eb = c["batch"], c["heads"], c["dim"], _eb(c)
    if c["kind"] in ("step", "layers"):
        by, fl = _step_work(c, c["at"])
    elif c["kind"] == "attend":
        cb = 1 if c["cache"] == "e4m3" else eb
        rows = (c["longest"] * (B + 1) + c["shortest"] * (B - 1)) // 2      # expected over the batch
        by = 2 * rows * H * d * cb + 2 * B * H * d * eb + 4 * B * c["vis"]
        fl = 4 * rows * H * d
    elif c["kind"] == "prefill":
        n = c["sys"] + c["vis"] + c["txt"]
        by, fl = 4 * B * H * n * d * eb + 4 * B * c["vis"], 4 * B * H * d * n * (n + 1) // 2
    elif c["kind"] == "prune":
        rows = c["sys"] + c["keep"] + c["txt"]
        by, fl = 6 * B * H * rows * d * eb + 8 * B * (c["alive"] + c["keep"]), B * c["alive"]
    else:
        by = fl = 0
        for k in _keep0(c):
            n = c["sys"] + k + c["txt"]
            by += (3 + 2 + 1) * B * H * n * d * eb          # Q, K, V read, K and V cached, the output written
            fl += 4 * B * H * d * n * (n + 1) // 2
        for t in range(1, c["steps"] + 1):
            b, f = _step_work(c, t, last=t == c["steps"])
            by, fl = by + b, fl + f
    return {"bytes": int(by), "flops": int(fl)}


def tolerance(case):
    if case["kind"] == "prune":
        return "exact"                  # rows are copied, tokens are picked by given scores
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    return {"rel": 1e-2}


# ---------------------------------------------------------------------------------------------------
# the same results in 64 bits
# ---------------------------------------------------------------------------------------------------
def _wide(c, x):
    """Cached rows as 64-bit values."""
    if c.get("cache") == "e4m3":
        return x.contiguous().view(torch.float8_e4m3fn).to(torch.float64) * float(torch.tensor(_unit(c), dtype=torch.float32))
    return x.to(torch.float64)


def _stored(c, x):
    """A new token's row as the cache will hold it."""
    if c.get("cache") != "e4m3":
        return x
    codes = (x.float() / torch.tensor(_unit(c), dtype=torch.float32, device=DEV)).clamp(-448.0, 448.0)
    return codes.to(torch.float8_e4m3fn).view(torch.uint8)


def exact(case, seed):
    c = case
    kind = c["kind"]
    root = 1.0 / math.sqrt(c["dim"])
    if kind == "job":
        return None     # which tokens survive hangs on near ties that 64 bits decide otherwise
    if kind in ("step", "layers"):
        s = _step_inputs(c, seed)
        L, B, H, d = c["layers"], c["batch"], c["heads"], c["dim"]
        out = torch.zeros((L, B, H, d), dtype=torch.float64, device=DEV)
        mass = torch.zeros((L, B, c["vis"]), dtype=torch.float64, device=DEV)
        kept = {}
        for l in range(L):
            n = s.now[l]
            rows = torch.cat([torch.arange(c["sys"] + n), torch.arange(s.tail[l], s.rows[l])]).to(DEV)

            def held(cache, new):
                return _wide(c, torch.cat([cache.index_select(2, rows), _stored(c, new)[:, :, None]], dim=2))

            q, kn, vn = s.qkv[l]
            if s.src[l] < 0:
                p = torch.softmax(torch.matmul(held(s.k[l], kn), q.double()[..., None])[..., 0] * root, dim=-1)
                if l in s.src:
                    kept[l] = p
            else:
                p = kept[s.src[l]]
            out[l] = torch.matmul(p[:, :, None], held(s.v[l], vn))[:, :, 0]
            mass[l, :, :n] = p[:, :, c["sys"]:c["sys"] + n].mean(dim=1)
            s.k[l] = s.v[l] = None
        return {"out": out, "mass": mass}
    if kind == "attend":
        s = _attend_inputs(c, seed)
        B = c["batch"]
        out = torch.zeros(s.q.shape, dtype=torch.float64, device=DEV)
        mass = torch.zeros((B, max(1, c["vis"])), dtype=torch.float64, device=DEV)
        for b in range(B):
            n, nv = int(s.lens[b]), int(s.nvis[b])
            p = torch.softmax(torch.matmul(_wide(c, s.k[b, :, :n]), s.q[b].double()[..., None])[..., 0] * root, dim=-1)
            out[b] = torch.matmul(p[:, None], _wide(c, s.v[b, :, :n]))[:, 0]
            mass[b, :nv] = p[:, c["sys"]:c["sys"] + nv].mean(dim=0)
        return {"out": out, "mass": mass}
    if kind == "prefill":
        s = _prefill_inputs(c, seed)
        n, W = s.n, c["window"]
        out = torch.empty(s.q.shape, dtype=torch.float64, device=DEV)
        mass = torch.zeros((c["batch"], c["vis"]), dtype=torch.float64, device=DEV)
        above = torch.ones((n, n), dtype=torch.bool, device=DEV).triu_(1)
        step = max(1, min(c["heads"], int(4e8 / n ** 2)))       # heads at a time
        for b in range(c["batch"]):
            for h in range(0, c["heads"], step):
                q, k, v = (x[b, h:h + step, :n].double() for x in (s.q, s.k, s.v))
                x = torch.matmul(q, k.transpose(1, 2).contiguous()).mul_(root).masked_fill_(above, -math.inf)
                p = torch.softmax(x, dim=-1)
                out[b, h:h + step] = torch.matmul(p, v)
                mass[b] += p[:, n - W:, c["sys"]:c["sys"] + c["vis"]].sum(dim=(0, 1)) / c["heads"]
        return {"out": out, "mass": mass}
    return None         # prune: nothing is computed, rows and numbers are moved
