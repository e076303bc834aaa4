"""End-to-end parity of the Alg. 3 call sequence (prefill with PVTP, decode with VTA) against
the CPU oracle, on the tiny workload in full and on cut-down versions of the large ones."""
import dataclasses

import numpy as np
import pytest
import torch

from gpu_util import (DEV, TORCH_DTYPE, assert_attention_close, assert_mass_close, assert_selection_matches, to_dev,
                      to_np64)
from oracle import st3_oracle as orc
from paper_2412_20105_amd import binding as st3
from paper_2412_20105_amd import pipeline
from workloads import decode_qkv, get_workload, prefill_qkv

pytestmark = pytest.mark.gpu


def _run_and_compare(w, B, mode="static", compact_mode=st3.ST3_HOLE_FILL, window=1, steps=None, whole_step=False,
                     lazy=None, kv_scale=None, fixed_tail=True, min_compared=0.8, gen=None):
    """Runs the workload through the pipeline and the oracle side by side.  A (layer, sequence) pair
    stops being compared once a near-tie was resolved the other way (values then differ
    legitimately); the share of pairs compared to the end is printed and must reach min_compared.
    gen: a Generation of the same shape to run the job on (one that has served other jobs before)."""
    T = w.steps if steps is None else steps
    keep = [row[:T + 1] for row in pipeline.keep_table_for(w)]
    keep_np = np.array(keep)
    assert np.array_equal(keep_np, orc.schedule_for(w)[:, :T + 1])
    if gen is None:
        gen = pipeline.Generation(w.layers, w.heads, w.head_dim, TORCH_DTYPE[w.dtype], B, w.n_sys, w.n_vis, w.n_txt,
                                  T, keep, window=window, mode=mode, compact_mode=compact_mode, device=DEV,
                                  lazy=lazy, kv_scale=kv_scale, fixed_tail=fixed_tail)

    def phys_len(l, k_vis, t):
        """kv_len[b] the device must hold: the end of the tail, which does not move when it is fixed."""
        return orc.kv_len(w.n_sys, keep[l][0] if fixed_tail else k_vis, w.n_txt, t)

    fp8 = {} if kv_scale is None else dict(kv_format="e4m3", k_scale=np.full((B, w.heads), kv_scale, np.float32),
                                           v_scale=np.full((B, w.heads), kv_scale, np.float32))
    ref = orc.Generation(w.layers, w.heads, w.head_dim, w.n_sys, w.n_vis, w.n_txt, keep_np, window=window, mode=mode,
                         lazy=lazy, **fp8)
    pre = [prefill_qkv(w, l, B) for l in range(w.layers)]
    r = ref.prefill(lambda l: pre[l])
    diverged = np.zeros((w.layers, B), bool)      # a near-tie was resolved differently: values no longer comparable
    near_ties = 0

    def check_sets(l, b, prev_scores, prev_ids, k, what):
        nonlocal near_ties
        lc = gen.layers[l]
        ids = lc.ids[b, :lc.h_vis].cpu().numpy()
        assert lc.h_vis == k
        if prev_scores is None:
            assert sorted(ids.tolist()) == list(range(w.n_vis))
            return
        same = assert_selection_matches(ids, prev_scores, prev_ids, k, what)
        if not same:
            near_ties += 1
            diverged[l:, b] = True

    for l in range(w.layers):
        print(f"{w.name} prefill layer {l}", flush=True)
        q, k, v = (to_dev(x, w.dtype) for x in pre[l])
        out, mass = gen.prefill_layer(l, q, k, v)
        torch.cuda.synchronize()
        got_o, got_m = to_np64(out), to_np64(mass)
        lc = gen.layers[l]
        for b in range(B):
            if l == 0:
                check_sets(l, b, None, None, keep[l][0], "")
            elif not diverged[l - 1, b]:
                check_sets(l, b, r["mass"][l - 1][b], r["ids"][l - 1][b], keep[l][0], f"prefill l={l} b={b}")
            if diverged[l, b]:
                continue
            # prefill storage is order preserving: ids ascending
            assert np.array_equal(lc.ids[b, :lc.h_vis].cpu().numpy(), r["ids"][l][b])
            assert_attention_close(got_o[b], r["out"][l][b], w.dtype, f"prefill out l={l} b={b}")
            assert_mass_close(got_m[b], r["mass"][l][b], f"prefill mass l={l} b={b}")
            assert_mass_close(lc.score[b, :lc.h_vis].double().cpu().numpy(), ref.rho[l][b], f"rho l={l} b={b}")
    gen.begin_decode()                            # the eviction ahead of the first step (Alg. 3)
    torch.cuda.synchronize()
    for t in range(1, T + 1):
        if t % 16 == 1:
            print(f"{w.name} decode step {t}", flush=True)
        dec = [decode_qkv(w, l, t, B) for l in range(w.layers)]
        rho_before = [[x.copy() for x in ref.rho[l]] for l in range(w.layers)]
        ids_before = [[x.copy() for x in ref.ids[l]] for l in range(w.layers)]
        s = ref.decode_step(lambda l: dec[l])
        # the rows each layer attends over at step t are already in place: the kept set of step t
        ids_attn = []
        for l in range(w.layers):
            lc = gen.layers[l]
            assert lc.vis_len.cpu().tolist() == [keep[l][t]] * B
            assert lc.kv_len.cpu().tolist() == [phys_len(l, keep[l][t], t) - 1] * B
            assert gen.kv_lens()[l] + 1 == s["kv_len"][l][0]
            for b in range(B):
                if not diverged[l, b]:
                    check_sets(l, b, rho_before[l][b], ids_before[l][b], keep[l][t], f"t={t} l={l} b={b}")
            ids_attn.append(lc.ids[:, :lc.h_vis].cpu().numpy())
        if whole_step:                              # one library call for all layers of the step
            qkv = torch.stack([torch.stack([to_dev(x, w.dtype) for x in dec[l]]) for l in range(w.layers)]).contiguous()
            outs = gen.decode_step(t, qkv)
            torch.cuda.synchronize()
        for l in range(w.layers):
            lc = gen.layers[l]
            if whole_step:
                out = outs[l]
            else:
                q, k, v = (to_dev(x, w.dtype) for x in dec[l])
                out, _ = gen.decode_layer(l, t, q, k, v)
                torch.cuda.synchronize()
            got_o = to_np64(out)
            k_next = keep[l][t + 1] if t < T else keep[l][t]
            assert lc.h_vis == k_next
            assert lc.vis_len.cpu().tolist() == [k_next] * B
            assert lc.kv_len.cpu().tolist() == [phys_len(l, k_next, t)] * B
            ids_after = lc.ids[:, :lc.h_vis].cpu().numpy()
            for b in range(B):
                if diverged[l, b]:
                    continue
                assert_attention_close(got_o[b], s["out"][l][b], w.dtype, f"decode out t={t} l={l} b={b}")
                if mode == "static":
                    # the mass comes back in the cache order the attention saw; map through those ids
                    pos = np.searchsorted(s["ids"][l][b], ids_attn[l][b])
                    assert_mass_close(to_np64(lc.mass[b, :len(pos)]), s["mass"][l][b][pos],
                                      f"decode mass t={t} l={l} b={b}")
                else:
                    # the mass became the ranking column, which the eviction compacted with the rows
                    pos = np.searchsorted(s["ids"][l][b], ids_after[b])
                    assert np.array_equal(s["ids"][l][b][pos], ids_after[b])
                    assert_mass_close(to_np64(lc.score[b, :lc.h_vis]), s["mass"][l][b][pos],
                                      f"ranking column after t={t} l={l} b={b}")
    # KV bytes actually held == closed form
    ebytes = 1 if kv_scale is not None else 2 if w.dtype == "bf16" else 4
    assert gen.kv_bytes() == orc.kv_bytes(B, w.heads, w.head_dim, ebytes, ref.cache_lens(), value_only=lazy or ())
    compared = int((~diverged).sum())
    print(f"{w.name}: {compared} of {diverged.size} (layer, sequence) pairs compared through the last step, "
          f"{near_ties} selections resolved a near-tie the other way", flush=True)
    assert compared >= min_compared * diverged.size, f"only {compared} of {diverged.size} pairs were compared"
    return near_ties, diverged


@pytest.mark.parametrize("fixed_tail", [True, False])
@pytest.mark.parametrize("mode", ["static", "current"])
@pytest.mark.parametrize("compact_mode", [st3.ST3_HOLE_FILL, st3.ST3_STABLE])
def test_tiny_workload_full(mode, compact_mode, fixed_tail):
    w = get_workload("tiny")
    near, div = _run_and_compare(w, 1, mode=mode, compact_mode=compact_mode, fixed_tail=fixed_tail)
    assert not div.any(), "tiny workload resolved a near-tie differently from the oracle"


@pytest.mark.parametrize("whole_step", [False, True])
def test_one_generation_serves_two_jobs(whole_step):
    """A second prefill on the same Generation starts clean: the layers before the first prune event
    rank by their own mass again, not by what the previous job's last prune event left behind."""
    w = get_workload("tiny")
    keep = pipeline.keep_table_for(w)
    gen = pipeline.Generation(w.layers, w.heads, w.head_dim, TORCH_DTYPE[w.dtype], 2, w.n_sys, w.n_vis, w.n_txt,
                              w.steps, keep, device=DEV)
    for seed in (w.seed, w.seed + 1):
        near, div = _run_and_compare(dataclasses.replace(w, seed=seed), 2, whole_step=whole_step, gen=gen)
        assert not div.any()


def test_13b_shape_cut_down_current_mode():
    w = dataclasses.replace(get_workload("llava15_13b"), layers=4, heads=8, steps=10,
                            step_schedule={"kind": "cos", "tau": 10})
    _run_and_compare(w, 2, mode="current")


@pytest.mark.parametrize("mode", ["static", "current"])
def test_tiny_workload_whole_step_call(mode):
    w = get_workload("tiny")
    near, div = _run_and_compare(w, 2, mode=mode, whole_step=True)
    assert not div.any()


def test_many_layers_whole_step_call_current_mode():
    """Every layer's eviction rides in the next layer's launch; each step's mass feeds the next ranking."""
    w = dataclasses.replace(get_workload("llava15_7b"), layers=19, heads=2, steps=5, n_vis=120, n_txt=9,
                            step_schedule={"kind": "cos", "tau": 6})
    _run_and_compare(w, 2, mode="current", whole_step=True)


def _many_layers_with_a_group_across_the_fork():
    """34 layers; layers 15-17 inherit from layer 14 (the group lies on both sides of layer 16, where the by-value
    plan launches of the per-layer path change batch)."""
    keep = [120] * 3 + [100] * 11 + [80] * 4 + [60] * 16
    w = dataclasses.replace(get_workload("llava15_7b"), layers=34, heads=2, steps=4, n_vis=120, n_txt=9,
                            layer_schedule={"kind": "table", "keep": keep}, step_schedule={"kind": "cos", "tau": 5})
    return w, {15: 14, 16: 14, 17: 14}


@pytest.mark.parametrize("mode", ["static", "current"])
def test_many_layers_and_a_heredity_group_in_one_plan_launch(mode):
    """34 layers, three of them lazy: the entries of all of them travel to the launch behind the attention in one argument
    block (41 entries of a finish launch, 35 where the columns take the mass)."""
    w, lazy = _many_layers_with_a_group_across_the_fork()
    _run_and_compare(w, 2, mode=mode, whole_step=True, lazy=lazy)


def _run_job_whole_steps(w, lazy, B, stream=None):
    """The job through whole-step calls (no oracle): per step the outputs and every layer's columns and lengths."""
    T = w.steps
    keep = [row[:T + 1] for row in pipeline.keep_table_for(w)]
    with torch.cuda.stream(stream if stream is not None else torch.cuda.current_stream()):
        gen = pipeline.Generation(w.layers, w.heads, w.head_dim, TORCH_DTYPE[w.dtype], B, w.n_sys, w.n_vis, w.n_txt, T,
                                  keep, mode="current", device=DEV, lazy=lazy)
        for l in range(w.layers):
            gen.prefill_layer(l, *(to_dev(x, w.dtype) for x in prefill_qkv(w, l, B)))
        seen = []
        for t in range(1, T + 1):
            qkv = torch.stack([torch.stack([to_dev(x, w.dtype) for x in decode_qkv(w, l, t, B)])
                               for l in range(w.layers)]).contiguous()
            outs = gen.decode_step(t, qkv)
            torch.cuda.current_stream().synchronize()
            seen.append([outs.clone()] + [x.clone() for lc in gen.layers
                                          for x in (lc.ids, lc.score, lc.mass, lc.vis_len, lc.kv_len)])
        torch.cuda.current_stream().synchronize()
    return seen


def _assert_same_bits(a_steps, b_steps, what):
    assert len(a_steps) == len(b_steps)
    for t, (a, b) in enumerate(zip(a_steps, b_steps)):
        assert len(a) == len(b)
        for i, (x, y) in enumerate(zip(a, b)):
            assert torch.equal(x.view(torch.uint8), y.view(torch.uint8)), f"{what}: step {t + 1}, tensor {i}"


def test_whole_step_calls_repeat_bit_for_bit():
    """The same job twice through whole-step calls: outputs, masses, kept ids and lengths are equal bit for bit at
    every step (head and chunk reductions run in a fixed order)."""
    w, lazy = _many_layers_with_a_group_across_the_fork()
    runs = [_run_job_whole_steps(w, lazy, 3) for _ in range(2)]
    _assert_same_bits(runs[0], runs[1], "second run against first")


def test_two_threads_run_whole_step_calls_at_once():
    """Two host threads run a job each, on streams of their own: both get the bits a job gets alone."""
    import threading
    w, lazy = _many_layers_with_a_group_across_the_fork()
    alone = _run_job_whole_steps(w, lazy, 2)
    streams = [torch.cuda.Stream(device=DEV) for _ in range(2)]
    got, errors = [None, None], []

    def job(i):
        try:
            torch.cuda.set_device(DEV)
            got[i] = _run_job_whole_steps(w, lazy, 2, streams[i])
        except Exception as e:                  # surfaced in the main thread below
            errors.append(e)

    threads = [threading.Thread(target=job, args=(i,)) for i in range(2)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for i in range(2):
        _assert_same_bits(alone, got[i], f"thread {i} against a job alone")


@pytest.mark.parametrize("fixed_tail", [True, False])
def test_large_evictions_whole_step_call(fixed_tail):
    """Evictions above the in-kernel row-move threshold: the separate row-move launch after the plans."""
    w = dataclasses.replace(get_workload("llava15_13b"), layers=5, heads=4, steps=3, n_txt=20,
                            step_schedule={"kind": "cos", "tau": 3})
    _run_and_compare(w, 2, whole_step=True, fixed_tail=fixed_tail)


def _lazy_workload(name, **kw):
    """Six layers, the last three a QK-heredity group: layers 4 and 5 inherit from layer 3 (the
    paper's "28 -> 29~31" pattern), so rows 3-5 of the keep table are equal."""
    base = dict(layers=6, heads=4, steps=6, n_vis=120, n_txt=9,
                layer_schedule={"kind": "table", "keep": [120, 120, 100, 80, 80, 80]},
                step_schedule={"kind": "cos", "tau": 6})
    base.update(kw)
    return dataclasses.replace(get_workload(name), **base)


@pytest.mark.parametrize("mode", ["static", "current"])
@pytest.mark.parametrize("compact_mode", [st3.ST3_HOLE_FILL, st3.ST3_STABLE])
def test_qk_heredity_group(mode, compact_mode):
    """Eq. 6 / Alg. 2: lazy layers take the source's probabilities, at prefill and at every step;
    K-less caches; the group evicts alike.  B*H is small, so the strips are split into chunks."""
    w = _lazy_workload("llava15_7b")
    _run_and_compare(w, 2, mode=mode, compact_mode=compact_mode, whole_step=True, lazy={4: 3, 5: 3})


def test_qk_heredity_fp32_many_heads_no_split_large_evictions():
    """fp32, enough (b,h) strips that no strip is split, evictions above the in-kernel move limit."""
    w = _lazy_workload("tiny", heads=40, head_dim=64, steps=3, n_vis=300, n_sys=8, n_txt=16,
                       layer_schedule={"kind": "table", "keep": [300, 300, 300, 260, 260, 260]},
                       step_schedule={"kind": "cos", "tau": 3})
    _run_and_compare(w, 28, whole_step=True, lazy={1: 0, 2: 0, 5: 4})


def test_qk_heredity_needs_the_whole_step_call():
    w = _lazy_workload("llava15_7b")
    keep = pipeline.keep_table_for(w)
    gen = pipeline.Generation(w.layers, w.heads, w.head_dim, torch.bfloat16, 1, w.n_sys, w.n_vis, w.n_txt, w.steps,
                              keep, device=DEV, lazy={4: 3})
    with pytest.raises(RuntimeError):
        gen.decode_layer(0, 1, None, None, None)
    with pytest.raises(ValueError):
        pipeline.Generation(w.layers, w.heads, w.head_dim, torch.bfloat16, 1, w.n_sys, w.n_vis, w.n_txt, w.steps,
                            keep, device=DEV, lazy={3: 2})          # keeps differ


@pytest.mark.parametrize("whole_step", [False, True])
def test_e4m3_kv_cache_13b_shape_cut_down(whole_step):
    """The caches in FP8 E4M3 (scale 6 sigma / 448 for every strip): prefill attends the unquantised
    prompt, its rows and every appended row go through the quantiser, decode reads code x scale."""
    w = dataclasses.replace(get_workload("llava15_13b"), layers=5, heads=8, steps=8,
                            step_schedule={"kind": "cos", "tau": 8})
    _run_and_compare(w, 2, whole_step=whole_step, kv_scale=6 * w.sigma / 448)


@pytest.mark.parametrize("fixed_tail", [True, False])
def test_e4m3_kv_cache_with_heredity_group_and_current_mode(fixed_tail):
    w = _lazy_workload("llava15_7b")
    _run_and_compare(w, 2, mode="current", whole_step=True, lazy={4: 3, 5: 3}, kv_scale=6 * w.sigma / 448,
                     fixed_tail=fixed_tail)


def test_tiny_workload_batched_window():
    w = get_workload("tiny")
    _run_and_compare(w, 3, window=2)


@pytest.mark.parametrize("fixed_tail", [True, False])
def test_13b_shape_cut_down(fixed_tail):
    """Head dim, token counts and schedule form of the 13B workload; fewer layers, heads, steps.  With a
    fixed tail the visual segments empty out while the tail stays 600 rows further on."""
    w = dataclasses.replace(get_workload("llava15_13b"), layers=6, heads=8, steps=12,
                            step_schedule={"kind": "cos", "tau": 12})
    _run_and_compare(w, 2, fixed_tail=fixed_tail)


def test_7b_shape_cut_down_stable_compaction():
    w = dataclasses.replace(get_workload("llava15_7b"), layers=5, heads=4, steps=6,
                            step_schedule={"kind": "linear", "tau": 8})
    _run_and_compare(w, 1, compact_mode=st3.ST3_STABLE)


def test_highres_shape_cut_down():
    w = dataclasses.replace(get_workload("llava_next_hr"), layers=4, heads=2, steps=3,
                            step_schedule={"kind": "cos", "tau": 3})
    _run_and_compare(w, 1)


def test_skewed_workload_ties():
    """Planted exact ties (lowest id must win) and one-ulp near-ties (tolerance rule)."""
    w = dataclasses.replace(get_workload("skewed_13b"), layers=5, heads=4, steps=6,
                            step_schedule={"kind": "cos", "tau": 8})
    _run_and_compare(w, 2, min_compared=0.0)        # planted near-ties may go either way


def test_pvtp_stride_schedule_with_exp_annealing():
    """The paper's own 13B setting (S=4, R=5%, P=50%) on a cut-down model, exponential decay."""
    w = dataclasses.replace(get_workload("llava15_13b"), layers=12, heads=4, steps=5, n_vis=200, n_txt=20,
                            layer_schedule={"kind": "pvtp", "S": 4, "P_bp": 5000, "R_bp": 500},
                            step_schedule={"kind": "exp", "sigma": 3})
    _run_and_compare(w, 1)


@pytest.mark.parametrize("name,kw,B,lazy", [
    ("tiny", {}, 2, None),
    ("llava15_13b", dict(layers=6, heads=8, steps=5, step_schedule={"kind": "cos", "tau": 5}), 2, None),
    ("llava15_7b", dict(layers=6, heads=4, steps=4, n_vis=120, n_txt=9,
                        layer_schedule={"kind": "table", "keep": [120, 120, 100, 80, 80, 80]},
                        step_schedule={"kind": "cos", "tau": 6}), 2, {4: 3, 5: 3}),
])
def test_layers_called_one_at_a_time_with_a_data_dependency(name, kw, B, lazy):
    """The step as a real decoder calls it (Alg. 3, loop over l): st3_decode_layer_attend per layer, the next
    layer's query formed on the HOST from the previous layer's output after it was read back, then
    st3_decode_plans once.  The oracle replays the step with the queries the device path used."""
    w = dataclasses.replace(get_workload(name), **kw)
    T = w.steps
    keep = [row[:T + 1] for row in pipeline.keep_table_for(w)]
    for l, src in (lazy or {}).items():
        assert keep[l] == keep[src]
    gen = pipeline.Generation(w.layers, w.heads, w.head_dim, TORCH_DTYPE[w.dtype], B, w.n_sys, w.n_vis, w.n_txt, T, keep,
                              device=DEV, lazy=lazy)
    ref = orc.Generation(w.layers, w.heads, w.head_dim, w.n_sys, w.n_vis, w.n_txt, np.array(keep), lazy=lazy)
    pre = [prefill_qkv(w, l, B) for l in range(w.layers)]
    r = ref.prefill(lambda l: pre[l])
    for l in range(w.layers):
        q, k, v = (to_dev(x, w.dtype) for x in pre[l])
        gen.prefill_layer(l, q, k, v)
    compared = 0
    alive = np.ones((w.layers, B), bool)
    for t in range(1, T + 1):
        dec = [list(decode_qkv(w, l, t, B)) for l in range(w.layers)]
        gen.begin_step(t)
        torch.cuda.synchronize()
        ids_attn = [gen.layers[l].ids[:, :gen.layers[l].h_vis].cpu().numpy() for l in range(w.layers)]
        rho_before = [[x.copy() for x in ref.rho[l]] for l in range(w.layers)]
        ids_before = [[x.copy() for x in ref.ids[l]] for l in range(w.layers)]
        outs, keepalive = [], []
        prev = None
        for l in range(w.layers):
            if prev is not None:        # the data dependency: this layer's query needs the previous layer's output
                dec[l][0] = dec[l][0] + 0.25 * prev
            q, k, v = (to_dev(x, w.dtype) for x in dec[l])
            dec[l][0] = q.float().cpu().numpy().astype(np.float64)     # what the device path really used (rounded to dtype)
            keepalive.append((q, k, v))
            out = gen.attend_layer(l, q, k, v)
            torch.cuda.synchronize()
            prev = out.float().cpu().numpy()                            # read back before the next layer's inputs exist
            outs.append(to_np64(out))
        gen.finish_step()
        torch.cuda.synchronize()
        s = ref.decode_step(lambda l: tuple(dec[l]))
        for l in range(w.layers):
            lc = gen.layers[l]
            for b in range(B):
                if alive[l, b]:
                    alive[l, b] = assert_selection_matches(ids_attn[l][b], rho_before[l][b], ids_before[l][b], keep[l][t],
                                                           f"t={t} l={l} b={b}")
                if not alive[l, b]:
                    continue
                assert_attention_close(outs[l][b], s["out"][l][b], w.dtype, f"out t={t} l={l} b={b}")
                pos = np.searchsorted(s["ids"][l][b], ids_attn[l][b])
                assert_mass_close(to_np64(lc.mass[b, :len(pos)]), s["mass"][l][b][pos], f"mass t={t} l={l} b={b}")
                compared += 1
            k_next = keep[l][t + 1] if t < T else keep[l][t]
            assert lc.vis_len.cpu().tolist() == [k_next] * B
    print(f"{w.name}: {compared} of {w.layers * B * T} (layer, sequence, step) triples compared", flush=True)
    assert compared >= 0.8 * w.layers * B * T


def _random_generation(seed):
    """A whole job of random shape, retention tables, heredity groups and options (seeded)."""
    rng = np.random.default_rng(77000 + seed)
    base = "tiny" if rng.random() < 0.35 else "llava15_7b"              # float32 / bf16 values
    L = int(rng.integers(2, 12)) if rng.random() < 0.8 else int(rng.integers(17, 36))
    H, D, B = int(rng.choice([1, 2, 3, 4, 8])), int(rng.choice([64, 128])), int(rng.integers(1, 4))
    n_sys, n_vis, n_txt, T = int(rng.integers(0, 40)), int(rng.integers(4, 200)), int(rng.integers(1, 40)), int(rng.integers(2, 6))
    keep = [n_vis] * int(rng.integers(1, 4))                             # full for the first layers, then never growing
    while len(keep) < L:
        keep.append(int(rng.integers(0, keep[-1] + 1)) if rng.random() < 0.6 else keep[-1])
    keep = keep[:L]
    lazy = {}
    if rng.random() < 0.4:                                               # heredity groups of 1-3 lazy layers
        l = int(rng.integers(1, L))
        while l < L:
            src = lazy.get(l - 1, l - 1)
            n = int(rng.integers(1, 4))
            for j in range(l, min(l + n, L)):
                lazy[j] = src
            l += n + int(rng.integers(1, 6))
        for j in range(1, L):
            keep[j] = keep[lazy[j]] if j in lazy else min(keep[j], keep[j - 1])
    ss = {"cos": {"kind": "cos", "tau": int(rng.integers(max(T - 1, 1), 2 * T + 1))},
          "linear": {"kind": "linear", "tau": int(rng.integers(max(T - 1, 1), 2 * T + 1))},
          "exp": {"kind": "exp", "sigma": float(rng.uniform(0.5, 3 * T))},
          "drop": {"kind": "drop", "per_step": int(rng.integers(1, 30))},
          "none": {"kind": "none"}}[str(rng.choice(["cos", "linear", "exp", "drop", "none"]))]
    w = dataclasses.replace(get_workload(base), layers=L, heads=H, head_dim=D, n_sys=n_sys, n_vis=n_vis, n_txt=n_txt, steps=T,
                            layer_schedule={"kind": "table", "keep": keep}, step_schedule=ss)
    opts = dict(mode=str(rng.choice(["static", "current"])), compact_mode=int(rng.choice([st3.ST3_HOLE_FILL, st3.ST3_STABLE])),
                fixed_tail=bool(rng.random() < 0.5), whole_step=bool(lazy) or bool(rng.random() < 0.5),
                window=min(int(rng.choice([1, 1, 2, 4])), n_txt), lazy=lazy or None,
                kv_scale=6 * w.sigma / 448 if (w.dtype == "bf16" and rng.random() < 0.3) else None)
    rng.choice([0, 2])                                                  # (keeps the later draws of older seeds in place)
    return w, B, opts


@pytest.mark.parametrize("block", range(4))
def test_whole_generations_of_random_shape_and_options(block):
    """Shapes, retention tables, annealing kinds, heredity groups, both cache layouts and compaction modes, both ways of
    calling a step, score windows, E4M3 caches, 2 to 35 layers."""
    compared = total = 0
    for seed in range(block * 20, block * 20 + 20):
        w, B, opts = _random_generation(seed)
        print("generation case", seed, w.layers, w.heads, w.head_dim, B, (w.n_sys, w.n_vis, w.n_txt), w.steps,
              w.layer_schedule["keep"], w.step_schedule, opts, flush=True)
        _, div = _run_and_compare(w, B, min_compared=0.0, **opts)
        compared += int((~div).sum())
        total += div.size
    assert compared >= 0.9 * total, f"only {compared} of {total} (layer, sequence) pairs were compared to the end"
