"""Generation's host-side bookkeeping, with the library's device calls replaced (no GPU)."""
import pytest
import torch

from paper_2412_20105_amd import binding as st3
from paper_2412_20105_amd import pipeline


@pytest.mark.parametrize("fixed_tail", [True, False])
def test_a_refused_eviction_leaves_the_lengths(monkeypatch, fixed_tail):
    """begin_decode(): the host's lengths follow the device's, which an error does not change; called again, it evicts."""
    calls = []

    def refuse(shape, arr, n, mode, stream=None):
        calls.append([(arr[l].keep_after, arr[l].seg.max_vis_len, arr[l].seg.max_kv_len) for l in range(n)])
        if len(calls) == 1:
            raise RuntimeError("refused")

    monkeypatch.setattr(st3, "st3_workspace_init", lambda *a, **k: None)
    monkeypatch.setattr(st3, "st3_select_compact_layers", refuse)
    monkeypatch.setattr(st3, "kv_layer", lambda *a: st3.KvLayer())                  # (they take device tensors only)
    monkeypatch.setattr(st3, "segments", lambda *a: st3.Segments(*a[:3]))
    gen = pipeline.Generation(3, 2, 64, torch.float32, 1, 4, 20, 6, 2, [[20, 15, 12], [20, 20, 20], [10, 7, 7]], device="cpu",
                              fixed_tail=fixed_tail)
    for lc, vis in zip(gen.layers, (20, 20, 10)):
        lc.h_vis, lc.h_kv = vis, 10 + vis
    with pytest.raises(RuntimeError, match="refused"):
        gen.begin_decode()
    assert [(lc.h_vis, lc.h_kv) for lc in gen.layers] == [(20, 30), (20, 30), (10, 20)]
    gen.begin_decode()
    assert calls[1] == calls[0] == [(15, 20, 30), (-1, 20, 30), (7, 10, 20)]
    closed = 0 if fixed_tail else 1
    assert [(lc.h_vis, lc.h_kv) for lc in gen.layers] == [(15, 30 - 5 * closed), (20, 30), (7, 20 - 3 * closed)]


def test_current_stream_without_the_raw_handle(monkeypatch):
    """A torch that lacks the two functions behind the raw handle: the public interface is asked."""
    class Stream:
        cuda_stream = 0x1234

    monkeypatch.setattr(torch.cuda, "current_stream", lambda: Stream)
    monkeypatch.setattr(st3, "_raw_stream", lambda device: 0x5678 + device)
    monkeypatch.setattr(st3, "_raw_device", lambda: 1)
    assert st3._stream(None) == 0x5679 and st3._stream(7) == 7 and st3._stream(Stream) == 0x1234
    for missing in ("_raw_stream", "_raw_device"):
        with monkeypatch.context() as m:
            m.setattr(st3, missing, None)
            assert st3._stream(None) == 0x1234


class RecordingLibrary:
    """The library's calls, noted instead of made; pointers to structures as the structures' fields."""

    def __init__(self):
        self.calls = []

    def __getattr__(self, name):
        def call(*args):
            self.calls.append((name, args))
            return 1 << 12 if name == "st3_workspace_bytes" else 0
        return call

    def gathered(self):
        """Sources of the last gather, and the queries and the name of the attention call behind it."""
        (_, g), (name, a) = [c for c in self.calls if c[0] in ("st3_gather_rows", "st3_prefill_attention", "st3_prefill_attention_kept")][-2:]
        return [g[0][i].src for i in range(g[1])], a[1]._obj.data, name


@pytest.fixture
def host(monkeypatch):
    """make(...) -> (a Generation on host memory, its recorded calls)."""
    rec = RecordingLibrary()
    monkeypatch.setattr(st3, "lib", lambda: rec)
    monkeypatch.setattr(st3, "_stream", lambda s: 0)
    monkeypatch.setattr(st3, "tensor4", lambda t: st3.Tensor4(t.data_ptr(), t.stride(0), t.stride(1), t.stride(2)))
    monkeypatch.setattr(st3, "kv_layer", lambda *a: st3.KvLayer())                  # (they take device tensors only)
    monkeypatch.setattr(st3, "segments", lambda *a: st3.Segments(*a[:3]))

    def make(keep, dtype=torch.bfloat16, B=2, **more):
        gen = pipeline.Generation(len(keep), 3, 64, dtype, B, 4, keep[0][0], 6, len(keep[0]) - 1, keep, device="cpu", **more)
        return gen, rec, [torch.zeros((B, 3, gen.N0, 64), dtype=dtype) for _ in range(3)]
    return make


def _overlapping_queries(gen, where):
    lc = gen.layers[1]
    if where == "returned":             # what layer 0's prefill has returned
        return gen.out_stage[:, :, :gen.N0]
    if where == "workspace":
        lc.ws = torch.zeros(2 * gen.B * gen.H * gen.N0 * gen.d, dtype=torch.uint8)
        return lc.ws.view(torch.bfloat16).view(gen.B, gen.H, gen.N0, gen.d)
    base = {"last_rows": gen.out_stage, "cache": lc.v if gen.kv_scale is None else gen.v_stage, "stage": gen.q_stage}[where]
    if where != "last_rows":
        return base[:, :, :gen.N0]
    wide = torch.zeros(2 * base.numel(), dtype=base.dtype)      # rows whose end reaches into the output's first row
    gen.out_stage = wide[base.numel() - 8:][:base.numel()].view(base.shape)
    return wide[:base.numel()].view(base.shape)


@pytest.mark.parametrize("kv_scale", [None, 0.01])
@pytest.mark.parametrize("where", ["returned", "last_rows", "cache", "stage", "workspace"])
@pytest.mark.parametrize("kept", [20, 12])
def test_queries_that_a_layers_prefill_writes_over_are_copied_first(host, where, kept, kv_scale):
    gen, rec, (Q, K, V) = host([[20], [kept]], kv_scale=kv_scale)
    gen.prefill_layer(0, Q, K, V)
    assert rec.gathered() == ([K.data_ptr(), V.data_ptr()], Q.data_ptr(), "st3_prefill_attention")
    q = _overlapping_queries(gen, where)
    gen.prefill_layer(1, q, K, V)
    assert rec.gathered() == ([q.data_ptr(), K.data_ptr(), V.data_ptr()], gen.q_stage.data_ptr(), "st3_prefill_attention")
    gen.prefill_layer(1, Q, K, V)
    assert rec.gathered() == ([K.data_ptr(), V.data_ptr()], Q.data_ptr(), "st3_prefill_attention_kept" if kept < 20 else "st3_prefill_attention")


@pytest.mark.parametrize("which", [(1,), (2,), (1, 2)])
def test_keys_and_values_of_another_element_size_are_refused(host, which):
    """A row's bytes are those of the first tensor that is copied: elements of twice the size would be written past the caches' rows."""
    gen, rec, x = host([[20], [12]])
    x = [t.float() if i in which else t for i, t in enumerate(x)]
    with pytest.raises(AssertionError):
        gen.prefill_layer(0, *x)
    assert not any(name.startswith(("st3_gather", "st3_prefill")) for name, _ in rec.calls)


def test_queries_in_another_memory_are_copied(host):
    """Queries that the device can read but does not hold (pinned host memory, a peer's): the gather reads them, not every tile."""
    class Elsewhere(torch.Tensor):
        device = torch.device("meta")

    gen, rec, (Q, K, V) = host([[20], [12]])
    away = Q.as_subclass(Elsewhere)
    for l in range(2):
        gen.prefill_layer(l, away, K, V)
        assert rec.gathered() == ([Q.data_ptr(), K.data_ptr(), V.data_ptr()], gen.q_stage.data_ptr(), "st3_prefill_attention")


@pytest.mark.parametrize("fixed_tail", [True, False])
def test_layer_0_prefilled_again_leaves_the_other_layers_lengths(host, fixed_tail):
    """Behind decode steps every layer's lengths on the device are the host's, whichever layers are prefilled again."""
    gen, rec, x = host([[20, 15, 12], [20, 20, 18], [10, 7, 7]], fixed_tail=fixed_tail)

    def lengths():
        return [lc.lens[:2].tolist() for lc in gen.layers]

    for l in range(3):
        gen.prefill_layer(l, *x)
        assert lengths()[l] == [[gen.layers[l].h_vis] * 2, [gen.layers[l].h_kv] * 2]
    gen.decode_step(1, torch.zeros((3, 3, 2, 3, 64), dtype=torch.bfloat16))
    for lc in gen.layers:                   # what the step's launches do
        lc.vis_len.fill_(lc.h_vis)
        lc.kv_len.fill_(lc.h_kv)
    for again in (0, 2, 0):
        before = lengths()
        gen.prefill_layer(again, *x)
        for l, (lc, was) in enumerate(zip(gen.layers, before)):
            assert lengths()[l] == [[lc.h_vis] * 2, [lc.h_kv] * 2], (again, l)
            assert l == again or lengths()[l] == was
