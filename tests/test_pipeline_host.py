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
