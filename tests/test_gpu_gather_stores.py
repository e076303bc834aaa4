"""st3_gather_rows on both sides of the size from which its stores go past the caches (400 MB written): bytes equal to an
index lookup, rows behind a bad index untouched."""
import pytest
import torch

from paper_2412_20105_amd import binding as st3

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
STREAM = 400 << 20


@pytest.mark.parametrize("words,kept,past", [
    (32, 3196, False),      # 4 + 3196 rows of 128 bytes in 2 pairs x 8 x 64 strips: 400 MB to the byte
    (32, 3197, True),
    (20, 5117, True),       # rows of five 16-byte vectors: no power of two, and strips that end inside a workgroup's last turn
])
def test_gather_around_the_store_threshold(words, kept, past):
    B, H, n, head, tail = 8, 64, kept + 80, 3, 1
    assert ((head + kept + tail) * words * 4 * H * B * 2 > STREAM) == past
    g = torch.Generator(device=DEV).manual_seed(kept)
    src = [torch.randint(-2 ** 31, 2 ** 31 - 1, (B, H, head + n + tail, words), generator=g, device=DEV, dtype=torch.int32) for _ in range(2)]
    dst = [torch.full((B, H, head + kept + tail + 2, words), 7, dtype=torch.int32, device=DEV) for _ in range(2)]
    idx = torch.rand((B, n), generator=g, device=DEV).argsort(dim=1)[:, :kept].sort(dim=1)[0].to(torch.int32)
    idx[1, 5] = -1
    idx[2, 9] = n
    st3.st3_gather_rows(list(zip(src, dst)), head, idx, kept, n, tail)
    rows = torch.cat([torch.arange(head, device=DEV).expand(B, head), head + idx.long().clamp(0, n - 1),
                      torch.arange(head + n, head + n + tail, device=DEV).expand(B, tail)], dim=1)
    for s, d in zip(src, dst):
        want = s.gather(2, rows[:, None, :, None].expand(B, H, rows.shape[1], words))
        want[1, :, head + 5] = 7
        want[2, :, head + 9] = 7
        assert torch.equal(d[:, :, :head + kept + tail], want)
        assert bool((d[:, :, head + kept + tail:] == 7).all())
