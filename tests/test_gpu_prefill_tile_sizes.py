"""bf16 prefill attention on either side of the rules that pick key groups and, without those, 32- or 64-key tiles, at the edges
of those tiles, against the same attention in 64 bits (bounds in _run)."""
import pytest

from test_gpu_prefill_key_groups import _run

pytestmark = pytest.mark.gpu


def _strips(d, n, short_tiles):
    """(batch, heads) with strips * (query tiles + 1) just at the rule's line, or just below it."""
    units = (n + 127) // 128 + 1
    least = -(-(1200 if d == 128 else 2600) // units)
    heads = 25
    return (-(-least // heads), heads) if short_tiles else ((least - 1) // heads, heads)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("short_tiles", [True, False])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 64, 65, 96, 97, 127, 128, 129, 161, 192, 224, 257, 290, 385])
def test_either_tile_at_the_rules_line(n, d, short_tiles):
    _run(*_strips(d, n, short_tiles), d, n, n // 9, n - n // 9, 1, extra_rows=3)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("short_tiles", [True, False])
@pytest.mark.parametrize("window,sys_len,short", [(16, 33, 3), (5, 64, 30), (16, 0, 0)])
def test_window_rows_and_visual_edges(d, short_tiles, window, sys_len, short):
    _run(*_strips(d, 200, short_tiles), d, 200, sys_len, 200 - sys_len - short, window)


@pytest.mark.parametrize("B,H,d,n", [
    (1, 8, 128, 1000), (4, 3, 128, 2047), (4, 3, 128, 2050), (1, 13, 128, 600), (8, 16, 128, 255), (8, 16, 128, 257), (3, 43, 128, 128),
    (2, 32, 128, 767), (2, 32, 128, 770), (1, 16, 64, 3071), (1, 16, 64, 3073), (1, 17, 64, 1900), (16, 16, 64, 190), (16, 16, 64, 194),
    (1, 257, 64, 128), (2, 32, 64, 1535)])
def test_key_groups_at_the_rules_lines(B, H, d, n):
    _run(B, H, d, n, 5, n - 20, 2)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("short_tiles", [True, False])
def test_keys_that_weigh_nothing(d, short_tiles):
    """Whole tiles of logit -inf in the middle and up to the diagonal of some rows."""
    _run(*_strips(d, 230, short_tiles), d, 230, 4, 200, 1, dead=[*range(32, 96), *range(160, 200)])
