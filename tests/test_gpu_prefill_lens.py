"""Lengths of every layer behind its prefill, however the layers are called: a whole job, a second one on the same object, a layer
prefilled again behind decode steps, a keep table changed between jobs."""
import pytest
import torch

from paper_2412_20105_amd.pipeline import Generation

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("B,fixed_tail", [(1, True), (3, False)])
def test_lengths_follow_the_prefill(B, fixed_tail):
    L, H, d, ns, nv, nx, T = 5, 2, 64, 3, 40, 7, 4
    keep = [[n] + [n - 2 * t for t in range(1, T + 1)] for n in (40, 40, 30, 30, 20)]
    gen = Generation(L, H, d, torch.float32, B, ns, nv, nx, T, keep, device=DEV, fixed_tail=fixed_tail)
    g = torch.Generator(device=DEV).manual_seed(B)
    Q, K, V = (torch.randn((B, H, ns + nv + nx, d), generator=g, device=DEV) for _ in range(3))

    def prefill(layers):
        for l in layers:
            gen.prefill_layer(l, Q, K, V)

    def check(counts, layers=range(L)):
        for l in layers:
            n = counts[l]
            assert gen.layers[l].lens.tolist() == [[n] * B, [ns + n + nx] * B, [ns + n] * B], l

    def decode(steps):
        for t in steps:
            gen.decode_step(t, torch.randn((L, 3, B, H, d), generator=g, device=DEV))

    prefill(range(L)); check([40, 40, 30, 30, 20])
    decode((1, 2))
    assert gen.layers[4].lens[0].tolist() == [gen.layers[4].h_vis] * B != [20] * B
    prefill((4,)); check([40, 40, 30, 30, 20], (4,))
    gen.keep[3] = [25] + gen.keep[3][1:]
    prefill(range(L)); check([40, 40, 30, 25, 20])
    decode((1,))
    gen.keep[4] = [22] + gen.keep[4][1:]
    prefill(range(L)); check([40, 40, 30, 25, 22])
    prefill((4,)); prefill((4,)); check([40, 40, 30, 25, 22])
