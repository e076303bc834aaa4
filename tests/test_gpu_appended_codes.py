"""The appended token's row of an E4M3 cache, which one wave of an attention workgroup quantises four elements a lane: every code
is the oracle's, for K and V, with scales of their own, in ordinary and lazy layers and in either form of the step."""
import numpy as np
import pytest
import torch

from oracle import st3_oracle as orc
from gpu_util import rand_values
from test_gpu_parity import _e4m3_adversarial
from test_gpu_step_launches import BF, DEV, Step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["whole", "layer_by_layer"])
@pytest.mark.parametrize("d,B,H,vis,tail", [(64, 3, 5, 70, 3), (128, 2, 3, 200, 9), (128, 1, 1, 0, 0)])
def test_codes_of_the_appended_row(form, d, B, H, vis, tail):
    rng = np.random.default_rng(d + B)
    s = Step(L=3, B=B, H=H, d=d, dtype=BF, vis=[vis], tail=tail, e4m3=True, lazy={1: 0}, drop=0)
    k_scale, v_scale = (rng.uniform(0.003, 0.05, (3, B, H)).astype(np.float32) for _ in range(2))
    dev = [[torch.from_numpy(x[l]).to(DEV) for x in (k_scale, v_scale)] for l in range(3)]
    new = rand_values(rng, (3, 2, B, H, d), "bf16")
    for l in range(3):
        for i, scale in enumerate((k_scale, v_scale)):
            new[l, i] = _e4m3_adversarial(rng, (B, H, d), scale[l][:, :, None].astype(np.float64))
        new[l, :, 0, 0, [0, 3, 4, d - 1]] = np.array([np.nan, np.inf, -np.inf, -0.0], np.float32)[:, None]
        s.arr[l].keep_after = -1
        s.arr[l].kv.k_scale, s.arr[l].kv.v_scale = None if l == 1 else dev[l][0].data_ptr(), dev[l][1].data_ptr()
    s.qkv[:, 1:] = torch.from_numpy(new).to(DEV).to(BF)
    held = s.qkv[:, 1:].float().cpu().numpy()
    row = 3 + vis + tail
    getattr(s, form)()
    for l, st in enumerate(s.state):
        for i, (name, scale) in enumerate((("k", k_scale), ("v", v_scale))):
            if st[name] is None:
                continue
            want = orc.e4m3_quantize(held[l, i], scale[l][:, :, None])
            got = st[name][:, :, row].cpu().numpy()
            assert np.array_equal(got, want), (l, name, np.argwhere(got != want)[:5])
