"""st3_compact_rows without a tail: calls around the sizes at which a workgroup's one pass (1024 or 4096 units) is exceeded."""
import numpy as np
import pytest
import torch

from paper_2412_20105_amd import binding as st3

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("row_bytes,k", [(4, 1), (4, 257), (4, 1023), (4, 1024), (4, 1025), (4, 4095), (4, 4096), (4, 4097), (8, 512),
                                         (8, 2048), (8, 2049), (12, 300), (24, 513), (256, 64), (256, 65), (256, 256), (256, 257),
                                         (4112, 3), (4112, 17)])
@pytest.mark.parametrize("inner", [1, 3])
def test_compact_without_tail(row_bytes, k, inner):
    rng = np.random.default_rng(k * 8 + row_bytes)
    B, n = 3, k + k // 7 + 2
    pad = 16 if row_bytes % 16 == 0 else 4
    stride = row_bytes + pad
    buf = rng.integers(0, 255, (B, inner, n, stride), dtype=np.uint8)
    keep = np.stack([np.sort(rng.choice(n, k, replace=False)) for _ in range(B)]).astype(np.int32)
    run = [k, k // 2, 0]                # valid indices in front of the first invalid one
    keep[1, k // 2] = -1
    keep[2, 0] = n
    d, d_idx = torch.from_numpy(buf.copy()).to(DEV), torch.from_numpy(keep).to(DEV)
    st3.st3_compact_rows(d.data_ptr(), B, inner, inner * n * stride, n * stride, stride, row_bytes, d_idx, k, n, 0)
    got = d.cpu().numpy()
    for b in range(B):
        want = buf[b].copy()
        want[:, :run[b], :row_bytes] = buf[b][:, keep[b, :run[b]], :row_bytes]
        assert np.array_equal(got[b], want), b
