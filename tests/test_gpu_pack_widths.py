"""Packing at every width around a word and around the rows' last word, with
the masks at every byte alignment, bit for bit against numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W", [1, 2, 15, 31, 32, 33, 40, 63, 64, 65, 95, 96, 97, 127, 1279, 1281])
@pytest.mark.parametrize("offset", [0, 1, 2, 3, 8, 13])
def test_pack(W, offset):
    import torch
    import paper_1903_11785_amd as fvv
    n, H = 2, 5
    rng = np.random.default_rng(W * 16 + offset)
    m = rng.integers(0, 256, (n, H, W), dtype=np.uint8) * (rng.random((n, H, W)) < 0.4).astype(np.uint8)
    m[0, 0], m[1, -1] = 255, 0
    buf = torch.full((offset + m.size,), 255, dtype=torch.uint8, device="cuda")
    masks = buf[offset:].view(n, H, W)              # the last row ends with the allocation
    masks.copy_(torch.from_numpy(m))
    ctx = fvv.Context(max_cams=2, max_w=1281, max_h=8, max_coarse=1, max_fine=1, max_rois=1,
                      max_points=1, max_jobs=1)
    got = ctx.pack_silhouettes(masks).cpu().numpy().view(np.uint32)
    ctx.close()
    wpr = (W + 31) // 32
    bits = np.zeros((n, H, wpr * 32), bool)
    bits[:, :, :W] = m != 0
    want = np.packbits(bits, axis=-1, bitorder="little").view("<u4").reshape(n, H, wpr)
    assert np.array_equal(got, want)
