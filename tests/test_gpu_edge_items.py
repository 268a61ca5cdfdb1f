"""Crossing edges of a lattice whose bitmap has more work items than the write
pass has workgroups (8 per CU, 256 words each), with empty items, an empty
start and an empty end among them: keys and count against numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("first,last", [(0, 9100), (40, 9099), (5000, 5001)])
def test_edges_over_many_items(first, last):
    import torch

    import paper_1903_11785_amd as fvv
    nx, ny, nz = 9, 64, 9100                 # one word per row: 582400 words, 2275 items
    rng = np.random.default_rng(first + last)
    occ = np.zeros((nz, ny, nx), np.uint8)
    for z in range(first, last, 37):         # blobs with many empty items between them
        occ[z:min(z + 3, last), 10:30, 2:7] = rng.integers(0, 2, (min(3, last - z), 20, 5))
    ctx = fvv.Context(max_cams=1, max_w=64, max_h=64, max_coarse=1, max_fine=occ.size, max_rois=1,
                      max_points=1 << 20, max_jobs=1)
    grid = fvv.Grid(origin=(0.0, 0.0, 0.0), h=np.float32(0.001), lo=(0, 0, 0), dims=(nx, ny, nz))
    P = np.array([[1, 0, 0, 0], [0, 1, 0, 0], [0, 0, 0, 1]], np.float32)
    sils = torch.zeros((1, 64, 2), dtype=torch.int32, device="cuda")
    lin = np.arange(occ.size, dtype=np.int64).reshape(occ.shape)
    want = np.sort(np.concatenate([
        3 * lin[:, :, :-1][occ[:, :, :-1] != occ[:, :, 1:]],
        3 * lin[:, :-1][occ[:, :-1] != occ[:, 1:]] + 1,
        3 * lin[:-1][occ[:-1] != occ[1:]] + 2]))
    keys, _, n = ctx.surface(grid, torch.from_numpy(occ).cuda(), P, 64, 64, sils, 4, 1 << 20)
    assert ctx.check() == fvv.FVV_OK
    assert int(n.cpu()[0]) == want.size
    np.testing.assert_array_equal(keys.cpu().numpy().view(np.uint32)[:want.size], want)
    ctx.close()
