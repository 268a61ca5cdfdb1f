"""The labels' write pass, four samples at a time where the buffers' alignment
allows and one by one elsewhere, at the ends of its pieces and at every
alignment: labels and filtered occupancy identical to the oracle's (Sec.
II-B-2), the bytes around the buffers untouched."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


# (nz, ny, nx): below and above the size that goes four samples at a time, with
# remainders of 0 to 3 samples, and more samples than one sweep of the
# pass's workgroups (8 per CU, 256 threads, 16 samples)
@pytest.mark.parametrize("shape", [(1, 1, 1), (7, 9, 66), (16, 512, 512), (19, 401, 551),
                                   (13, 577, 563), (70, 401, 301)])
@pytest.mark.parametrize("occ_off,lab_off", [(0, 0), (1, 0), (0, 1), (4, 4), (3, 2)])
def test_label_write_alignments(shape, occ_off, lab_off):
    import torch

    import paper_1903_11785_amd as fvv
    rng = np.random.default_rng(sum(shape) + 7 * occ_off + lab_off)
    occ = (rng.uniform(size=shape) < 0.02).astype(np.uint8)
    occ.reshape(-1)[-1] = 1
    V = occ.size
    ctx = fvv.Context(max_coarse=V, max_fine=1, max_rois=1, max_points=1, max_jobs=1)
    ob = torch.full((V + 16,), 7, dtype=torch.uint8, device="cuda")
    lb = torch.full((V + 16,), -7, dtype=torch.int32, device="cuda")
    ob[occ_off:occ_off + V] = torch.from_numpy(occ.reshape(-1)).cuda()
    grid = fvv.Grid(origin=(0.0, 0.0, 0.0), h=np.float32(1.0), lo=(0, 0, 0), dims=shape[::-1])
    _, labels, _, _ = oracle.label(occ, 2, max_rois=1)
    ctx.label(grid, ob[occ_off:occ_off + V], t_np=2, max_rois=V,
              labels=lb[lab_off:lab_off + V])
    assert ctx.check() == fvv.FVV_OK
    o, l = ob.cpu().numpy(), lb.cpu().numpy()
    np.testing.assert_array_equal(l[lab_off:lab_off + V], labels.reshape(-1))
    np.testing.assert_array_equal(o[occ_off:occ_off + V], (labels.reshape(-1) != 0))
    assert (np.delete(o, np.s_[occ_off:occ_off + V]) == 7).all()
    assert (np.delete(l, np.s_[lab_off:lab_off + V]) == -7).all()
    ctx.close()
