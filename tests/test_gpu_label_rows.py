"""The labelling at the edges of its row listing (a wave per row-mask word up to
128 words, a thread per word beyond), of its row coordinates (65536 rows, the
most that stay in LDS) and of a thread per (neighbouring row, run): labels, ROI
boxes and smallest indices identical to the oracle's (Sec. II-B-2)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


# (nz, ny, nx): 128 and 129 words of 64 rows; 65536 rows with ny of 1, a prime
# and the most; one row past LDS; 4 runs per thread
@pytest.mark.parametrize("shape,density", [
    ((64, 128, 5), 0.05), ((43, 191, 9), 0.05), ((65536, 1, 3), 0.02), ((1, 65536, 3), 0.02),
    ((521, 125, 4), 0.01), ((65537, 1, 2), 0.02), ((6, 40, 250), 0.12)])
def test_label_rows(shape, density):
    import torch

    import paper_1903_11785_amd as fvv
    rng = np.random.default_rng(shape[0] + shape[1])
    occ = (rng.uniform(size=shape) < density).astype(np.uint8)
    occ[0, 0, 0] = occ[-1, -1, -1] = 1
    ref_occ, labels, rois, K = oracle.label(occ, 2, 50)
    ctx = fvv.Context(max_coarse=occ.size, max_fine=1, max_rois=1, max_points=1, max_jobs=1)
    d = torch.from_numpy(occ).cuda()
    grid = fvv.Grid(origin=(0.0, 0.0, 0.0), h=np.float32(1.0), lo=(0, 0, 0), dims=shape[::-1])
    lab, r, n = ctx.label(grid, d, t_np=2, t_nb=50, max_rois=max(K, 1))
    assert ctx.check() == fvv.FVV_OK and int(n.cpu()[0]) == K
    np.testing.assert_array_equal(lab.cpu().numpy(), labels)
    np.testing.assert_array_equal(d.cpu().numpy(), ref_occ)
    np.testing.assert_array_equal(r.cpu().numpy()[:K], rois)
    ctx.close()
