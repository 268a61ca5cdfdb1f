"""A batched carve of a lattice whose side is nearly 2^31 samples (Sec. II-B-3): the
units' row numbers reach past what a signed count holds; every byte as the kernel
that tests each sample against each camera (depth-1 tiles) writes it."""
import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu


def test_side_of_nearly_2_31():
    import torch

    import paper_1903_11785_amd as fvv
    sc = scenes.scene_tiny(3, 4)
    n, W, H, ny = 4, sc.W, sc.H, (1 << 31) - 5
    h = np.float32(1.5e-9)                 # a line of 3.2 m through the first ellipsoid
    jobs = np.zeros(1, fvv.JOB_DTYPE)
    jobs["origin"] = sc.ellipsoids[0].center - np.array([0, 1.6, 0])
    jobs["h"], jobs["dims"], jobs["n_cams"] = h, (1, ny, 1), n
    jobs["width"], jobs["height"] = W, H
    ctx = fvv.Context(max_cams=n, max_w=W, max_h=H, max_coarse=1, max_fine=1, max_rois=1,
                      max_points=1, max_jobs=1)
    sils = ctx.pack_silhouettes(torch.from_numpy(sc.masks).cuda())
    cams, jobs_d = fvv.cameras_to_device(sc.P32, W, H), fvv.jobs_to_device(jobs)
    out = [torch.full((ny + 3,), 7, dtype=torch.uint8, device="cuda") for _ in range(2)]
    ctx.carve_batched(jobs_d, 1, cams, sils, out[0], fvv.tile(64, 1))
    ctx.carve_batched(jobs_d, 1, cams, sils, out[1])
    assert ctx.check() == fvv.FVV_OK
    inside = int((out[0][:ny] == 1).sum())
    assert 0 < inside < ny and (out[0][ny:] == 7).all()
    assert torch.equal(out[0], out[1])
    ctx.close()
