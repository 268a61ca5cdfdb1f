"""A batched carve of more jobs than one launch can give a workgroup each (2^32
threads are 1.7e7 workgroups, the zeroing's and the preparing's together, Sec.
II-B-3): every job one sample, byte for byte the samples of fvv_carve."""
import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu


def test_fifteen_million_jobs():
    import torch

    import paper_1903_11785_amd as fvv
    sc = scenes.scene_tiny(3, 4)
    n, W, H, h = 4, sc.W, sc.H, scenes.um_to_h(50000)
    n_jobs, dims = 15_000_000, (80, 80, 40)
    ctx = fvv.Context(max_cams=n, max_w=W, max_h=H, max_coarse=1, max_fine=1, max_rois=1,
                      max_points=1, max_jobs=n_jobs)
    sils = ctx.pack_silhouettes(torch.from_numpy(sc.masks).cuda())
    whole = ctx.carve(sc.P32, W, H, sils, fvv.Grid(tuple(sc.origin), h, (0, 0, 0), dims))
    whole = whole.reshape(-1)
    V = whole.numel()
    at = np.arange(n_jobs) % V
    jobs = np.zeros(n_jobs, fvv.JOB_DTYPE)
    jobs["origin"], jobs["h"], jobs["dims"] = sc.origin, h, (1, 1, 1)
    jobs["lo"] = np.stack([at % dims[0], at // dims[0] % dims[1], at // (dims[0] * dims[1])], 1)
    jobs["n_cams"], jobs["width"], jobs["height"] = n, W, H
    jobs["out_offset"] = np.arange(n_jobs)
    out = torch.full((n_jobs,), 7, dtype=torch.uint8, device="cuda")
    ctx.carve_batched(fvv.jobs_to_device(jobs), n_jobs, fvv.cameras_to_device(sc.P32, W, H), sils,
                      out)
    assert ctx.check() == fvv.FVV_OK
    assert 0 < int(whole.sum()) < V
    assert torch.equal(out, whole[torch.arange(n_jobs, device="cuda") % V])
    ctx.close()
