"""Jobs of a batched carve that write the same output bytes (a table that lists an
ROI more than once, Sec. II-B-3): the workgroups of one copy may overwrite what
those of another read, and the bytes are the ROI's own whatever their order."""
import numpy as np
import pytest

import oracle
import scenes

pytestmark = pytest.mark.gpu

DIMS = [(40, 130, 41), (17, 33, 9), (65, 20, 12)]


@pytest.mark.parametrize("copies", [2, 100])
def test_one_roi_listed_many_times(copies):
    import torch

    import paper_1903_11785_amd as fvv
    sc = scenes.scene_tiny(5, 4)
    n, W, H, h = 4, sc.W, sc.H, scenes.um_to_h(20000)
    ctr = np.round((sc.ellipsoids[0].center - np.asarray(sc.origin, float)) * 50).astype(int)
    jobs = np.zeros(len(DIMS), fvv.JOB_DTYPE)
    off, refs, packed = 0, [], oracle.pack(sc.masks)
    for t, d in enumerate(DIMS):
        lo = ctr - np.asarray(d) // 2
        jobs[t]["origin"], jobs[t]["h"], jobs[t]["lo"], jobs[t]["dims"] = sc.origin, h, lo, d
        jobs[t]["n_cams"], jobs[t]["width"], jobs[t]["height"] = n, W, H
        jobs[t]["out_offset"] = off
        off += int(np.prod(d))
        refs.append(oracle.carve(sc.P32, packed, W, H, oracle.Lattice(
            origin=sc.origin, h=h, lo=tuple(int(v) for v in lo), dims=d))[0].reshape(-1))
    table = np.concatenate([jobs] * copies)
    ctx = fvv.Context(max_cams=n, max_w=W, max_h=H, max_coarse=1, max_fine=1, max_rois=1,
                      max_points=1, max_jobs=len(table))
    sils = ctx.pack_silhouettes(torch.from_numpy(sc.masks).cuda())
    cams, jobs_d = fvv.cameras_to_device(sc.P32, W, H), fvv.jobs_to_device(table)
    for _ in range(5):
        out = torch.full((off + 3,), 7, dtype=torch.uint8, device="cuda")
        ctx.carve_batched(jobs_d, len(table), cams, sils, out)
        assert ctx.check() == fvv.FVV_OK
        o = out.cpu().numpy()
        np.testing.assert_array_equal(o[:off], np.concatenate(refs))
        assert (o[off:] == 7).all()
    ctx.close()
