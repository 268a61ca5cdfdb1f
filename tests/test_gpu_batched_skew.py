"""Batched carves whose jobs' sizes lie far apart (Sec. II-B-3): a job longer than
the zeroing workgroups that its place in the table gives it is finished by the
ones that all jobs share.  The long jobs stand first, in the middle and last,
among more jobs than a table step holds, and beside a job out of range; every
job's bytes as fvv_carve writes them, those between the jobs untouched."""
import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu

PART = 128 * 4096          # bytes of a job that one of its own workgroups zeroes


@pytest.mark.parametrize("n_jobs,long_at,bad_at", [
    (300, [0], None),
    (300, [150, 299], 151),
    (1024, [1023], None),
    (1025, [0, 1024], 1),
    (2300, [5, 1023, 1024, 2299], 1025),
])
def test_long_jobs_among_short_ones(n_jobs, long_at, bad_at):
    import torch

    import paper_1903_11785_amd as fvv
    sc = scenes.scene_tiny(3, 4)
    n, W, H, h = 4, sc.W, sc.H, scenes.um_to_h(10000)
    n_cus = torch.cuda.get_device_properties(0).multi_processor_count
    parts = -(-16 * n_cus // n_jobs)
    ny = -(-parts * PART // (201 * 101)) + 3
    long_dims, short = (201, ny, 101), [(9, 5, 3), (20, 17, 6), (1, 40, 2)]
    assert np.prod(long_dims) > parts * PART + 8192
    ctr = np.round((sc.ellipsoids[0].center - np.asarray(sc.origin, float)) * 100).astype(int)
    jobs, at, gap = np.zeros(n_jobs, fvv.JOB_DTYPE), 0, 3
    for t in range(n_jobs):
        d = long_dims if t in long_at else short[t % 3]
        jobs[t]["origin"], jobs[t]["h"] = sc.origin, h
        jobs[t]["lo"], jobs[t]["dims"] = ctr - np.asarray(d) // 2, d
        jobs[t]["n_cams"], jobs[t]["width"], jobs[t]["height"] = n, W, H
        at += gap
        jobs[t]["out_offset"] = at
        at += int(np.prod(d))
    if bad_at is not None:
        jobs[bad_at]["n_cams"] = 0
    ctx = fvv.Context(max_cams=n, max_w=W, max_h=H, max_coarse=1, max_fine=1, max_rois=1,
                      max_points=1, max_jobs=n_jobs)
    sils = ctx.pack_silhouettes(torch.from_numpy(sc.masks).cuda())
    ref = torch.full((at + gap,), 7, dtype=torch.uint8, device="cuda")
    seen = {}
    for t, j in enumerate(jobs):
        d = tuple(int(v) for v in j["dims"])
        if d not in seen:
            grid = fvv.Grid(tuple(sc.origin), h, tuple(int(v) for v in j["lo"]), d)
            seen[d] = ctx.carve(sc.P32, W, H, sils, grid).reshape(-1)
        if t != bad_at:
            o = int(j["out_offset"])
            ref[o:o + seen[d].numel()] = seen[d]
    out = torch.full_like(ref, 7)
    ctx.carve_batched(fvv.jobs_to_device(jobs), n_jobs, fvv.cameras_to_device(sc.P32, W, H), sils,
                      out)
    assert ctx.check() == (fvv.FVV_OK if bad_at is None else fvv.FVV_EINVAL)
    assert 0 < int(seen[long_dims].sum()) < seen[long_dims].numel()
    assert torch.equal(out, ref)
    ctx.close()
