"""The culled batched carve (zero, mark and carve passes over units of 16 sample
rows x 4 layers and tiles of 16 samples) at the edges of its units, tiles and
tables, byte for byte against the oracle (Sec. II-B-3), with the bytes between
the jobs' outputs untouched."""
import numpy as np
import pytest

import oracle
import scenes

pytestmark = pytest.mark.gpu

# edges of a tile (16), a unit (16 rows x 4 layers), a group of units (64 rows)
# and of 64 tiles' marks (1024 samples)
DIMS = [(1, 1, 1), (15, 16, 4), (16, 17, 5), (17, 15, 3), (33, 64, 8), (31, 65, 4), (257, 20, 9),
        (1030, 18, 5), (40, 130, 41)]


def _run(fvv, ctx, sc, h_um, dims_list, gap):
    import torch
    n, W, H = len(sc.cams), sc.W, sc.H
    h = scenes.um_to_h(h_um)
    ctr = np.round((sc.ellipsoids[0].center - np.asarray(sc.origin, float)) * 1e6 / h_um).astype(int)
    jobs = np.zeros(len(dims_list), fvv.JOB_DTYPE)
    off = gap
    for t, d in enumerate(dims_list):
        jobs[t]["origin"], jobs[t]["h"] = sc.origin, h
        jobs[t]["lo"] = ctr - np.asarray(d) // 2
        jobs[t]["dims"], jobs[t]["n_cams"] = d, n
        jobs[t]["width"], jobs[t]["height"] = W, H
        jobs[t]["out_offset"] = off
        off += int(np.prod(d)) + gap
    sils = ctx.pack_silhouettes(torch.from_numpy(sc.masks).cuda())
    cams = fvv.cameras_to_device(sc.P32, W, H)
    out = torch.full((off,), 7, dtype=torch.uint8, device="cuda")
    ctx.carve_batched(fvv.jobs_to_device(jobs), len(jobs), cams, sils, out)
    assert ctx.check() == fvv.FVV_OK
    return jobs, h, out.cpu().numpy()


def _check(sc, jobs, h, out, gap, seen):
    packed, at = oracle.pack(sc.masks), 0
    for j in jobs:
        o, d = int(j["out_offset"]), tuple(int(v) for v in j["dims"])
        lo = tuple(int(v) for v in j["lo"])
        assert o - at == gap and (out[at:o] == 7).all()
        if (lo, d) not in seen:
            seen[lo, d] = oracle.carve(sc.P32, packed, sc.W, sc.H,
                                       oracle.Lattice(origin=sc.origin, h=h, lo=lo, dims=d))[0]
        ref = seen[lo, d].reshape(-1)
        at = o + ref.size
        np.testing.assert_array_equal(out[o:at], ref, err_msg=f"dims {d}")
    assert out.size - at == gap and (out[at:] == 7).all()


@pytest.mark.parametrize("n_cams", [3, 4, 9])
@pytest.mark.parametrize("h_um", [10000, 20000, 120000])
def test_units_and_tiles_at_their_edges(n_cams, h_um):
    import paper_1903_11785_amd as fvv
    sc = scenes.scene_tiny(3, n_cams)
    ctx = fvv.Context(max_cams=n_cams, max_w=sc.W, max_h=sc.H, max_coarse=1, max_fine=1,
                      max_rois=1, max_points=1, max_jobs=2048)
    jobs, h, out = _run(fvv, ctx, sc, h_um, DIMS, 5)
    _check(sc, jobs, h, out, 5, {})
    ctx.close()


def test_more_jobs_than_the_tables_hold():
    import paper_1903_11785_amd as fvv
    sc = scenes.scene_tiny(4, 4)
    ctx = fvv.Context(max_cams=4, max_w=sc.W, max_h=sc.H, max_coarse=1, max_fine=1, max_rois=1,
                      max_points=1, max_jobs=2048)
    dims = [[(9, 5, 3), (20, 17, 6), (1, 40, 2)][t % 3] for t in range(1030)]
    jobs, h, out = _run(fvv, ctx, sc, 20000, dims, 3)
    _check(sc, jobs, h, out, 3, {})
    ctx.close()
