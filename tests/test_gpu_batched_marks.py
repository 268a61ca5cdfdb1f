"""Both routes of a culled batched carve (Sec. II-B-3) at their edges, byte for byte
against the oracle, with the bytes between the jobs untouched: strips of 4 rows up
to 12288 tiles of 64 x 4 x 4 samples (a job of up to 6 cameras counts twice), marks above; marks unit by unit up to 128 units
per CU, above in groups of 4 whose cameras are left at the first four that reject;
tables inside the LDS and past it.  The jobs' cameras (4, 9 and 17) and images
differ from job to job, so a workgroup that takes several units takes new cameras
with them."""
import numpy as np
import pytest

import oracle
import scenes

pytestmark = pytest.mark.gpu

# (frame, box): edges of a tile (16, 64), a strip (4), a unit (16 x 4), a group (64)
BOXES = [(t % 3, d) for t, d in enumerate(
    [(1, 1, 1), (15, 16, 4), (16, 17, 5), (17, 15, 3), (33, 64, 8), (31, 65, 4), (257, 20, 9),
     (65, 3, 7), (64, 5, 1), (40, 130, 41), (9, 129, 30), (5, 130, 61)])]


def _units(d):
    return 4 * -(-d[1] // 64) * -(-d[2] // 4)


def _tiles(f, d):
    return -(-d[0] // 64) * -(-d[1] // 4) * -(-d[2] // 4) * (2 if f == 0 else 1)


def _frames():
    """Three rigs and images of the tiny scenes: 4 cameras, 9 with cropped images, 17."""
    out = []
    for seed, n, w, h in [(3, 4, 320, 240), (4, 9, 301, 211), (5, 17, 320, 200)]:
        sc = scenes.scene_tiny(seed, n)
        out.append((sc, np.ascontiguousarray(sc.masks[:, :h, :w]), w, h))
    return out


@pytest.mark.parametrize("copies,marks,groups,lds", [
    (1, False, False, True),
    (7, False, False, True),
    (8, True, False, True),
    (68, True, False, True),
    (69, True, True, True),
    (85, True, True, True),
    (86, True, True, False),
])
@pytest.mark.parametrize("h_um", [10000, 60000])
def test_routes_at_their_edges(copies, marks, groups, lds, h_um):
    import torch

    import paper_1903_11785_amd as fvv
    n_cus = torch.cuda.get_device_properties(0).multi_processor_count
    table = BOXES * copies
    assert (sum(_tiles(f, d) for f, d in table) > 12288) == marks
    assert (sum(_units(d) for _, d in table) > 128 * n_cus) == groups
    assert (len(table) <= 1024) == lds
    frames, h, gap = _frames(), scenes.um_to_h(h_um), 5
    ctx = fvv.Context(max_cams=17, max_w=320, max_h=240, max_coarse=1, max_fine=1, max_rois=1,
                      max_points=1, max_jobs=len(table))
    sils, cams, at_sil, at_cam = [], [], [0], [0]
    for sc, masks, w, hh in frames:
        sils.append(ctx.pack_silhouettes(torch.from_numpy(masks).cuda()).reshape(-1))
        cams.append(fvv.cameras_to_device(sc.P32, w, hh).reshape(-1))
        at_sil.append(at_sil[-1] + sils[-1].numel())
        at_cam.append(at_cam[-1] + len(sc.P32))
    jobs, off, refs = np.zeros(len(table), fvv.JOB_DTYPE), 0, {}
    for t, (f, d) in enumerate(table):
        sc, masks, w, hh = frames[f]
        ctr = np.round((sc.ellipsoids[0].center - np.asarray(sc.origin, float)) * 1e6 / h_um)
        lo = tuple(int(v) for v in ctr.astype(int) - np.asarray(d) // 2)
        off += gap
        jobs[t]["origin"], jobs[t]["h"], jobs[t]["lo"], jobs[t]["dims"] = sc.origin, h, lo, d
        jobs[t]["cam_base"], jobs[t]["n_cams"] = at_cam[f], len(sc.P32)
        jobs[t]["sil_base"] = at_sil[f]
        jobs[t]["width"], jobs[t]["height"], jobs[t]["out_offset"] = w, hh, off
        off += int(np.prod(d))
        if (f, d) not in refs:
            refs[f, d] = oracle.carve(sc.P32, oracle.pack(masks), w, hh, oracle.Lattice(
                origin=sc.origin, h=h, lo=lo, dims=d))[0].reshape(-1)
    ref = np.full(off + gap, 7, np.uint8)
    for j, key in zip(jobs, table):
        ref[int(j["out_offset"]):int(j["out_offset"]) + refs[key].size] = refs[key]
    assert 0 < sum(int(r.sum()) for r in refs.values()) < sum(r.size for r in refs.values())
    out = torch.full((off + gap,), 7, dtype=torch.uint8, device="cuda")
    ctx.carve_batched(fvv.jobs_to_device(jobs), len(jobs), torch.cat(cams), torch.cat(sils), out)
    assert ctx.check() == fvv.FVV_OK
    np.testing.assert_array_equal(out.cpu().numpy(), ref)
    ctx.close()
