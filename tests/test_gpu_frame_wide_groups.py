"""A frame whose fine carve goes by groups of up to 64 bricks (Sec. II-B-3, from 65536
tiles of 1024 samples on) with an ROI wider than a group (1024 samples), so that
a row takes two groups and the second is partial, and with more than 16 cameras:
fine occupancy, crossing edges and exit points against the oracle."""
import numpy as np
import pytest

import oracle
import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_cams", [5, 20])
def test_rows_of_two_wide_groups(n_cams):
    import torch

    import paper_1903_11785_amd as fvv
    cams = scenes.tiny_rig(n_cams)
    W, H = cams[0].W, cams[0].H
    body = scenes.Ellipsoid(center=np.array([0.02, -0.1, 0.03]), Q=np.eye(3),
                            axes=np.array([1.75, 0.35, 0.45]))
    masks = scenes.render_masks(cams, [body])
    P = np.stack([np.asarray(c.P32, np.float32) for c in cams])
    origin, hc_um, hf_um, dims = np.array([-2, -2, -1], np.float32), 62500, 3200, (64, 64, 32)
    ref = oracle.frame(masks, P, origin, hc_um, hf_um, dims)
    assert ref.fine_voxels >= 65536 * 1024
    assert max(int(lat.dims[0]) for lat in ref.fine) > 1024
    coarse = fvv.Grid(origin=tuple(origin), h=scenes.um_to_h(hc_um), lo=(0, 0, 0), dims=dims)
    points = sum(len(k) for k in ref.keys)
    max_fine, max_points = ref.fine_voxels + 1, points + 1
    ctx = fvv.Context(max_cams=n_cams, max_w=W, max_h=H, max_coarse=coarse.size,
                      max_fine=max_fine, max_rois=8, max_points=max_points, max_jobs=8)
    params = fvv.frame_params(P, W, H, coarse, hc_um, hf_um)
    bufs = fvv.FrameBuffers(coarse, 8, max_fine, max_points)
    bufs.occ_fine.fill_(7)
    sils = torch.empty((n_cams, H, (W + 31) // 32), dtype=torch.int32, device="cuda")
    ctx.frame(params, sils, bufs, masks=torch.from_numpy(masks).cuda())
    assert ctx.check() == fvv.FVV_OK
    K = len(ref.rois)
    assert bufs.counts.cpu().tolist() == [K, ref.fine_voxels, points, K]
    jobs, occ = bufs.jobs_host(K), bufs.occ_fine.cpu().numpy()
    keys, xyz = bufs.keys.cpu().numpy().view(np.uint32), bufs.xyz.cpu().numpy()
    off = bufs.point_off.cpu().numpy()
    for t, lat in enumerate(ref.fine):
        o = int(jobs[t]["out_offset"])
        np.testing.assert_array_equal(occ[o:o + lat.size], ref.occ_fine[t].reshape(-1))
        np.testing.assert_array_equal(keys[off[t]:off[t + 1]], ref.keys[t])
        assert np.abs(xyz[off[t]:off[t + 1]] - ref.xyz[t]).max(initial=0) <= 1e-4 * float(lat.h)
    assert (occ[ref.fine_voxels:] == 7).all()
    ctx.close()
