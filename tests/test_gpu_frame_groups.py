"""A frame large enough that its fine carve goes by groups of bricks (Sec.
II-B-3), below the size at which groups take whole rows and above it: fine
occupancy, crossing edges (from the fine bitmap) and exit points of every ROI
against the oracle.  ROI lattices of any width leave partial bricks, groups and
bitmap words on every axis."""
import numpy as np
import pytest

import oracle
import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg,hf_um,n_cams", [
    (scenes.CFG_VOLLEYBALL, 6000, 16),    # 8-brick groups, one pass of 16 cameras
    (scenes.CFG_VOLLEYBALL, 3600, 9),     # whole-row groups
    (scenes.CFG_JUDO, 4000, 24),          # 8-brick groups, two passes
])
def test_frame_by_groups(cfg, hf_um, n_cams):
    import torch

    import paper_1903_11785_amd as fvv
    sc = scenes.make_scene(cfg, 0)
    masks, P = sc.masks[:n_cams], sc.P32[:n_cams]
    ref = oracle.frame(masks, P, sc.origin, sc.hc_um, hf_um, sc.coarse_dims, sc.t_np, sc.t_nb,
                       sc.n_steps)
    assert ref.fine_voxels >= 12288 * 1024
    coarse = fvv.Grid(origin=tuple(sc.origin), h=sc.hc, lo=(0, 0, 0), dims=sc.coarse_dims)
    max_fine = ref.fine_voxels + 1
    ctx = fvv.Context(max_cams=n_cams, max_w=sc.W, max_h=sc.H, max_coarse=coarse.size,
                      max_fine=max_fine, max_rois=64, max_points=1 << 22, max_jobs=64)
    params = fvv.frame_params(P, sc.W, sc.H, coarse, sc.hc_um, hf_um, sc.t_np, sc.t_nb, sc.n_steps)
    bufs = fvv.FrameBuffers(coarse, 64, max_fine, 1 << 22)
    bufs.occ_fine.fill_(7)
    sils = torch.empty((n_cams, sc.H, (sc.W + 31) // 32), dtype=torch.int32, device="cuda")
    ctx.frame(params, sils, bufs, masks=torch.from_numpy(masks).cuda())
    assert ctx.check() == fvv.FVV_OK
    K = len(ref.rois)
    assert bufs.counts.cpu().tolist() == [K, ref.fine_voxels, sum(len(k) for k in ref.keys), K]
    jobs, occ = bufs.jobs_host(K), bufs.occ_fine.cpu().numpy()
    keys, xyz = bufs.keys.cpu().numpy().view(np.uint32), bufs.xyz.cpu().numpy()
    off = bufs.point_off.cpu().numpy()
    for t, lat in enumerate(ref.fine):
        o = int(jobs[t]["out_offset"])
        np.testing.assert_array_equal(occ[o:o + lat.size], ref.occ_fine[t].reshape(-1))
        np.testing.assert_array_equal(keys[off[t]:off[t + 1]], ref.keys[t])
        d = np.abs(xyz[off[t]:off[t + 1]] - ref.xyz[t])
        assert d.max(initial=0) <= 1e-4 * float(lat.h)
    assert (occ[ref.fine_voxels:] == 7).all()
    ctx.close()
