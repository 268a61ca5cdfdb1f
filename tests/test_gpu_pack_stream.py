"""Frames whose masks are streamed when packed (60 MB and more), and just below:
image sides with a short last block row and a half-used last word, against the
oracle -- the packed rows exactly, and through the fine occupancy and the edges
the 8 x 8-pixel blocks (and, with the two-pass coarse carve of the judo lattice,
the bits of the non-empty ones)."""
import numpy as np
import pytest

import oracle
import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg,n_cams,W,H,hc_um,streamed", [
    (scenes.CFG_JUDO, 9, 3824, 2157, 40000, True),
    (scenes.CFG_JUDO, 7, 3840, 2153, 40000, False),
    (scenes.CFG_JUDO, 8, 3840, 2153, 100000, True),      # one-pass coarse carve: no block bits
])
def test_frame_of_streamed_masks(cfg, n_cams, W, H, hc_um, streamed):
    import torch

    import paper_1903_11785_amd as fvv
    sc = scenes.make_scene(cfg, 0)
    masks, P = np.ascontiguousarray(sc.masks[:n_cams, :H, :W]), sc.P32[:n_cams]
    assert (masks.size >= 60 << 20) == streamed
    dims = tuple(int((d - 1) * sc.hc_um // hc_um) + 1 for d in sc.coarse_dims)
    hf_um = 20000
    ref = oracle.frame(masks, P, sc.origin, hc_um, hf_um, dims, sc.t_np, sc.t_nb, sc.n_steps)
    coarse = fvv.Grid(origin=tuple(sc.origin), h=np.float32(hc_um * 1e-6), lo=(0, 0, 0), dims=dims)
    max_fine = ref.fine_voxels + 1
    ctx = fvv.Context(max_cams=n_cams, max_w=W, max_h=H, max_coarse=coarse.size, max_fine=max_fine,
                      max_rois=64, max_points=1 << 20, max_jobs=64)
    params = fvv.frame_params(P, W, H, coarse, hc_um, hf_um, sc.t_np, sc.t_nb, sc.n_steps)
    bufs = fvv.FrameBuffers(coarse, 64, max_fine, 1 << 20)
    sils = torch.full((n_cams, H, (W + 31) // 32), -1, dtype=torch.int32, device="cuda")
    ctx.frame(params, sils, bufs, masks=torch.from_numpy(masks).cuda())
    assert ctx.check() == fvv.FVV_OK
    assert np.array_equal(sils.cpu().numpy().view(np.uint32), oracle.pack(masks))
    K = len(ref.rois)
    assert K > 0 and bufs.counts.cpu().tolist() == [K, ref.fine_voxels,
                                                    sum(len(k) for k in ref.keys), K]
    jobs, occ = bufs.jobs_host(K), bufs.occ_fine.cpu().numpy()
    keys, off = bufs.keys.cpu().numpy().view(np.uint32), bufs.point_off.cpu().numpy()
    for t, lat in enumerate(ref.fine):
        o = int(jobs[t]["out_offset"])
        np.testing.assert_array_equal(occ[o:o + lat.size], ref.occ_fine[t].reshape(-1))
        np.testing.assert_array_equal(keys[off[t]:off[t + 1]], ref.keys[t])
    ctx.close()
