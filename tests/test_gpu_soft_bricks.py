"""The soft hull at the edges of its kernels' work split against the float64
oracle: camera counts around the four waves' shares (1..17, 32), lattices that
are no multiple of a brick's four samples a side or of the forward's 64, one
whose bricks' pixel windows do not fit the LDS (samples tens of pixels apart) and one that reaches beyond the images; and, against its own slabs,
one of many bricks per workgroup.

Tolerances as for the whole scene: 1e-4 on o, 1e-5 relative on the loss, 1e-3 of the norm
on the logits' gradient and, per camera, on the pose gradient, relative to the larger of its own
norm and the rig's mean (fp32 projections against fp64)."""
import numpy as np
import pytest

import scenes
from oracle import soft as osoft

pytestmark = pytest.mark.gpu

CASES = [  # cameras, samples per axis, spacing relative to the scene's
    (1, (1, 1, 1), 1.0), (2, (4, 4, 4), 1.0), (3, (5, 3, 2), 2.0), (4, (64, 1, 1), 1.0),
    (5, (65, 1, 3), 1.0), (15, (9, 13, 7), 3.0), (16, (13, 11, 6), 8.0), (17, (3, 70, 5), 1.0),
    (32, (21, 18, 17), 2.0), (6, (12, 12, 12), 16.0),
]


@pytest.mark.parametrize("n,dims,step", CASES)
def test_soft_hull_at_the_edges_of_the_split(n, dims, step):
    import torch
    import paper_1903_11785_amd as fvv
    from paper_1903_11785_amd.soft import SoftHull
    s = scenes.scene_soft(n, n_cams=n)
    K, R0, t0 = s.base_pose()
    h = np.float32(s.h * step)
    mid = np.asarray(s.origin) + s.h * (np.asarray(s.lo) + (np.asarray(s.dims) - 1) / 2)
    lo = tuple(int(v) for v in -(np.asarray(dims) // 2))
    origin = tuple(np.float32(v) for v in mid)
    V = int(np.prod(dims))
    target = np.random.default_rng(n).random(V).astype(np.float32)
    ctx = fvv.Context(max_cams=32, max_w=640, max_h=480, max_coarse=1, max_fine=1, max_rois=1,
                      max_points=1, max_jobs=1)
    hull = SoftHull(ctx, fvv.Grid(origin=origin, h=h, lo=lo, dims=dims), K, R0, t0, s.W, s.H)
    L = torch.from_numpy(s.logits).cuda().requires_grad_(True)
    w = torch.from_numpy(s.omega).requires_grad_(True)
    t = torch.from_numpy(s.tau).requires_grad_(True)
    with torch.no_grad():
        o = hull.occupancy(L, w, t).cpu().numpy()
    loss = hull.l2_loss(L, w, t, torch.from_numpy(target).cuda())
    gL, gw, gt = (g.cpu().numpy() for g in torch.autograd.grad(loss, (L, w, t)))
    ref, ref_loss = osoft.soft_forward(s.logits, K, R0, t0, s.omega, s.tau, origin, h, lo, dims, target)
    _, rL, rw, rt = osoft.soft_grad(s.logits, K, R0, t0, s.omega, s.tau, origin, h, lo, dims,
                                    target=target)
    ctx.close()
    pose, rpose = np.concatenate([gw, gt], 1), np.concatenate([rw, rt], 1)
    scale = np.linalg.norm(rpose, axis=1)
    ep = np.linalg.norm(pose - rpose, axis=1) / np.maximum(np.maximum(scale, scale.mean()), 1e-30)
    eL = np.linalg.norm(gL - rL) / max(np.linalg.norm(rL), 1e-30)
    print(n, dims, step, "o", np.abs(o - ref).max(), "logits", eL, "pose", ep.max())
    assert np.abs(o - ref).max() < 1e-4
    assert abs(float(loss.detach()) - ref_loss) <= 1e-5 * ref_loss
    assert eL < 1e-3 and ep.max() < 1e-3


def test_many_bricks_per_workgroup_are_the_sum_of_their_slabs():
    """The gradients of a lattice of more bricks than workgroups are the sums
    of those of its slabs, which have a workgroup per brick.  Both take the
    same bricks and projections (so the pose derivative's jumps at pixel
    centres are on the same side): a camera's pose sums differ by the order of
    double additions only, 1e-9 of their norm; the logits' by the order of
    float atomics over up to 1e4 terms of either sign, 1e-4."""
    import torch
    import paper_1903_11785_amd as fvv
    n, dims, slab = 4, (96, 96, 72), 8
    s = scenes.scene_soft(n, n_cams=n)
    K, R0, t0 = s.base_pose()
    h = np.float32(s.h * 0.5)
    origin = tuple(np.float32(v) for v in
                   np.asarray(s.origin) + s.h * (np.asarray(s.lo) + (np.asarray(s.dims) - 1) / 2))
    ctx = fvv.Context(max_cams=32, max_w=640, max_h=480, max_coarse=1, max_fine=1, max_rois=1,
                      max_points=1, max_jobs=1)
    cams = fvv.soft_cameras(K, R0, t0, s.omega, s.tau)
    L = torch.from_numpy(s.logits).cuda()
    target = torch.from_numpy(np.random.default_rng(n).random(np.prod(dims)).astype(np.float32)).cuda()

    def grads(z0, z1):
        grid = fvv.Grid(origin=origin, h=h, lo=(-48, -48, z0 - 36), dims=(96, 96, z1 - z0))
        gl, gp = torch.empty_like(L), torch.empty((n, 6), dtype=torch.float64, device="cuda")
        loss = torch.empty(1, dtype=torch.float64, device="cuda")
        part = target[z0 * 96 * 96:z1 * 96 * 96].contiguous()
        ctx.soft_forward(grid, cams, s.W, s.H, L, target=part, loss=loss)
        ctx.soft_backward(grid, cams, s.W, s.H, L, gl, gp, target=part)
        return gl.double(), gp, loss

    whole = grads(0, dims[2])
    parts = [grads(z, z + slab) for z in range(0, dims[2], slab)]
    ctx.close()
    for q, tol in ((0, 1e-4), (1, 1e-9), (2, 1e-9)):
        total = sum(p[q] for p in parts)
        err = float(torch.linalg.norm(whole[q] - total) / torch.linalg.norm(total))
        print(q, err)
        assert err < tol
