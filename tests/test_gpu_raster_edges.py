"""The raster's tight boxes and shared reciprocals where they could go wrong:
slivers and nearly collinear triangles, triangles much smaller and much larger
than a pixel, vertices on pixel centres and edges, images past the width the
tight box allows, and projections outside the plain range of the quotients.
Depth images and masks bit-identical to the oracle (Sec. II-D, Eq. (4))."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _triangles(kind, rng, W, H, T):
    """Image positions [T][3][2] and depths [T][3]."""
    c = rng.uniform([-2, -2], [W + 2, H + 2], (T, 1, 2))
    if kind == "pixel":
        p = c + rng.uniform(-1.2, 1.2, (T, 3, 2))
    elif kind == "tiny":
        p = c + rng.uniform(-1, 1, (T, 3, 2)) * 10.0 ** rng.uniform(-5, -1, (T, 1, 1))
    elif kind == "large":
        p = c + rng.uniform(-40, 40, (T, 3, 2))
    elif kind == "sliver":
        d = rng.normal(size=(T, 1, 2))
        t = rng.uniform(-3, 3, (T, 3, 1))
        p = c + t * d + rng.normal(size=(T, 3, 2)) * 10.0 ** rng.uniform(-7, -2, (T, 1, 1))
    else:                                        # "grid": halves of pixels, shared edges
        p = np.round(2 * (c + rng.uniform(-2, 2, (T, 3, 2)))) / 2
    return p, rng.uniform(1, 4, (T, 3))


@pytest.mark.parametrize("kind", ["pixel", "tiny", "large", "sliver", "grid"])
@pytest.mark.parametrize("W,H,scale", [(97, 61, 1.0), (8192, 5, 1.0), (8193, 5, 1.0),
                                       (64, 48, 1e-25), (64, 48, 1e20)])
def test_raster_edges(kind, W, H, scale):
    import torch

    import paper_1903_11785_amd as fvv
    rng = np.random.default_rng(len(kind) + W)
    T = 4000
    p, z = _triangles(kind, rng, W, H, T)
    # camera 0: X / Z and Y / Z are the image position; camera 1: seen at an angle
    X = np.concatenate([p * z[..., None], z[..., None]], -1).reshape(-1, 3).astype(np.float32)
    P = np.array([[1, 0, 0, 0, 0, 1, 0, 0, 0, 0, 1, 0],
                  [1, 0.1, 0, 1, 0, 1, 0.2, -1, 0.0001, 0, 1, 0.5]]) * scale
    P = P.astype(np.float32)
    tris = np.arange(3 * T, dtype=np.uint32).reshape(T, 3)
    ref = oracle.depth(P, W, H, X, tris)
    ref_vis = oracle.visibility(P, W, H, X, tris, ref, 0.05 * scale)
    ctx = fvv.Context(max_cams=2, max_w=W, max_h=H, max_coarse=1, max_fine=1, max_rois=1,
                      max_points=1, max_jobs=1)
    n = lambda v: torch.tensor([v], dtype=torch.int32, device="cuda")
    depth, vis = ctx.visibility(P.reshape(2, 3, 4), W, H, torch.from_numpy(X).cuda(), n(3 * T),
                                torch.from_numpy(tris.view(np.int32)).cuda(), n(T), 0.05 * scale)
    np.testing.assert_array_equal(depth.cpu().numpy().view(np.uint32), ref.view(np.uint32))
    np.testing.assert_array_equal(vis.cpu().numpy().view(np.uint32), ref_vis)
    assert np.isfinite(ref).any()
    ctx.close()
