"""Timed cases of the visual-hull library: the work a program has it do, through the public calls
of the Python binding.

Every input is made on the GPU from (case, seed): a camera rig around a volume, people (five
ellipsoids each) or plain ellipsoids in it, and each camera's silhouettes, rendered analytically in
float64.  Sizes are those of the repository's benchmark and tests, and odd ones of the same ranges.

  frame       one multi-camera frame, masks in, ROIs, fine occupancy, edges and exit points out
  calls       packing, carving and labelling of a whole volume as separate calls
  roi         carving, exit points and triangles of one ROI as separate calls
  batched     many ROIs of many frames carved in one launch
  visibility  depth images and per-triangle visibility of a frame's mesh
  soft        one optimisation step of the differentiable soft hull
"""
import math

import numpy as np
import torch

import paper_1903_11785_amd as fvv
from paper_1903_11785_amd.soft import SoftHull

DEV = "cuda"
CALIB = (0.94, 1.25)        # focal length over image width of the court rigs
PERSON_M3 = 0.37            # volume of a person's ROI box, and the surface it holds (m^2)
PERSON_M2 = 1.9
TESTS = 6                   # cameras a sample is tested against until one rejects it


# ---------------------------------------------------------------------------- the cases
def _frame(name, cams, width, height, people, vol, hc_mm, hf_mm, **more):
    case = dict(name=name, kind="frame", cams=cams, width=width, height=height, people=people,
                vol_x=vol[0], vol_y=vol[1], vol_z=vol[2], hc_um=int(hc_mm * 1000),
                hf_um=int(hf_mm * 1000), pairs=False, noise=0.0, masks=True, graph=True,
                in_flight=1, mesh=False, bresenham=False)
    case.update(more)
    return case


def listed():
    return [
        # the smallest frame: four small cameras, two objects.  Launch-bound.
        _frame("frame_tiny", 4, 320, 240, 0, (4, 4, 2), 62.5, 20),
        # the benchmark's frame, one at a time: a frame's latency in a live broadcast
        _frame("frame_volleyball", 16, 1920, 1080, 12, (18, 9, 4), 100, 10),
        # the same as a serving loop runs it: four frames in flight, a stream each
        _frame("serve_volleyball", 16, 1920, 1080, 12, (18, 9, 4), 100, 10, in_flight=4),
        # a large volume at the paper's own lattice (360 x 360 x 180), few 4K cameras
        _frame("frame_large_volume", 10, 3840, 2160, 14, (18, 18, 9), 50, 20),
        # many 4K cameras, touching people, noisy silhouettes
        _frame("frame_judo", 24, 3840, 2160, 4, (10, 10, 3), 40, 5, pairs=True, noise=0.01),
        # the largest frame: the same at 2 mm, over 1e8 fine samples
        _frame("frame_judo_2mm", 24, 3840, 2160, 4, (10, 10, 3), 40, 2, pairs=True, noise=0.01),
        # a frame with its triangles, eagerly, from silhouettes packed by the segmentation,
        # with the paper's own estimator; image sides that are no multiple of 8
        _frame("frame_mesh_odd", 12, 1278, 717, 6, (12, 9, 3), 80, 12.5, graph=False, masks=False,
               mesh=True, bresenham=True),
        # a program that wants the coarse hull only, call by call, at odd sizes
        dict(name="coarse_calls", kind="calls", cams=9, width=1279, height=719, people=6,
             vol_x=13, vol_y=9, vol_z=3, hc_um=70000),
        # one person's ROI call by call: carve, exit points, triangles
        dict(name="roi_calls", kind="roi", cams=16, width=1920, height=1080, h_um=10000, steps=8),
        # many recorded frames' ROIs at once, the tile the tuner picks for them
        dict(name="batched_rois", kind="batched", cams=4, width=320, height=240, frames=64,
             rois=12, h_um=10000, edge_lo=0.6, edge_hi=2.5, tx=16, blocks=16384),
        # what rendering needs of a finished mesh
        dict(name="visibility", kind="visibility", cams=16, width=1920, height=1080, people=12,
             vol_x=18, vol_y=9, vol_z=4, hc_um=100000, hf_um=10000, t_v=0.1),
        # refining silhouettes and calibration by gradient descent: loss and its gradients
        dict(name="soft_step", kind="soft", cams=16, width=320, height=240, h_um=20000),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _image(rng, lo, hi):
    """An image size: as cameras give it, or cut to an odd region of interest."""
    w = int(_log(rng, lo, hi))
    h = int(w * rng.uniform(0.5, 0.6))
    if rng.random() < 0.5:
        w, h = max(64, w // 32 * 32), max(48, h // 8 * 8)
    return w, h


def draw(rng):
    kind = rng.choice(["frame"] * 6 + ["calls", "roi", "batched", "visibility", "soft"])
    if kind == "frame":
        w, h = _image(rng, 320, 3840)
        people = rng.randint(1, 14)
        small = people <= 4
        vol = ((rng.randint(8, 10), rng.randint(8, 10), 3) if small else
               (rng.randint(14, 18), rng.randint(9, 12), rng.randint(3, 6)))
        hf = _log(rng, 3 if small else 5, 25)
        return {k: v for k, v in _frame(
            "", rng.randint(4 if small else 8, 32), w, h, people, vol,
            round(_log(rng, max(45, 2 * hf), 120), 1), round(hf, 1), pairs=small and people > 1,
            noise=rng.choice([0.0, 0.01]), masks=rng.random() < 0.75, graph=rng.random() < 0.75,
            mesh=rng.random() < 0.3, bresenham=rng.random() < 0.2).items() if k != "name"}
    if kind == "calls":
        w, h = _image(rng, 320, 3840)
        return dict(kind=kind, cams=rng.randint(4, 32), width=w, height=h,
                    people=rng.randint(1, 14), vol_x=rng.randint(12, 18), vol_y=rng.randint(9, 18),
                    vol_z=rng.randint(3, 6), hc_um=int(_log(rng, 55000, 120000)))
    if kind == "roi":
        w, h = _image(rng, 320, 3840)
        return dict(kind=kind, cams=rng.randint(4, 32), width=w, height=h,
                    h_um=int(_log(rng, 3000, 40000)), steps=rng.randint(6, 9))
    if kind == "batched":
        w, h = _image(rng, 200, 640)
        return dict(kind=kind, cams=rng.randint(4, 12), width=w, height=h,
                    frames=int(_log(rng, 2, 64)), rois=rng.randint(1, 12),
                    h_um=int(_log(rng, 10000, 25000)), edge_lo=0.5, edge_hi=rng.uniform(1.0, 2.5),
                    tx=rng.choice([16, 32, 64]), blocks=rng.choice([0, 2048, 16384]))
    if kind == "visibility":
        w, h = _image(rng, 640, 2560)
        return dict(kind=kind, cams=rng.randint(6, 24), width=w, height=h,
                    people=rng.randint(4, 12), vol_x=rng.randint(14, 18), vol_y=9, vol_z=4,
                    hc_um=100000, hf_um=int(_log(rng, 8000, 25000)),
                    t_v=round(rng.uniform(0.02, 0.3), 3))
    w, h = _image(rng, 200, 640)
    return dict(kind="soft", cams=rng.randint(4, 32), width=w, height=h,
                h_um=int(_log(rng, 10000, 30000)))


# ---------------------------------------------------------------------------- scenes
def _rng(seed, what):
    return np.random.Generator(np.random.PCG64([int(seed), what]))


def _rot(axis, a):
    c, s = math.cos(a), math.sin(a)
    m = np.eye(3)
    i, j = [(1, 2), (2, 0), (0, 1)][axis]
    m[i, i] = m[j, j] = c
    m[i, j], m[j, i] = -s, s
    return m


def _look_at(C, target, f, W, H):
    """(P float32 [3][4], K, R, C) of a camera at C looking at target, world z up."""
    C = np.asarray(C, np.float64)
    fwd = np.asarray(target, np.float64) - C
    fwd /= np.linalg.norm(fwd)
    right = np.cross(fwd, [0.0, 0.0, 1.0])
    right /= np.linalg.norm(right)
    R = np.stack([right, np.cross(fwd, right), fwd])
    K = np.array([[f, 0, W / 2], [0, f, H / 2], [0, 0, 1]], np.float64)
    return (K @ np.hstack([R, (-R @ C)[:, None]])).astype(np.float32), K, R, C


def _court_rig(case, seed, lo, hi):
    """Cameras around the volume, each as near as keeps the volume in its image."""
    rng = _rng(seed, 0)
    n, W, H = case["cams"], case["width"], case["height"]
    t = (lo + hi) / 2
    pts = np.array([[x, y, z] for x in (lo[0], hi[0]) for y in (lo[1], hi[1])
                    for z in (lo[2], hi[2])])
    rig = []
    for k in range(n):
        az = 2 * math.pi * k / n + math.radians(rng.uniform(-5, 5))
        z, f = rng.uniform(3, 8), W * rng.uniform(*CALIB)

        def at(d):
            return _look_at([t[0] + d * math.cos(az), t[1] + d * math.sin(az), z], t, f, W, H)

        near, far = 0.5, 1000.0
        for _ in range(40):
            d = (near + far) / 2
            _, K, R, C = at(d)
            q = (pts - C) @ R.T @ K.T
            ok = (q[:, 2] > 0.1).all()
            if ok:
                u, v = q[:, 0] / q[:, 2], q[:, 1] / q[:, 2]
                ok = (u.min() >= 0.02 * W and u.max() <= 0.98 * W and v.min() >= 0.02 * H
                      and v.max() <= 0.98 * H)
            near, far = (near, d) if ok else (d, far)
        rig.append(at(far))
    return rig


def _ring(n, W, H):
    return [_look_at([6 * math.cos(2 * math.pi * k / n), 6 * math.sin(2 * math.pi * k / n), 0.0],
                     [0, 0, 0], 300.0 * W / 320, W, H) for k in range(n)]


def _balls(rng, n, spread):
    """n ellipsoids (centre, principal axes, semi-axes)."""
    out = []
    for _ in range(n):
        Q = np.linalg.qr(rng.normal(size=(3, 3)))[0]
        out.append((rng.uniform(-1, 1, 3) * spread, Q, rng.uniform(0.2, 0.5, 3)))
    return out


def _half(e):
    return np.sqrt(((e[1] * e[2]) ** 2).sum(1))


def _person(rng, xy, yaw, tilt, lift):
    s = rng.uniform(0.9, 1.1)
    parts = [([0, 0, 0.45], np.eye(3), [0.18, 0.12, 0.45]),
             ([0, 0, 1.20], np.eye(3), [0.20, 0.13, 0.32]),
             ([0, 0, 1.68], np.eye(3), [0.10, 0.10, 0.12])]
    for side in (1.0, -1.0):
        Q = _rot(0, side * math.radians(rng.uniform(0, 150)))
        parts.append((np.array([0, side * 0.24, 1.45]) + 0.32 * (Q @ [0.0, 0.0, -1.0]), Q,
                      [0.05, 0.05, 0.32]))
    R = _rot(2, yaw) @ _rot(1, tilt)
    out = [(R @ np.asarray(c, float) * s, R @ Q, np.asarray(a, float) * s) for c, Q, a in parts]
    dz = 0.02 - min((e[0] - _half(e))[2] for e in out) + lift
    return [(c + np.array([xy[0], xy[1], dz]), Q, a) for c, Q, a in out]


def _people(case, seed, lo, hi):
    """The people of a frame: spread over the court, or in touching pairs."""
    rng = _rng(seed, 1)
    n, out, spots = case["people"], [], []
    pairs = case.get("pairs", False)
    gap = 2.5 if pairs else 1.0
    tries = 0
    while len(spots) < (-(-n // 2) if pairs else n):
        p = np.array([rng.uniform(lo[a] + 1.0, hi[a] - 1.0) for a in (0, 1)])
        tries += 1
        if tries > 2000 or all(np.linalg.norm(p - q) >= gap for q in spots):
            spots.append(p)
    for k in range(n):
        tilt, lift, yaw = 0.0, 0.0, rng.uniform(0, 2 * math.pi)
        xy = spots[k // 2 if pairs else k]
        if pairs:
            tilt = math.radians(rng.uniform(45, 90)) if rng.uniform() < 0.3 else 0.0
            yaw = k * math.pi + 0.7 * (k // 2)
            xy = xy + (0.19 if k % 2 else -0.19) * np.array([math.cos(yaw), math.sin(yaw)])
        elif rng.uniform() < 0.25:
            lift = rng.uniform(0.2, 0.8)
        out += _person(rng, xy, yaw, tilt, lift)
    return out


def _render(rig, ells, W, H):
    """uint8 [N][H][W] on the GPU: 1 where the ray through a pixel's centre hits an ellipsoid."""
    out = torch.zeros((len(rig), H, W), dtype=torch.uint8, device=DEV)
    px = torch.arange(W, device=DEV, dtype=torch.float64) + 0.5
    py = torch.arange(H, device=DEV, dtype=torch.float64) + 0.5
    for c, (_, K, R, C) in enumerate(rig):
        ux, uy = ((px - K[0, 2]) / K[0, 0])[None, :], ((py - K[1, 2]) / K[1, 1])[:, None]
        for ctr, Q, ax in ells:
            h = _half((ctr, Q, ax))
            box = ctr + h * np.array([[x, y, z] for x in (-1, 1) for y in (-1, 1)
                                      for z in (-1, 1)])
            q = (box - C) @ R.T @ K.T
            if (q[:, 2] <= 0).any():
                continue
            u, v = q[:, 0] / q[:, 2], q[:, 1] / q[:, 2]
            x0, x1 = max(int(u.min()) - 2, 0), min(int(u.max()) + 3, W)
            y0, y1 = max(int(v.min()) - 2, 0), min(int(v.max()) + 3, H)
            if x0 >= x1 or y0 >= y1:
                continue
            M = Q @ np.diag(1 / ax ** 2) @ Q.T
            e = C - ctr
            g = float(e @ M @ e - 1)
            m, b = R @ M @ R.T, R @ (M @ e)
            x, y = ux[:, x0:x1], uy[y0:y1]
            A = (m[0, 0] * x * x + 2 * m[0, 2] * x) + (m[1, 1] * y * y + 2 * m[1, 2] * y
                                                       + m[2, 2]) + 2 * m[0, 1] * x * y
            B = b[0] * x + (b[1] * y + b[2])
            out[c, y0:y1, x0:x1] |= ((B * B >= A * g) & (B < 0)).to(torch.uint8)
    return out


def _flip_boundary(masks, share, seed):
    """Flip a share of each silhouette's boundary pixels (segmentation noise)."""
    edge = torch.zeros_like(masks, dtype=torch.bool)
    dx, dy = masks[:, :, 1:] != masks[:, :, :-1], masks[:, 1:] != masks[:, :-1]
    edge[:, :, 1:] |= dx
    edge[:, :, :-1] |= dx
    edge[:, 1:] |= dy
    edge[:, :-1] |= dy
    at = edge.nonzero()
    g = torch.Generator(DEV).manual_seed(int(seed))
    at = at[torch.rand(at.shape[0], generator=g, device=DEV) < share]
    masks[at[:, 0], at[:, 1], at[:, 2]] ^= 1
    return masks


def _scene(case, seed):
    """(P, masks, ellipsoids, coarse grid) of one frame."""
    size = np.array([case["vol_x"], case["vol_y"], case["vol_z"]], float)
    if case["people"]:
        lo = np.array([-size[0] / 2, -size[1] / 2, 0.0])
        ells = _people(case, seed, lo, lo + size)
    else:
        lo = -size / 2
        ells = _balls(_rng(seed, 1), 2, size * [0.35, 0.35, 0.2])
    rig = _court_rig(case, seed, lo, lo + size)
    masks = _render(rig, ells, case["width"], case["height"])
    if case.get("noise"):
        masks = _flip_boundary(masks, case["noise"], seed)
    um = case["hc_um"]
    dims = tuple(int(-(-round(s * 1e6) // um)) for s in size)
    coarse = fvv.Grid(tuple(lo.astype(np.float32)), np.float32(um * 1e-6), (0, 0, 0), dims)
    return np.stack([r[0] for r in rig]), masks, ells, coarse


def _fine_samples(case):
    """About how many fine samples a frame's ROIs hold."""
    return (max(case["people"], 2) * PERSON_M3) / (case["hf_um"] * 1e-6) ** 3


# ---------------------------------------------------------------------------- prepare
def _frame_slot(case, seed):
    P, masks, _, coarse = _scene(case, seed)
    n, H, W = masks.shape
    max_fine = 1 << int(math.ceil(math.log2(2.5 * _fine_samples(case) + (1 << 22))))
    edges = max(case["people"], 2) * PERSON_M2 / (case["hf_um"] * 1e-6) ** 2
    max_points = 1 << int(math.ceil(math.log2(2.5 * edges + (1 << 18))))
    ctx = fvv.Context(max_cams=n, max_w=W, max_h=H, max_coarse=coarse.size, max_fine=max_fine,
                      max_rois=256, max_points=max_points, max_jobs=256)
    params = fvv.frame_params(
        P, W, H, coarse, case["hc_um"], case["hf_um"],
        exit_estimator=fvv.EXIT_BRESENHAM if case["bresenham"] else fvv.EXIT_BISECTION)
    sils = torch.empty((n, H, (W + 31) // 32), dtype=torch.int32, device=DEV)
    if not case["masks"]:
        ctx.pack_silhouettes(masks, out=sils)
        masks = None
    bufs = fvv.FrameBuffers(coarse, 256, max_fine, max_points,
                            max_tris=2 * max_points if case["mesh"] else 0)
    slot = dict(ctx=ctx, params=params, sils=sils, bufs=bufs, masks=masks, P=P, coarse=coarse)
    if case["graph"]:
        slot["graph"] = ctx.frame_graph(params, sils, bufs, masks=masks)
    return slot


def _prepare_frame(case, seed):
    slots = [_frame_slot(case, seed + 7919 * k) for k in range(case["in_flight"])]
    st = dict(slots=slots)
    if len(slots) > 1:
        st["streams"] = [torch.cuda.Stream() for _ in slots]
        st["done"] = [torch.cuda.Event() for _ in slots]
    return st


def _prepare_calls(case, seed):
    P, masks, _, coarse = _scene(case, seed)
    n, H, W = masks.shape
    ctx = fvv.Context(max_cams=n, max_w=W, max_h=H, max_coarse=coarse.size, max_fine=1,
                      max_rois=256, max_points=1, max_jobs=1)
    return dict(ctx=ctx, P=P, masks=masks, W=W, H=H, coarse=coarse,
                sils=torch.empty((n, H, (W + 31) // 32), dtype=torch.int32, device=DEV),
                occ=torch.empty(coarse.shape, dtype=torch.uint8, device=DEV),
                labels=torch.empty(coarse.shape, dtype=torch.int32, device=DEV),
                rois=torch.zeros((256, 8), dtype=torch.int32, device=DEV),
                n_rois=torch.zeros(1, dtype=torch.int32, device=DEV))


def _roi_scene(case, seed):
    """One person in a court's rig and the lattice around them."""
    lo, hi = np.array([-9.0, -4.5, 0.0]), np.array([9.0, 4.5, 4.0])
    rng = _rng(seed, 1)
    ells = _person(rng, rng.uniform([-7, -3], [7, 3]), rng.uniform(0, 2 * math.pi), 0.0, 0.0)
    rig = _court_rig(case, seed, lo, hi)
    masks = _render(rig, ells, case["width"], case["height"])
    a = np.min([e[0] - _half(e) for e in ells], 0) - 0.1 - lo
    b = np.max([e[0] + _half(e) for e in ells], 0) + 0.1 - lo
    h = case["h_um"] * 1e-6
    first = np.floor(a / h).astype(int)
    dims = np.ceil(b / h).astype(int) - first + 1
    grid = fvv.Grid(tuple(lo.astype(np.float32)), np.float32(h), tuple(int(v) for v in first),
                    tuple(int(v) for v in dims))
    return np.stack([r[0] for r in rig]), masks, grid


def _prepare_roi(case, seed):
    P, masks, grid = _roi_scene(case, seed)
    n, H, W = masks.shape
    # buffers with room for any person's ROI, as a program keeps them
    points = int(4 * PERSON_M2 / (case["h_um"] * 1e-6) ** 2) + 4096
    room = int(5.0 / (case["h_um"] * 1e-6) ** 3) + (1 << 16)
    ctx = fvv.Context(max_cams=n, max_w=W, max_h=H, max_coarse=1, max_fine=room,
                      max_rois=1, max_points=points, max_jobs=1)
    z = lambda shape, dt=torch.int32: torch.zeros(shape, dtype=dt, device=DEV)
    buf = z(room, torch.uint8)
    return dict(ctx=ctx, P=P, W=W, H=H, grid=grid, steps=case["steps"],
                sils=ctx.pack_silhouettes(masks), buf=buf, occ=buf[:grid.size].view(grid.shape),
                keys=z(points), xyz=z((points, 3), torch.float32), n_points=z(1),
                tris=z((2 * points, 3)), n_tris=z(1))


def _prepare_batched(case, seed):
    n, W, H = case["cams"], case["width"], case["height"]
    rig = _ring(n, W, H)
    P = np.stack([r[0] for r in rig])
    size, h = np.array([4.0, 4.0, 2.0]), case["h_um"] * 1e-6
    rng, box = _rng(seed, 3), _rng(0, 5)     # the boxes' sizes are the case's
    masks, boxes = [], []
    for f in range(case["frames"]):
        masks.append(_render(rig, _balls(rng, 2, [1.4, 1.4, 0.4]), W, H))
        for _ in range(case["rois"]):
            dims = np.maximum(np.round(box.uniform(case["edge_lo"], case["edge_hi"], 3) / h), 1)
            lo = np.round(rng.uniform(0, size) / h) - dims // 2
            boxes.append((f, [int(v) for v in lo], [int(v) for v in dims]))
    ctx = fvv.Context(max_cams=n, max_w=W, max_h=H, max_coarse=1, max_fine=1, max_rois=1,
                      max_points=1, max_jobs=len(boxes))
    sils = ctx.pack_silhouettes(torch.cat(masks))
    jobs, total = fvv.frame_major_jobs(boxes, [tuple((-size / 2).astype(np.float32))] * len(masks),
                                       [np.float32(h)] * len(masks), n, W, H)
    st = dict(ctx=ctx, sils=sils, jobs=fvv.jobs_to_device(jobs),
              cams=fvv.cameras_to_device(np.concatenate([P] * len(masks)), W, H),
              out=torch.zeros(total, dtype=torch.uint8, device=DEV))
    st["graph"] = ctx.carve_batched_graph(st["jobs"], len(boxes), st["cams"], sils, st["out"],
                                          fvv.tile(case["tx"], 4, case["blocks"]))
    return st


def _prepare_visibility(case, seed):
    frame = dict(_frame("", 1, 1, 1, 1, (1, 1, 1), 1, 1), **case)
    frame.update(mesh=True, graph=False)
    s = _frame_slot(frame, seed)
    s["ctx"].frame(s["params"], s["sils"], s["bufs"], masks=s["masks"])
    torch.cuda.synchronize()
    b = s["bufs"]
    k = int(b.counts[0])
    n, W, H = case["cams"], case["width"], case["height"]
    # the mesh as a frame leaves it: buffers with room, the numbers in use on the device
    return dict(ctx=s["ctx"], P=s["P"], W=W, H=H, t_v=case["t_v"], xyz=b.xyz, tris=b.tris,
                n_p=b.counts[2:3], n_t=b.tri_off[k:k + 1],
                depth=torch.empty((n, H, W), dtype=torch.float32, device=DEV),
                vis=torch.zeros(b.tris.shape[0], dtype=torch.int32, device=DEV))


def _prepare_soft(case, seed):
    n, W, H = case["cams"], case["width"], case["height"]
    rig, rng = _ring(n, W, H), _rng(seed, 4)
    ells = _balls(rng, 2, [1.2, 1.2, 0.3])
    s = _render(rig, ells, W, H).float()[:, None]
    for _ in range(2):
        s = torch.nn.functional.avg_pool2d(torch.nn.functional.pad(s, (1, 1, 1, 1),
                                                                   mode="replicate"), 3, 1)
    g = torch.Generator(DEV).manual_seed(int(seed))
    logits = 6 * (2 * s[:, 0] - 1) + 0.1 * torch.randn((n, H, W), generator=g, device=DEV)
    h = case["h_um"] * 1e-6
    origin = np.array([-2.0, -2.0, -1.0])
    first = np.floor((ells[0][0] - _half(ells[0]) - 0.06 - origin) / h).astype(int)
    dims = np.ceil((ells[0][0] + _half(ells[0]) + 0.06 - origin) / h).astype(int) - first + 1
    grid = fvv.Grid(tuple(origin.astype(np.float32)), np.float32(h),
                    tuple(int(v) for v in first), tuple(int(v) for v in dims))
    ax = [origin[a] + (first[a] + np.arange(dims[a])) * h - ells[0][0][a] for a in range(3)]
    X = np.stack(np.meshgrid(ax[2], ax[1], ax[0], indexing="ij")[::-1], -1).reshape(-1, 3)
    inside = (((X @ ells[0][1]) / ells[0][2]) ** 2).sum(1) <= 1
    ctx = fvv.Context(max_cams=n, max_w=W, max_h=H, max_coarse=1, max_fine=1, max_rois=1,
                      max_points=1, max_jobs=1)
    K = np.array([[r[1][0, 0], r[1][1, 1], r[1][0, 2], r[1][1, 2]] for r in rig])
    hull = SoftHull(ctx, grid, K, np.stack([r[2] for r in rig]),
                    np.stack([-r[2] @ r[3] for r in rig]), W, H)
    pose = lambda sigma: torch.from_numpy(rng.normal(0, sigma, (n, 3)).astype(np.float32))
    return dict(hull=hull, logits=logits.contiguous().requires_grad_(True),
                omega=pose(math.radians(0.5)).requires_grad_(True),
                tau=pose(0.01).requires_grad_(True),
                target=torch.from_numpy(inside.astype(np.float32)).to(DEV))


def prepare(case, seed):
    st = {"frame": _prepare_frame, "calls": _prepare_calls, "roi": _prepare_roi,
          "batched": _prepare_batched, "visibility": _prepare_visibility,
          "soft": _prepare_soft}[case["kind"]](case, int(seed))
    st["kind"] = case["kind"]
    return st


# ---------------------------------------------------------------------------- run
def _frame_out(s):
    b = s["bufs"]
    return [t for t in (b.occ_coarse, b.labels, b.rois, b.jobs, b.occ_fine, b.keys, b.xyz,
                        b.point_off, b.counts, s["sils"], b.tris, b.tri_off) if t is not None]


def _run_frame(st):
    slots = st["slots"]
    if len(slots) == 1:
        s = slots[0]
        if "graph" in s:
            s["graph"].launch()
        else:
            s["ctx"].frame(s["params"], s["sils"], s["bufs"], masks=s["masks"])
    else:
        main = torch.cuda.current_stream()
        for s, stream, done in zip(slots, st["streams"], st["done"]):
            stream.wait_stream(main)
            s["graph"].launch(stream)
            done.record(stream)
        for done in st["done"]:
            main.wait_event(done)
    return [_frame_out(s) for s in slots]


def _run_calls(st):
    c = st["ctx"]
    c.pack_silhouettes(st["masks"], out=st["sils"])
    c.carve(st["P"], st["W"], st["H"], st["sils"], st["coarse"], fvv.tile(64, 1), out=st["occ"])
    c.label(st["coarse"], st["occ"], max_rois=256, labels=st["labels"], rois=st["rois"],
            n_rois=st["n_rois"])
    return [st[k] for k in ("sils", "occ", "labels", "rois", "n_rois")]


def _run_roi(st):
    c, a = st["ctx"], (st["P"], st["W"], st["H"], st["sils"])
    c.carve(*a, st["grid"], out=st["occ"])
    c.surface(st["grid"], st["occ"], *a, n_steps=st["steps"], max_points=st["keys"].numel(),
              keys=st["keys"], xyz=st["xyz"], n_points=st["n_points"])
    c.mesh(st["grid"], st["occ"], st["keys"], st["n_points"], tris=st["tris"],
           n_tris=st["n_tris"])
    return {k: st[k] for k in ("buf", "keys", "xyz", "n_points", "tris", "n_tris")}


def _run_batched(st):
    st["graph"].launch()
    return st["out"]


def _run_visibility(st):
    st["ctx"].visibility(st["P"], st["W"], st["H"], st["xyz"], st["n_p"], st["tris"], st["n_t"],
                         st["t_v"], depth=st["depth"], vis=st["vis"])
    return {"depth": st["depth"], "vis": st["vis"]}


def _run_soft(st):
    loss = st["hull"].l2_loss(st["logits"], st["omega"], st["tau"], st["target"])
    g = torch.autograd.grad(loss, (st["logits"], st["omega"], st["tau"]))
    return {"loss": loss.detach(), "logits": g[0], "omega": g[1], "tau": g[2]}


def run(state):
    return {"frame": _run_frame, "calls": _run_calls, "roi": _run_roi, "batched": _run_batched,
            "visibility": _run_visibility, "soft": _run_soft}[state["kind"]](state)


# ---------------------------------------------------------------------------- work
def work(case):
    """Masks or logits in, everything the calls return out; the arithmetic is the projections
    (21 operations each) that decide a sample or an exit point."""
    kind, n = case["kind"], case["cams"]
    px = n * case["width"] * case["height"]
    if kind in ("frame", "calls", "visibility"):
        coarse = math.prod(case["vol_" + a] for a in "xyz") / (case["hc_um"] * 1e-6) ** 3
    if kind in ("frame", "visibility"):
        # touching people share ROIs, which hold more air
        fine = _fine_samples(case) * (1.7 if case.get("pairs") else 1.0)
        edges = max(case["people"], 2) * PERSON_M2 / (case["hf_um"] * 1e-6) ** 2
    if kind == "frame":
        k = case["in_flight"]
        sil = px * 9 / 8 if case["masks"] else px / 8
        steps = 1 if case["bresenham"] else 8
        return {"bytes": k * (sil + 5 * coarse + fine + (40 if case["mesh"] else 16) * edges),
                "flops": k * 21 * (2 * coarse + TESTS * fine + steps * 2 * edges)}
    if kind == "calls":
        return {"bytes": px * 9 / 8 + 5 * coarse, "flops": 21 * 2 * coarse}
    if kind == "roi":
        fine = PERSON_M3 / (case["h_um"] * 1e-6) ** 3
        edges = PERSON_M2 / (case["h_um"] * 1e-6) ** 2
        return {"bytes": px / 8 + fine + 40 * edges,
                "flops": 21 * (TESTS * fine + 2 * case["steps"] * edges)}
    if kind == "batched":
        a, b = case["edge_lo"], case["edge_hi"]
        total = case["frames"] * case["rois"] * ((a + b) / 2 / (case["h_um"] * 1e-6)) ** 3
        return {"bytes": total + case["frames"] * px / 8, "flops": 21 * 2 * total}
    if kind == "visibility":
        tris = 2 * edges
        return {"bytes": 4 * px + tris * (12 + 4) + 12 * edges + 4 * n * tris,
                "flops": 21 * n * 4 * tris}
    v = 0.6 / (case["h_um"] * 1e-6) ** 3
    return {"bytes": 2 * 4 * px + 8 * v, "flops": 2 * n * v * 60}


# ---------------------------------------------------------------------------- exact
def _f32(x):
    return x.float().double()


def _rows(P, X):
    """The three projected rows of X [..., 3] (values of float32) as fused float32 chains."""
    p = [float(v) for v in np.asarray(P, np.float32).reshape(-1)]
    return [_f32(p[4 * r + 2] * X[..., 2] + _f32(p[4 * r + 1] * X[..., 1] + _f32(
        p[4 * r] * X[..., 0] + p[4 * r + 3]))) for r in range(3)]


def _inside(st, masks, X):
    ok = torch.ones(X.shape[:-1], dtype=torch.bool, device=DEV)
    for c in range(masks.shape[0]):
        a, b, w = _rows(st["P"][c], X)
        u, v = torch.floor(a / w), torch.floor(b / w)
        seen = (w > 0) & (u >= 0) & (u < st["W"]) & (v >= 0) & (v < st["H"])
        u, v = torch.where(seen, u, 0).long(), torch.where(seen, v, 0).long()
        ok &= seen & (masks[c][v, u] != 0)
    return ok


def _exact_roi(case, seed):
    """The exit points by bisection against the hull, at positions in 64 bits."""
    st = _prepare_roi(case, seed)
    _, masks, grid = _roi_scene(case, seed)
    nx, ny, nz = grid.dims
    h, org = float(grid.h), [float(v) for v in grid.origin]
    at = [(grid.lo[a] + torch.arange(grid.dims[a], device=DEV)).double() for a in range(3)]
    pos = [_f32(at[a] * h + org[a]) for a in range(3)]
    occ = torch.stack([_inside(st, masks, torch.stack([
        pos[0].expand(ny, nx), pos[1][:, None].expand(ny, nx), z.expand(ny, nx)], -1))
        for z in pos[2]])
    keys = []
    for a, d in enumerate((2, 1, 0)):
        n = occ.shape[d]
        k = (occ.narrow(d, 0, n - 1) != occ.narrow(d, 1, n - 1)).nonzero()
        keys.append(3 * (k[:, 2] + nx * (k[:, 1] + ny * k[:, 0])) + a)
    keys = torch.cat(keys).sort()[0]
    lin, axis = keys // 3, keys % 3
    i = torch.stack([lin % nx, lin // nx % ny, lin // (nx * ny)], 1)
    on_first = occ[i[:, 2], i[:, 1], i[:, 0]]
    e = torch.nn.functional.one_hot(axis, 3)
    on = (i + torch.tensor(grid.lo, device=DEV) + e * (~on_first)[:, None]).double()
    way = torch.where(on_first, 1.0, -1.0).double()
    o = torch.tensor(org, device=DEV, dtype=torch.float64)

    def point(t):
        return (on + e * (way * t)[:, None]) * h + o

    lo, hi = torch.zeros_like(way), torch.ones_like(way)
    for _ in range(case["steps"]):
        mid = (lo + hi) / 2
        ok = _inside(st, masks, _f32(point(mid)))
        lo, hi = torch.where(ok, mid, lo), torch.where(ok, hi, mid)
    xyz = torch.zeros(st["xyz"].shape, dtype=torch.float64, device=DEV)
    xyz[:keys.numel()] = point((lo + hi) / 2)
    return dict(buf=None, keys=None, xyz=xyz, n_points=None, tris=None, n_tris=None)


def _exact_visibility(case, seed):
    """Depth images: each covered pixel's smallest distance, the distance in 64 bits."""
    st = _prepare_visibility(case, seed)
    V, T = st["xyz"][:int(st["n_p"])].double(), st["tris"][:int(st["n_t"])].long()
    W, H = st["W"], st["H"]
    depth = torch.full(st["depth"].shape, math.inf, dtype=torch.float64, device=DEV)
    ctr = V[T].sum(1) / 3
    for c in range(case["cams"]):
        a, b, w = _rows(st["P"][c], V)
        x, y = (a / w).float()[T], (b / w).float()[T]
        p = torch.from_numpy(st["P"][c].astype(np.float64)).to(DEV)
        d = ctr @ p[2, :3] + p[2, 3]

        def side(i, j, px, py):
            return (x[:, j] - x[:, i]) * (py - y[:, i]) - (y[:, j] - y[:, i]) * (px - x[:, i])

        ok = (w[T] > 0).all(1) & (d > 0) & (side(0, 1, x[:, 2], y[:, 2]) != 0)
        x0, y0 = x.min(1)[0].floor().clamp(min=0), y.min(1)[0].floor().clamp(min=0)
        x1, y1 = x.max(1)[0].floor().clamp(max=W - 1), y.max(1)[0].floor().clamp(max=H - 1)
        ok &= (x1 >= x0) & (y1 >= y0)
        if not ok.any():
            continue
        img = depth[c].view(-1)
        for dy in range(int((y1 - y0)[ok].max()) + 1):
            for dx in range(int((x1 - x0)[ok].max()) + 1):
                px, py = x0 + dx, y0 + dy
                f = [side(i, j, px + 0.5, py + 0.5) for i, j in ((0, 1), (1, 2), (2, 0))]
                hit = ok & (px <= x1) & (py <= y1) & (
                    ((f[0] >= 0) & (f[1] >= 0) & (f[2] >= 0))
                    | ((f[0] <= 0) & (f[1] <= 0) & (f[2] <= 0)))
                img.scatter_reduce_(0, (py * W + px).long()[hit], d[hit], "amin")
    return {"depth": depth, "vis": None}


def _exact_soft(case, seed):
    """The loss and its gradients in float64, by autograd."""
    st = _prepare_soft(case, seed)
    hull, W, H = st["hull"], case["width"], case["height"]
    L, om, ta = (st[k].detach().double().to(DEV).requires_grad_(True)
                 for k in ("logits", "omega", "tau"))
    g = hull.grid
    ax = [float(np.float32(g.origin[a])) + (g.lo[a] + torch.arange(g.dims[a], device=DEV).double())
          * float(np.float32(g.h)) for a in range(3)]
    Z, Y, X = torch.meshgrid(ax[2], ax[1], ax[0], indexing="ij")
    X = torch.stack([X, Y, Z], -1).reshape(-1, 3)
    occ = torch.ones(X.shape[0], dtype=torch.float64, device=DEV)
    zero = torch.zeros((), dtype=torch.float64, device=DEV)
    for c in range(case["cams"]):
        o = om[c]
        skew = torch.stack([zero, -o[2], o[1], o[2], zero, -o[0], -o[1], o[0], zero]).view(3, 3)
        R = torch.matrix_exp(skew) @ torch.from_numpy(hull.R0[c].astype(np.float32)).double().to(DEV)
        t = torch.from_numpy(hull.t0[c].astype(np.float32)).double().to(DEV) + ta[c]
        q = X @ R.T + t
        fx, fy, cx, cy = (float(np.float32(v)) for v in hull.K[c])
        z = q[:, 2]
        u, v = fx * q[:, 0] / z + cx - 0.5, fy * q[:, 1] / z + cy - 0.5
        iu, iv = u.detach().floor(), v.detach().floor()
        s = torch.sigmoid(L[c])
        p = 0
        for dy in (0, 1):
            for dx in (0, 1):
                x, y = iu + dx, iv + dy
                ok = (x >= 0) & (x < W) & (y >= 0) & (y < H) & (z.detach() > 0)
                at = (torch.where(ok, y, 0) * W + torch.where(ok, x, 0)).long()
                wx = u - iu if dx else 1 - (u - iu)
                wy = v - iv if dy else 1 - (v - iv)
                p = p + torch.where(ok, wx * wy * s.reshape(-1)[at], 0.0)
        occ = occ * p
    loss = ((occ - st["target"].double()) ** 2).sum()
    gl, go, gt = torch.autograd.grad(loss, (L, om, ta))
    return {"loss": loss.detach(), "logits": gl, "omega": go.cpu(), "tau": gt.cpu()}


def exact(case, seed):
    """A frame's floats are exit points of edges that integers select, so only a ROI's are
    recomputed; the other calls return whole numbers."""
    return {"roi": _exact_roi, "visibility": _exact_visibility,
            "soft": _exact_soft}.get(case["kind"], lambda *_: None)(case, int(seed))
