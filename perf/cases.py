"""Timed cases of the rasterizer: the work that a SLAM program has it do, each through the
public entry points of ``paper_2605_31419_amd``.

A case is a dict of plain values; ``kind`` picks the entry points:

* ``step``        ``Rasterizer.bin_and_sort`` + ``train_l1`` (one pose or map iteration)
* ``photometric`` ``bin_and_sort`` + ``train_photometric`` (L1, D-SSIM and depth terms)
* ``window``      ``MappingWindow.step`` (keyframe window; optionally the whole mapping energy)
* ``track``       ``Tracker``: load a frame, replay its captured pose iterations
* ``serve``       ``serve.GpuExecutor.run`` on one batch of render queries of mixed sizes
* ``autograd``    ``raster.rasterize`` and its backward on an indexed mesh
* ``stats``       ``bin_and_sort`` + ``Rasterizer.face_stats`` (map management)
* ``equi``        ``raster.equilateral`` over the map
* ``normals``     ``raster.sensor_normals`` of depth maps

Maps are seeded room soups (faces on the surfaces of a box room with rectangles in it) made on
the GPU; observed frames are ray-cast from the same room with 8-bit colours and millimetre
depths, as an RGB-D camera delivers them, from a pose 1 cm and 0.5 degrees off.
"""
import math

import numpy as np
import torch

from paper_2605_31419_amd import autotune, raster, scenes, serve, track, window

DEV = "cuda"


# ----------------------------------------------------------------------------- the cases

def listed():
    return [
        # the smallest frame a user renders (quick tests, thumbnails): launches and latency
        dict(name="step_64x48_2k", kind="step", width=64, height=48, views=1, faces=2000, soup="frustum", sigma=1.0),
        # tracking one VGA frame: pose iterations in a captured graph (a refinement: eight steps at a
        # tenth of the paper's rates, since a long L1 descent magnifies the rounding of atomics)
        dict(name="track_640x480_200k", kind="track", width=640, height=480, views=1, faces=200_000, soup="fine",
             sigma=1.0, iters=8),
        # the benchmark's step: one 1200x680 view of a 1M-face map
        dict(name="step_1200x680_1M", kind="step", width=1200, height=680, views=1, faces=1_000_000, soup="mixed",
             sigma=1.0),
        # the full photometric energy at the paper's window exponent
        dict(name="photometric_1200x680_1M", kind="photometric", width=1200, height=680, views=1, faces=1_000_000,
             soup="mixed", sigma=0.5),
        # a keyframe window over a map of small faces, L1 terms
        dict(name="window_8x1200x680_500k", kind="window", width=1200, height=680, views=8, faces=500_000,
             soup="fine", sigma=1.0, energy=False),
        # a keyframe window with the whole mapping energy: the largest call
        dict(name="mapping_8x1200x680_1M", kind="window", width=1200, height=680, views=8, faces=1_000_000,
             soup="mixed", sigma=1.0, energy=True),
        # one batch of the render server
        dict(name="serve_8_mixed_1M", kind="serve", width=1200, height=680, views=8, faces=1_000_000, soup="mixed",
             sigma=1.0),
        # differentiable render of an indexed mesh at an odd size, perspective-correct
        dict(name="autograd_mesh_333x251", kind="autograd", width=333, height=251, views=1, faces=60_000, soup="mesh",
             sigma=1.0, perspective=True),
        # the learnable-exponent variant with tight binning on a few odd-sized views
        dict(name="step_3x481x269_face_sigma", kind="step", width=481, height=269, views=3, faces=120_001,
             soup="fine", sigma=1.0, face_sigma=True, tight=True),
        # pruning and densification statistics of a view
        dict(name="stats_1200x680_1M", kind="stats", width=1200, height=680, views=1, faces=1_000_000, soup="mixed",
             sigma=1.0),
        # the equilateral regulariser over the map
        dict(name="equi_1M", kind="equi", width=1, height=1, views=1, faces=1_000_000, soup="mixed", sigma=1.0),
        # normal targets of incoming depth frames
        dict(name="normals_2x640x480", kind="normals", width=640, height=480, views=2, faces=0, soup="none",
             sigma=1.0),
    ]


def draw(rng):
    """One more case: the listed kinds over their ranges, odd sizes included, never more work
    than the 8-view mapping window of the 1M-face map."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["step", "step", "photometric", "window", "mapping", "track", "serve", "autograd", "stats",
                       "equi", "normals"])
    width = log_int(48, 1200)
    height = min(680, max(36, int(width * rng.uniform(0.5, 0.8)) | rng.randint(0, 1)))
    faces = log_int(2000, 1_000_000)
    sigma = rng.choice([1.0, 1.0, 0.5, 2.0, 0.8])
    views = 1
    if kind in ("window", "mapping"):
        views = rng.randint(2, 8)
    elif kind in ("step", "normals", "serve"):
        views = rng.choice([1, 1, 2, 3, 5, 8])
    soup = "mixed" if faces > 300_000 and rng.random() < 0.7 else "fine"
    if width * height < 20_000 and views == 1 and kind == "step":
        soup, faces = "frustum", min(faces, 20_000)
    c = dict(kind=kind, width=width, height=height, views=views, faces=faces, soup=soup, sigma=sigma)
    if kind == "step":
        variant = rng.choice(["", "", "face_sigma", "perspective", "tight", "opacity_min"])
        if variant:
            c[variant] = True
    elif kind in ("window", "mapping"):
        c.update(kind="window", energy=kind == "mapping")
    elif kind == "track":
        c.update(iters=rng.choice([4, 6, 8]))
    elif kind == "autograd":
        c.update(soup="mesh", faces=min(faces, 200_000), perspective=rng.random() < 0.5)
    elif kind == "equi":
        c.update(width=1, height=1, sigma=1.0)
    elif kind == "normals":
        c.update(faces=0, soup="none", sigma=1.0)
    return c


# ----------------------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) & 0x7FFFFFFF)
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV)


class _Room:
    """Six walls of a 4.0 x 3.0 x 2.6 m room and six rectangles in it, each with a smooth texture."""

    def __init__(self, seed):
        r = np.random.default_rng(seed)
        lx, ly, lz = scenes.ROOM_SIZE
        ex, ey, ez = np.eye(3)
        o = np.zeros(3)
        quads = [(o, lx * ex, ly * ey), (lz * ez, lx * ex, ly * ey), (o, lx * ex, lz * ez),
                 (ly * ey, lx * ex, lz * ez), (o, ly * ey, lz * ez), (lx * ex, ly * ey, lz * ez)]
        for _ in range(6):
            q, _ = np.linalg.qr(r.normal(size=(3, 3)))
            sa, sb = r.uniform(0.4, 1.5, size=2)
            c = np.array([r.uniform(0.8, lx - 0.8), r.uniform(0.8, ly - 0.8), r.uniform(0.5, lz - 0.5)])
            quads.append((c - 0.5 * sa * q[0] - 0.5 * sb * q[1], sa * q[0], sb * q[1]))

        def t(x):
            return torch.as_tensor(np.asarray(x, np.float32), device=DEV)
        self.o, self.a, self.b = (t([q[k] for q in quads]) for k in range(3))
        n = len(quads)
        self.k, self.ph = t(r.normal(scale=6.0, size=(n, 3, 3, 3))), t(r.uniform(0, 2 * np.pi, size=(n, 3, 3)))
        self.amp, self.base = t(r.uniform(0.05, 0.2, size=(n, 3, 3))), t(r.uniform(0.2, 0.8, size=(n, 3)))
        self.area = torch.linalg.norm(torch.linalg.cross(self.a, self.b), dim=1)

    def texture(self, s, p):
        """Colours [n, 3] of points p [n, 3] on surfaces s [n]."""
        out = self.base[s]
        for w in range(3):
            out = out + self.amp[s, :, w] * torch.sin((self.k[s, :, w] * p[:, None, :]).sum(2) + self.ph[s, :, w])
        return out

    def frame(self, pose, it, g):
        """Colour [3, P] (8 bit) and depth [P] (millimetres, some missing) seen from a pose."""
        R = torch.as_tensor(pose[:9].reshape(3, 3).copy(), device=DEV)
        t = torch.as_tensor(pose[9:].copy(), device=DEV)
        org = -(R.T @ t)
        v, u = torch.meshgrid(torch.arange(it.height, device=DEV, dtype=torch.float32),
                              torch.arange(it.width, device=DEV, dtype=torch.float32), indexing="ij")
        d = torch.stack([(u - it.cx) / it.fx, (v - it.cy) / it.fy, torch.ones_like(u)], -1).reshape(-1, 3) @ R
        best = torch.full((d.shape[0],), 1e9, device=DEV)
        who = torch.zeros(d.shape[0], dtype=torch.long, device=DEV)
        for s in range(self.o.shape[0]):
            n = torch.linalg.cross(self.a[s], self.b[s])
            z = ((self.o[s] - org) @ n) / (d @ n)
            h = org + z[:, None] * d - self.o[s]
            x, y = h @ self.a[s] / (self.a[s] @ self.a[s]), h @ self.b[s] / (self.b[s] @ self.b[s])
            hit = (z > 0.1) & (z < best) & (x > -1e-3) & (x < 1.001) & (y > -1e-3) & (y < 1.001)
            best, who = torch.where(hit, z, best), torch.where(hit, torch.full_like(who, s), who)
        best = torch.where(best < 1e8, best, torch.zeros_like(best))
        col = self.texture(who, org + best[:, None] * d).T
        col = col + 0.02 * torch.randn(col.shape, generator=g, device=DEV)
        dep = best * (1 + 0.002 * torch.randn(best.shape, generator=g, device=DEV))
        dep = torch.where(_rand(g, dep.numel()) < 0.03, torch.zeros_like(dep), dep)
        return (torch.round(col.clamp(0, 1) * 255) / 255).contiguous(), torch.round(dep * 1000) / 1000


def _triangles(g, centres, sizes, t1, t2):
    """Vertices [m, 3, 3]: near-equilateral triangles of edge `sizes` in the planes (t1, t2)."""
    m = centres.shape[0]
    ang = (2 * math.pi / 3) * torch.arange(3, device=DEV) + (0.6 * _rand(g, m, 3) - 0.3) + 2 * math.pi * _rand(g, m, 1)
    rad = (sizes / math.sqrt(3.0))[:, None, None]
    return centres[:, None] + rad * (torch.cos(ang)[..., None] * t1[:, None] + torch.sin(ang)[..., None] * t2[:, None])


def _unit(x):
    return x / torch.linalg.norm(x, dim=-1, keepdim=True)


def _map(case, seed, room, it):
    """(pos [3, N], col [3, N], opa [N], faces or None, face_sigma or None) of the case's map."""
    g, m = _gen(seed), case["faces"]
    faces = None
    if case["soup"] == "frustum":          # faces scattered through the view of an identity pose
        z = torch.pow(0.5 ** 3 + _rand(g, m) * (4.0 ** 3 - 0.5 ** 3), 1 / 3)
        c = torch.stack([(_rand(g, m) * it.width - 0.5 - it.cx) * z / it.fx,
                         (_rand(g, m) * it.height - 0.5 - it.cy) * z / it.fy, z], 1)
        nrm = _unit(torch.randn(m, 3, generator=g, device=DEV))
        t1 = _unit(torch.linalg.cross(nrm, _unit(torch.randn(m, 3, generator=g, device=DEV))))
        verts = _triangles(g, c, torch.exp(math.log(0.01) + _rand(g, m) * math.log(10.0)), t1,
                           torch.linalg.cross(nrm, t1))
        col = _rand(g, m * 3, 3)
    elif case["soup"] == "mesh":           # a wavy indexed sheet in front of the camera, two layers deep
        n = max(2, int(math.sqrt(m / 4)))
        layers, idx, pts = 2, [], []
        for k in range(layers):
            y, x = torch.meshgrid(torch.linspace(-1, 1, n + 1, device=DEV), torch.linspace(-1, 1, n + 1, device=DEV),
                                  indexing="ij")
            jit = 0.2 / n * torch.randn(2, n + 1, n + 1, generator=g, device=DEV)
            z = 1.6 + 0.5 * k + 0.2 * torch.sin(3 * x + k) * torch.cos(4 * y) + 0.3 * x
            pts.append(torch.stack([(x + jit[0]) * z * it.width / (1.9 * it.fx),
                                    (y + jit[1]) * z * it.height / (1.9 * it.fy), z], -1).reshape(-1, 3))
            i, j = torch.meshgrid(torch.arange(n, device=DEV), torch.arange(n, device=DEV), indexing="ij")
            a = (i * (n + 1) + j + k * (n + 1) ** 2).reshape(-1)
            idx += [torch.stack([a, a + 1, a + n + 1], 1), torch.stack([a + 1, a + n + 2, a + n + 1], 1)]
        verts, faces = torch.cat(pts), torch.cat(idx).to(torch.int32).contiguous()
        col = _rand(g, verts.shape[0], 3)
    else:                                  # faces on the room's surfaces: 0.5-3 cm, or 90 % 0.5-2 cm and 10 % 5-20 cm
        s = torch.multinomial(room.area, m, replacement=True, generator=g)
        c = room.o[s] + _rand(g, m, 1) * room.a[s] + _rand(g, m, 1) * room.b[s]
        big = _rand(g, m) < (0.1 if case["soup"] == "mixed" else 0.0)
        lo, hi = (0.005, 0.02) if case["soup"] == "mixed" else (0.005, 0.03)
        r = _rand(g, m)
        sizes = torch.where(big, 0.05 * torch.pow(torch.full_like(r, 4.0), r),
                            lo * torch.pow(torch.full_like(r, hi / lo), r))
        t1, nrm = _unit(room.a[s]), _unit(torch.linalg.cross(room.a[s], room.b[s]))
        verts = _triangles(g, c, sizes, t1, torch.linalg.cross(nrm, t1))
        col = torch.cat([room.texture(s, verts[:, k]) for k in range(3)], 1).reshape(-1, 3)
        col = (col + 0.03 * torch.randn(col.shape, generator=g, device=DEV)).clamp(0, 1)
    pos = verts.reshape(-1, 3).T.contiguous()
    opa = 0.3 + 0.7 * _rand(g, pos.shape[1])
    sig = None
    if case.get("face_sigma"):
        sig = 0.4 + 1.2 * _rand(g, m)
    return pos, col.T.contiguous(), opa, faces, sig


def _intrinsics(case):
    if case["kind"] == "serve":            # the server's three resolutions, up to the case's own size
        res = [r for r in scenes.SERVE_RESOLUTIONS if r[0] < case["width"]] + [(case["width"], case["height"])]
        return [scenes.intrinsics_for(*res[v % len(res)]) for v in range(case["views"])]
    return [scenes.intrinsics_for(case["width"], case["height"])] * case["views"]


def _inputs(case, seed):
    """The map, poses [V, 12], intrinsics and observed frames of a case, made from the seed alone."""
    intrs = _intrinsics(case)
    g = np.random.default_rng(seed + 17)
    ident = np.concatenate([np.eye(3).reshape(9), np.zeros(3)]).astype(np.float32)
    room = None
    if case["soup"] in ("frustum", "mesh"):
        poses = [ident] * len(intrs)
    else:
        room = _Room(seed)
        if case["kind"] == "serve":
            poses = [scenes.random_room_pose(g) for _ in intrs]
        else:
            poses = scenes.room_trajectory(g, len(intrs))
    x = dict(intrs=intrs, poses=torch.as_tensor(np.stack(poses), device=DEV),
             map=_map(case, seed + 1, room, intrs[0]) if case["soup"] != "none" else None)
    if case["kind"] in ("step", "photometric", "window", "track", "normals"):
        tg, cs, ds = _gen(seed + 2), [], []
        for it, p in zip(intrs, poses):
            if room is None:
                n = it.width * it.height
                c, d = _rand(tg, 3, n), 0.5 + 3.5 * _rand(tg, n)
            else:
                c, d = room.frame(scenes.perturb_pose(p, g), it, tg)
            cs.append(c.reshape(-1))
            ds.append(d.reshape(-1))
        x.update(tc=torch.cat(cs), td=torch.cat(ds))
    elif case["kind"] == "autograd":
        n = sum(it.width * it.height for it in intrs)
        tg = _gen(seed + 2)
        x.update(gc=torch.randn(3 * n, generator=tg, device=DEV), gd=torch.randn(n, generator=tg, device=DEV),
                 gt=torch.randn(n, generator=tg, device=DEV),
                 tau=(0.02 * torch.randn(len(intrs), 6, generator=tg, device=DEV)))
    return x


def _params(case):
    return raster.Params(sigma=case["sigma"], opacity_min=bool(case.get("opacity_min")),
                         tight_tiles=bool(case.get("tight")), perspective=bool(case.get("perspective")))


def prepare(case, seed):
    kind, x = case["kind"], _inputs(case, seed)
    s = dict(kind=kind, case=case, **x)
    if kind == "normals":
        s["normals"] = torch.empty(3 * x["td"].numel(), device=DEV)
        return s
    scene = s["scene"] = raster.DeviceScene(*x["map"])
    if kind == "equi":
        s.update(grad=torch.empty(3, scene.n_vertices, device=DEV), loss=torch.empty(1, device=DEV))
    elif kind == "window":
        w = dict(w_ssim=0.2, w_equi=1.2, w_norm=0.05) if case["energy"] else {}
        win = s["win"] = window.MappingWindow(scene, x["intrs"], _params(case), **w)
        win.prepare(x["poses"])
        s["tn"] = raster.sensor_normals(x["td"], x["intrs"]) if case["energy"] else None
    elif kind == "track":
        trk = s["trk"] = track.Tracker(scene, x["intrs"][0], _params(case), lr_trans=1e-4,
                                       lr_rot=3e-4, iters=case["iters"])
        trk.set_frame(x["poses"][0], x["tc"], x["td"])
        trk.rast.schedule = autotune.lookup(x["intrs"], trk.rast.count(trk.pose.view(1, 12)))
        trk.capture()
    elif kind == "serve":
        ex = s["ex"] = serve.GpuExecutor(scene, _params(case), pairs_per_tile=160.0,
                                         max_resolution=(case["width"], case["height"]))
        ex.setup(1, 8 << 30, case["views"], case["views"] * case["width"] * case["height"])
        s["slot"] = ex.make_slot(0)
        s["host_poses"] = list(x["poses"].cpu().numpy())
    else:
        rast = s["rast"] = raster.Rasterizer(scene, x["intrs"], _params(case))
        k = rast.fit(x["poses"], slack=1.5)
        if kind in ("step", "photometric"):
            rast.schedule = autotune.lookup(x["intrs"], k)
            n = rast.total_pixels
            s.update(color=torch.empty(3 * n, device=DEV), depth=torch.empty(n, device=DEV),
                     trans=torch.empty(n, device=DEV), loss=torch.empty(case["views"], device=DEV),
                     grads=rast.grad_buffers())
        elif kind == "autograd":
            rast.fit(raster.compose_poses(x["tau"], x["poses"]), slack=1.5)
            for t in (scene.pos, scene.col, scene.opa, s["tau"]):
                t.requires_grad_(True)
    return s


def run(s):
    kind = s["kind"]
    if kind in ("step", "photometric"):
        rast = s["rast"]
        rast.bin_and_sort(s["poses"], check_capacity=False)
        out = dict(color=s["color"], depth=s["depth"], trans=s["trans"], loss=s["loss"])
        train = rast.train_l1 if kind == "step" else rast.train_photometric
        g = train(s["poses"], s["tc"], s["td"], out=s["grads"], **out)
        out.update(grad_pos=g[0], grad_col=g[1], grad_opa=g[2], grad_pose=g[3])
        if rast.grad_face_sigma is not None:
            out["grad_sigma"] = rast.grad_face_sigma
        return out
    if kind == "window":
        win = s["win"]
        g = win.step(s["poses"], s["tc"], s["td"], target_normals=s["tn"])
        out = dict(color=win.color, depth=win.depth, loss=win.loss, grad_pos=g[0], grad_col=g[1], grad_opa=g[2],
                   grad_pose=g[3])
        if s["tn"] is not None:
            out.update(equi_loss=win.equi_loss, norm_loss=win.norm_loss)
        return out
    if kind == "track":
        trk = s["trk"]
        trk.set_frame(s["poses"][0], s["tc"], s["td"])
        return dict(pose=trk.replay(), loss=trk.loss_hist)
    if kind == "serve":
        batch = [serve.Request(i, it, p) for i, (it, p) in enumerate(zip(s["intrs"], s["host_poses"]))]
        s["ex"].run(s["slot"], batch)
        return dict(color=[r.color for r in batch], depth=[r.depth for r in batch])
    if kind == "autograd":
        sc = s["scene"]
        out = raster.rasterize(s["rast"], s["poses"], s["tau"])
        g = torch.autograd.grad(out, (sc.pos, sc.col, sc.opa, s["tau"]), (s["gc"], s["gd"], s["gt"]))
        color, depth, trans = (t.detach() for t in out)
        return dict(color=color, depth=depth, trans=trans, grad_pos=g[0], grad_col=g[1], grad_opa=g[2], grad_tau=g[3])
    if kind == "stats":
        s["rast"].bin_and_sort(s["poses"], check_capacity=False)
        area, cov, vis = s["rast"].face_stats(s["poses"])
        return dict(area=area, coverage=cov, visible=vis)
    if kind == "equi":
        loss, grad = raster.equilateral(s["scene"], weight=1.2, grad=s["grad"], loss=s["loss"])
        return dict(loss=loss, grad=grad)
    return dict(normals=raster.sensor_normals(s["td"], s["intrs"], normals=s["normals"]))


# ----------------------------------------------------------------------------- least work

def _layers(case):
    """Mean number of faces that cover a pixel: their area over that of the room's surfaces."""
    def sq(lo, hi):                                  # mean area of faces of log-uniform edge length
        return math.sqrt(3) / 4 * (hi * hi - lo * lo) / (2 * math.log(hi / lo))
    if case["soup"] == "mixed":
        return case["faces"] * (0.9 * sq(0.005, 0.02) + 0.1 * sq(0.05, 0.2)) / 68.0
    if case["soup"] == "fine":
        return case["faces"] * sq(0.005, 0.03) / 68.0
    if case["soup"] == "frustum":                    # at the frustum's mean squared inverse depth
        return case["faces"] * sq(0.01, 0.1) * 0.5 * (52.5 * case["width"] / 64.0) ** 2 * 0.165 / (
            case["width"] * case["height"])
    return 2.0


def work(case):
    kind, m = case["kind"], case["faces"]
    px = sum(it.width * it.height for it in _intrinsics(case))
    n = 3 * m if case["soup"] != "mesh" else m // 2
    cov = px * _layers(case)                         # covered (pixel, face) pairs
    scene, grads = 28 * n, 28 * n                    # positions, colours, opacities; their gradients
    fwd, bwd = 40, 81                                # operations of one pair
    if kind == "step":
        return dict(bytes=scene + grads + 36 * px, flops=cov * (fwd + bwd))
    if kind == "photometric":
        return dict(bytes=scene + grads + 36 * px, flops=cov * (fwd + bwd) + 3 * px * 250)
    if kind == "window":
        e = case["energy"]
        return dict(bytes=scene + grads + (44 if e else 32) * px, flops=cov * (fwd + bwd + (20 if e else 0))
                    + (3 * px * 250 + 150 * m if e else 0))
    if kind == "track":
        return dict(bytes=32 * px + case["iters"] * (12 * n + 16 * px), flops=case["iters"] * cov * (fwd + bwd))
    if kind == "serve":
        return dict(bytes=scene + 16 * px, flops=cov * fwd)
    if kind == "autograd":
        return dict(bytes=scene + grads + 12 * m + 40 * px, flops=cov * (fwd + bwd))
    if kind == "stats":
        return dict(bytes=16 * n + 12 * m, flops=cov * fwd + 100 * m)
    if kind == "equi":
        return dict(bytes=24 * n, flops=150 * m)
    return dict(bytes=16 * px, flops=60 * px)


# ----------------------------------------------------------------------------- 64-bit reference
# Plain torch in 64 bits, block by block: every face whose box meets a 64 x 64 pixel block is
# evaluated at each of its pixels, sorted by depth and composited; gradients by autograd.

_BLOCK = 64


def _face_setup(v, R, t, xi, it):
    """Camera-space and projected vertices of faces v [m, 3, 3] at the pose (R, t) perturbed by xi."""
    c = v @ R.T + t
    c = c + xi[:3] + torch.linalg.cross(xi[3:].expand_as(c), c)
    q = torch.stack([it.fx * c[..., 0] / c[..., 2] + it.cx, it.fy * c[..., 1] / c[..., 2] + it.cy], -1)
    return c, q


def _geometry(q):
    e = torch.roll(q, -1, 1) - q                                  # edge k: q_k -> q_k+1
    a2 = (q[:, 1, 0] - q[:, 0, 0]) * (q[:, 2, 1] - q[:, 0, 1]) - (q[:, 1, 1] - q[:, 0, 1]) * (q[:, 2, 0] - q[:, 0, 0])
    ln = torch.linalg.norm(e, dim=2)
    sgn = torch.where(a2 >= 0, 1.0, -1.0).to(q)[:, None]
    n = torch.stack([sgn * e[..., 1] / ln, -sgn * e[..., 0] / ln], -1)
    return a2.abs(), ln, n, a2.abs() / ln.sum(1)


def _visible(v, R, t, it, z_near=0.1, r_min=1e-3):
    c, q = _face_setup(v, R, t, torch.zeros(6, dtype=v.dtype, device=v.device), it)
    a2, _, _, r = _geometry(q)
    lo, hi = q.amin(1), q.amax(1)
    size = torch.tensor([it.width, it.height], dtype=v.dtype, device=v.device)
    lo, hi = torch.ceil(lo.clamp(min=-1.0)).clamp(min=0.0), torch.minimum(torch.floor(torch.minimum(hi, size)), size - 1)
    ok = (c[..., 2] >= np.float32(z_near)).all(1) & (r >= np.float32(r_min)) & (lo <= hi).all(1)
    return ok, lo, hi, c[..., 2].mean(1).float(), a2


def _blend(v, col, opa, sig, R, t, xi, it, u, w, case, t_min=1e-6):
    """Colour [3, p], depth [p], transmittance [p] of depth-sorted faces at pixels (u, w)."""
    c, q = _face_setup(v, R, t, xi, it)
    _, ln, n, r = _geometry(q)
    p = torch.stack([u, w], -1)
    dist = (n[:, :, None] * (p[None, None] - q[:, :, None])).sum(3)            # [m, 3, p]
    E = -dist / r[:, None, None]
    rho = E.amin(1)
    inside = rho > 0
    I = torch.where(inside, torch.where(inside, rho, torch.ones_like(rho)).clamp(max=1.0) ** sig[:, None],
                    torch.zeros_like(rho))
    o = opa.amin(1) if case.get("opacity_min") else opa.mean(1)
    alpha = (o[:, None] * I).clamp(max=1 - 1e-12)
    logt = torch.log1p(-alpha)
    Tb = torch.exp(torch.cumsum(logt, 0) - logt)
    live = Tb.detach() >= np.float32(t_min)
    wgt = alpha * Tb * live
    lam = E * (ln / ln.sum(1, keepdim=True))[:, :, None]                        # of the vertex facing edge k
    lam = lam[:, [1, 2, 0]]                                                     # of vertex k
    if case.get("perspective"):
        lam = lam / c[..., 2][:, :, None]
        W = lam.sum(1)
        W = torch.where(inside, W, torch.ones_like(W))
        lam, z = lam / W[:, None], 1.0 / W
    else:
        z = c[..., 2].mean(1)[:, None]
    C = torch.stack([(wgt * (lam * col[:, :, k, None]).sum(1)).sum(0) for k in range(3)])
    return C, (wgt * z).sum(0), torch.exp((logt * live).sum(0))


def _blocks(case, x, view):
    """(face ids in depth order, pixel columns, pixel rows, packed pixel index) of a view's blocks."""
    pos, _, _, faces, _ = x["map"]
    it = x["intrs"][view]
    idx = (torch.arange(pos.shape[1] // 3 * 3, device=DEV).reshape(-1, 3) if faces is None else faces.long())
    P = x["eff"][view].double()
    R, t = P[:9].reshape(3, 3), P[9:]
    v = pos.double().T[idx]
    ok, lo, hi, z, _ = _visible(v, R, t, it)
    ids = torch.nonzero(ok).reshape(-1)
    ids = ids[torch.argsort(z[ids], stable=True)]
    lo, hi = lo[ids], hi[ids]
    for y in range(0, it.height, _BLOCK):
        for u in range(0, it.width, _BLOCK):
            x1, y1 = min(u + _BLOCK, it.width), min(y + _BLOCK, it.height)
            hit = (lo[:, 0] < x1) & (hi[:, 0] >= u) & (lo[:, 1] < y1) & (hi[:, 1] >= y)
            w, c = torch.meshgrid(torch.arange(y, y1, device=DEV), torch.arange(u, x1, device=DEV), indexing="ij")
            w, c = w.reshape(-1), c.reshape(-1)
            yield ids[hit], c.double(), w.double(), w * it.width + c, idx, R, t, it


def _face_data(case, x, ids, idx):
    pos, col, opa, _, sig = x["map"]
    vid = idx[ids]
    s = sig[ids].double() if sig is not None else torch.full((ids.numel(),), float(np.float32(case["sigma"])),
                                                             dtype=torch.float64, device=DEV)
    return [pos.double().T[vid] if ids.numel() else torch.zeros(0, 3, 3, dtype=torch.float64, device=DEV),
            col.T[vid].double(), opa[vid].double(), s], vid


def _render64(case, x):
    out = []
    for v, it in enumerate(x["intrs"]):
        n = it.width * it.height
        C, D = torch.zeros(3, n, dtype=torch.float64, device=DEV), torch.zeros(n, dtype=torch.float64, device=DEV)
        T = torch.ones_like(D)
        for ids, u, w, pix, idx, R, t, it in _blocks(case, x, v):
            if ids.numel():
                d, _ = _face_data(case, x, ids, idx)
                C[:, pix], D[pix], T[pix] = _blend(*d, R, t, torch.zeros(6, dtype=torch.float64, device=DEV), it, u, w,
                                                   case)
        out.append((C, D, T))
    return out


def _backward64(case, x, seeds):
    """Gradients of sum(seeds * images): positions, colours, opacities, exponents, pose per view."""
    pos, col, opa, faces, _ = x["map"]
    f64 = dict(dtype=torch.float64, device=DEV)
    gp, gc, go = torch.zeros(pos.shape[1], 3, **f64), torch.zeros(pos.shape[1], 3, **f64), torch.zeros(opa.numel(), **f64)
    gs = torch.zeros(case["faces"], **f64)
    gx = torch.zeros(len(x["intrs"]), 6, **f64)
    for v in range(len(x["intrs"])):
        sC, sD, sT = seeds[v]
        for ids, u, w, pix, idx, R, t, it in _blocks(case, x, v):
            if not ids.numel():
                continue
            d, vid = _face_data(case, x, ids, idx)
            xi = torch.zeros(6, **f64)
            leaves = [y.requires_grad_(True) for y in d + [xi]]
            C, D, T = _blend(*d, R, t, xi, it, u, w, case)
            val = (C * sC[:, pix]).sum() + (D * sD[pix]).sum() + (0 if sT is None else (T * sT[pix]).sum())
            a, b, c, s, k = torch.autograd.grad(val, leaves)
            vid = vid.reshape(-1)
            gp.index_add_(0, vid, a.reshape(-1, 3))
            gc.index_add_(0, vid, b.reshape(-1, 3))
            go.index_add_(0, vid, c.reshape(-1))
            if x["map"][4] is not None:
                gs.index_add_(0, ids, s)
            gx[v] += k
    return gp.T.reshape(-1), gc.T.reshape(-1), go, gs, gx


def _dssim64(a, b, it):
    """1 - mean SSIM of [3, H, W] images, 11 x 11 Gaussian window (deviation 1.5), zero padding."""
    k = torch.exp(-(torch.arange(-5, 6, device=DEV, dtype=torch.float64) ** 2) / 4.5)
    k = k / k.sum()
    a, b = a.reshape(3, it.height, it.width), b.reshape(3, it.height, it.width)

    def blur(i):
        p = torch.nn.functional.pad(i, (5, 5, 5, 5))
        p = sum(k[j] * p[:, :, j:j + it.width] for j in range(11))
        return sum(k[j] * p[:, j:j + it.height] for j in range(11))
    ma, mb = blur(a), blur(b)
    va, vb, vab = blur(a * a) - ma * ma, blur(b * b) - mb * mb, blur(a * b) - ma * mb
    s = (2 * ma * mb + 1e-4) * (2 * vab + 9e-4) / ((ma * ma + mb * mb + 1e-4) * (va + vb + 9e-4))
    return 1 - s.mean()


def exact(case, seed):
    kind = case["kind"]
    px = sum(it.width * it.height for it in _intrinsics(case))
    if kind == "track" or case.get("energy"):
        return None
    if kind in ("step", "window") and px * (2 + _layers(case)) > 4e7:      # over about ten seconds
        return None
    x = _inputs(case, seed)
    if kind == "equi":
        v = x["map"][0].double().requires_grad_(True)
        p = v.reshape(3, -1, 3)
        tot = 0.0
        for k in range(3):
            a, b = p[..., (k + 1) % 3] - p[..., k], p[..., (k + 2) % 3] - p[..., k]
            cos = (a * b).sum(0) / torch.sqrt((a * a).sum(0) * (b * b).sum(0))
            tot = tot + ((cos - 0.5) ** 2).sum()
        loss = tot / (3 * case["faces"])
        return dict(loss=loss.detach().reshape(1), grad=1.2 * torch.autograd.grad(loss, v)[0])
    if kind == "normals":
        out, off = [], 0
        for it in x["intrs"]:
            n = it.width * it.height
            d = x["td"][off:off + n].double().reshape(it.height, it.width)
            off += n
            w, u = torch.meshgrid(torch.arange(it.height, device=DEV).double(),
                                  torch.arange(it.width, device=DEV).double(), indexing="ij")
            p = torch.stack([d * (u - it.cx) / it.fx, d * (w - it.cy) / it.fy, d])
            gx, gy = p[:, 1:-1, 2:] - p[:, 1:-1, :-2], p[:, 2:, 1:-1] - p[:, :-2, 1:-1]
            c = torch.linalg.cross(gx, gy, dim=0)
            ln = torch.linalg.norm(c, dim=0)
            ok = (d[1:-1, 1:-1] > 0) & (d[1:-1, 2:] > 0) & (d[1:-1, :-2] > 0) & (d[2:, 1:-1] > 0) & (d[:-2, 1:-1] > 0)
            ok = ok & (ln > 0)
            full = torch.zeros(3, it.height, it.width, dtype=torch.float64, device=DEV)
            full[:, 1:-1, 1:-1] = torch.where(ok, c / torch.where(ok, ln, torch.ones_like(ln)), torch.zeros_like(c))
            out.append(full.reshape(-1))
        return dict(normals=torch.cat(out))
    x["eff"] = x["poses"]
    if kind == "stats":
        P = x["poses"][0].double()
        v = x["map"][0].double().T.reshape(-1, 3, 3)
        ok, _, _, _, a2 = _visible(v, P[:9].reshape(3, 3), P[9:], x["intrs"][0])
        return dict(area=torch.where(ok, 0.5 * a2, torch.zeros_like(a2)), coverage=None, visible=None)
    if kind == "autograd":
        x["eff"] = _compose64(x["tau"].double(), x["poses"].double())
    img = _render64(case, x)
    if kind == "serve":
        return dict(color=[c.reshape(3, it.height, it.width) for (c, _, _), it in zip(img, x["intrs"])],
                    depth=[d.reshape(it.height, it.width) for (_, d, _), it in zip(img, x["intrs"])])
    out = dict(color=torch.cat([c.reshape(-1) for c, _, _ in img]), depth=torch.cat([d for _, d, _ in img]),
               trans=torch.cat([t for _, _, t in img]))
    if kind == "autograd":
        it = x["intrs"][0]
        n = it.width * it.height
        g = _backward64(case, x, [(x["gc"].double().reshape(3, n), x["gd"].double(), x["gt"].double())])
        out.update(grad_pos=g[0].reshape(3, -1), grad_col=g[1].reshape(3, -1), grad_opa=g[2], grad_tau=None)
        if case["sigma"] < 1:
            out["grad_pos"] = None           # as below
        return out
    seeds, losses, off = [], [], 0
    w_ssim = 0.2 if kind == "photometric" else 0.0
    for (C, D, _), it in zip(img, x["intrs"]):
        n = it.width * it.height
        tc, td = x["tc"][3 * off:3 * (off + n)].double().reshape(3, n), x["td"][off:off + n].double()
        off += n
        C, D = C.clone().requires_grad_(True), D.clone().requires_grad_(True)
        loss = 0.8 * (C - tc).abs().mean() + 0.05 * ((td > 0) * (D - td).abs()).mean()
        if w_ssim:
            loss = loss + w_ssim * _dssim64(C, tc, it)
        seeds.append((*torch.autograd.grad(loss, (C, D)), None))
        losses.append(loss.detach())
    g = _backward64(case, x, seeds)
    out.update(loss=torch.stack(losses), grad_pos=g[0], grad_col=g[1], grad_opa=g[2], grad_pose=g[4].reshape(-1))
    if case.get("face_sigma"):
        out["grad_sigma"] = g[3]
    if case["sigma"] < 1 or case.get("face_sigma"):
        # below an exponent of 1 the window's slope at a face's edge is unbounded: the gradients
        # through the edges of a pixel there have no digits that 32-bit coordinates determine
        out.update(grad_pos=None, grad_pose=None)
    if kind == "window":
        del out["trans"]
    return out


def _compose64(tau, poses):
    """Poses of Exp(tau) T, rounded to 32 bits as the pose a renderer is given."""
    out = []
    for x, p in zip(tau, poses):
        a = torch.zeros(4, 4, dtype=torch.float64, device=DEV)
        r, h = x[:3], x[3:]
        a[0, 1], a[0, 2], a[1, 2] = -h[2], h[1], -h[0]
        a[1, 0], a[2, 0], a[2, 1] = h[2], -h[1], h[0]
        a[:3, 3] = r
        e = torch.linalg.matrix_exp(a)
        m = torch.eye(4, dtype=torch.float64, device=DEV)
        m[:3, :3], m[:3, 3] = p[:9].reshape(3, 3), p[9:]
        m = e @ m
        out.append(torch.cat([m[:3, :3].reshape(9), m[:3, 3]]))
    return torch.stack(out).float()
