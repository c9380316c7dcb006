"""The walks at the edges of their batches: tiles that list exactly n faces, n on both sides of a
64-face batch (odd batches end on the empty record), of the spans that a workgroup stages together
(128 and 256 faces) and of several spans, walked to the end (faint faces) and stopped early (opaque
ones), one view (each wave stages for itself) and two (cooperative staging)."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2605_31419_amd import raster
from paper_2605_31419_amd import scenes as S
from tests import gpu_util as G
from tests import test_gpu_parity as PAR
from tests.helpers import IDENTITY, grad_close

pytestmark = pytest.mark.gpu

INTR = S.Intrinsics(16, 16, 20.0, 20.0, 7.5, 7.5)
NAMES = ["grad_pos", "grad_col", "grad_opa", "grad_pose"]
SHIFTED = S.pose_pack(np.eye(3), [0.05, -0.03, 0.1])


def _tile(n, opaque):
    """n small and large faces in front of one 16x16 image; every one overlaps it."""
    g = S.rng(9000 + 2 * n + opaque)
    z = g.uniform(1.0, 3.0, n)
    c = np.stack([g.uniform(-0.2, 0.2, n) * z, g.uniform(-0.2, 0.2, n) * z, z], 1)
    t1, t2 = S._tangents(S._random_unit(g, n) * 0.3 + np.array([0.0, 0.0, 1.0]))
    verts = S._triangles_around(g, c, np.exp(g.uniform(np.log(0.1), np.log(1.2), n)), t1, t2)
    lo, hi = (0.5, 0.95) if opaque else (0.002, 0.02)
    return S._pack_soup(verts, g.uniform(0, 1, (n, 3, 3)), g.uniform(lo, hi, (n, 3)))


@pytest.mark.parametrize("opaque", [False, True])
@pytest.mark.parametrize("n", [1, 2, 3, 63, 64, 65, 127, 128, 129, 255, 256, 257, 384, 513])
def test_walks_at_batch_edges(n, opaque):
    """Images and the separate backward against the oracle; the fused step, under every kind of
    tile schedule, against the separate backward from the L1 seeds of its own images (the same
    per-pixel arithmetic, so only the order of the sums differs)."""
    sc = _tile(n, opaque)
    for poses in ([IDENTITY], [IDENTITY, SHIFTED]):
        intrs = [INTR] * len(poses)
        rast, p = G.make(sc, intrs, poses)
        c, d, t = G.render(rast, p)
        cs, ds = G.per_view(rast, c, 3), G.per_view(rast, d, 1)
        for v, pose in enumerate(poses):
            oc, od, ot = O.render(sc, pose, INTR)
            err = max(np.abs(cs[v] - oc).max(), np.abs(ds[v] - od).max(),
                      np.abs(G.per_view(rast, t, 1)[v] - ot).max())
            assert err <= PAR.IMG_TOL, err
        P = rast.total_pixels
        g = np.random.default_rng(n)
        gc, gd = g.normal(size=3 * P).astype(np.float32), g.normal(size=P).astype(np.float32)
        masks = PAR._steep_masks(sc, poses, intrs, 1.0)
        for a, ch in ((gc, 3), (gd, 1)):
            PAR._apply_masks(a, masks, ch)
        got = rast.backward(p, G.to_dev(gc), G.to_dev(gd), None)
        ref, conds = PAR._oracle_backward_views(sc, poses, intrs, G.per_view(rast, gc, 3), G.per_view(rast, gd, 1), None,
                                                1.0, with_abs=True)
        for nm, a, b, cond in zip(NAMES, got, ref, conds + [None]):
            ok, msg, _ = grad_close(a.cpu().numpy().astype(np.float64), b, name=nm, cond=cond)
            assert ok, msg
        # the fused step against the separate backward of the same seeds
        tcs, tds, seeds = [], [], []
        for v in range(len(poses)):
            tc, td, _ = PAR._nudged_targets(cs[v], ds[v], 10 * n + v, None)
            tcs.append(tc.reshape(-1))
            tds.append(td.reshape(-1))
            seeds.append(O.l1_seeds(cs[v], ds[v], tc, td, 256)[1:])
        sep = rast.backward(p, G.to_dev(np.concatenate([s[0].reshape(-1) for s in seeds])),
                            G.to_dev(np.concatenate([s[1].reshape(-1) for s in seeds])), None)
        tc, td = G.to_dev(np.concatenate(tcs)), G.to_dev(np.concatenate(tds))
        for sched in ((0, 0, 0), (0, 1, 0), (1, 1, 64)):
            out = rast.train_l1(p, tc, td, schedule=sched)
            torch.cuda.synchronize()
            for nm, a, b in zip(NAMES, out, sep):
                a, b = a.cpu().numpy().astype(np.float64), b.cpu().numpy().astype(np.float64)
                assert np.linalg.norm(a - b) <= 1e-5 * np.linalg.norm(b), (sched, nm)


# 13 x 11 tiles, the faces of _tile around the middle one
WIDE = S.Intrinsics(203, 171, 20.0, 20.0, 103.5, 87.5)
PIX = 203 * 171


def _same(a, b, scale=1.0):
    a, b = a.detach().cpu().numpy().astype(np.float64), b.detach().cpu().numpy().astype(np.float64)
    return np.linalg.norm(scale * a - b) <= 1e-5 * np.linalg.norm(b)


def _longest(rast):
    ranges = G.binning_arrays(rast)[2]
    return int((ranges[:, 1] - ranges[:, 0]).max())


@pytest.mark.parametrize("n", [150, 200, 333])
@pytest.mark.parametrize("mode", [dict(sigma=1.0), dict(sigma=0.5), dict(sigma=2.0), dict(sigma=0.8), dict(face_sigma=True),
                                  dict(sigma=1.0, perspective=True), dict(sigma=0.8, perspective=True)], ids=str)
def test_split_tiles(mode, n):
    """A tile of more than 128 faces is walked in two halves by two workgroups where it is in a single
    view of at least 128 tiles, and whole where there are several views: the same view given once and
    twice.  Images and
    statistics are equal bit for bit, two equal views have twice the gradients, up to the order of
    the FP32 sums."""
    print(f"[split] mode={mode} n={n}", flush=True)
    sc = _tile(n, n == 200)
    mode = dict(mode)
    if mode.pop("face_sigma", False):
        sc = S.Scene(sc.pos, sc.col, sc.opa, None, np.linspace(0.4, 2.2, n).astype(np.float32))
    dev = raster.DeviceScene.from_numpy(sc)
    g = np.random.default_rng(n)
    seeds = [g.normal(size=k * PIX).astype(np.float32) for k in (3, 1, 1)]
    res = []
    for views in (1, 2):
        rast = raster.Rasterizer(dev, [WIDE] * views, raster.Params(**mode))
        p = raster.poses_tensor([SHIFTED] * views)
        rast.fit(p)
        rast.bin_and_sort(p)
        assert _longest(rast) > 128
        img = [x.clone() for x in rast.forward(p)]
        grads = [x.clone() for x in rast.backward(p, *[G.to_dev(np.tile(x, views)) for x in seeds])]
        stats = [x.clone() for x in rast.face_stats(p)]
        loss = torch.zeros(views, device="cuda")
        tc, td = G.to_dev(np.tile(np.abs(seeds[0]) % 1, views)), G.to_dev(np.tile(1 + np.abs(seeds[1]), views))
        fused = [[x.clone() for x in rast.train_l1(p, tc, td, loss=loss, schedule=s)] + [loss.clone()]
                 for s in ((0, 1, 0), (1, 1, 64))]
        res.append((img, grads, stats, fused))
    torch.cuda.synchronize()
    (img1, grads1, stats1, fused1), (img2, grads2, stats2, fused2) = res
    for a, b in zip(img1, img2):
        assert torch.equal(a, b[:a.numel()]) and torch.equal(a, b[a.numel():])
    for a, b in zip(stats1, stats2):
        assert torch.equal(a.reshape(-1), b.reshape(-1)[:a.numel()])
    for one, two in [(grads1, grads2)] + [(x[:4], y[:4]) for x, y in zip(fused1, fused2)]:
        for nm, a, b in zip(NAMES, one, two):
            if nm == "grad_pose":
                a = torch.cat([a.reshape(-1), a.reshape(-1)])
                assert _same(a, b.reshape(-1)), nm
            else:
                assert _same(a, b, 2.0), nm
    for x, y in zip(fused1, fused2):
        assert _same(torch.cat([x[4], x[4]]), y[4])


@pytest.mark.parametrize("n", [200, 333])
def test_split_tiles_with_the_normal_channels(n):
    """As test_split_tiles, the mapping step (colour, depth and normals in one walk)."""
    from paper_2605_31419_amd.window import MappingWindow
    print(f"[split] mapping step, n={n}", flush=True)
    dev = raster.DeviceScene.from_numpy(_tile(n, False))
    g = np.random.default_rng(n)
    tc, td = g.uniform(0, 1, 3 * PIX).astype(np.float32), g.uniform(0.5, 4.0, PIX).astype(np.float32)
    tn = g.normal(size=(3, PIX)).astype(np.float32)
    tn = (tn / np.linalg.norm(tn, axis=0)).reshape(-1)
    res = []
    for views in (1, 2):
        win = MappingWindow(dev, [WIDE] * views, w_ssim=0.2, w_norm=0.05)
        p = raster.poses_tensor([SHIFTED] * views)
        win.prepare(p)
        grads = win.step(p, G.to_dev(np.tile(tc, views)), G.to_dev(np.tile(td, views)),
                         target_normals=G.to_dev(np.tile(tn, views)))
        torch.cuda.synchronize()
        res.append([x.clone() for x in grads] + [win.loss.clone(), win.norm_loss.clone()])
    one, two = res
    for nm, a, b in zip(NAMES, one[:4], two[:4]):
        if nm == "grad_pose":
            a = torch.cat([a.reshape(-1), a.reshape(-1)])
            assert _same(a, b.reshape(-1)), nm
        else:
            assert _same(a, b, 2.0), nm
    for a, b in zip(one[4:], two[4:]):
        assert _same(torch.cat([a.reshape(-1), a.reshape(-1)]), b.reshape(-1))
