"""Binning of more (view, face) pairs than the one-launch scan's round of visible-list segments (10,240 of
256 pairs) over few tiles: eight views of 350,000 faces, most of them culled in long stretches, so that
whole chunks of segments are empty.  And a count between the binning and its use: with the same poses
it leaves the binning as it is."""
import numpy as np
import pytest
import torch

from paper_2605_31419_amd import raster
from paper_2605_31419_amd import scenes as S
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

M, VIEWS = 350_000, 8
INTR = S.Intrinsics(64, 48, 60.0, 60.0, 31.5, 23.5)
NAMES = ["grad_pos", "grad_col", "grad_opa", "grad_pose"]


def _scene():
    g = S.rng(77)
    z = np.full(M, -1.0)                                     # behind the camera
    for a in (0, 200_000, M - 1500):                         # three visible stretches
        z[a:a + 1500] = g.uniform(1.0, 3.0, 1500)
    c = np.stack([g.uniform(-0.5, 0.5, M) * z, g.uniform(-0.4, 0.4, M) * z, z], 1)
    t1, t2 = S._tangents(S._random_unit(g, M) * 0.3 + np.array([0.0, 0.0, 1.0]))
    verts = S._triangles_around(g, c, np.exp(g.uniform(np.log(0.02), np.log(0.3), M)), t1, t2)
    return raster.DeviceScene.from_numpy(S._pack_soup(verts, g.uniform(0, 1, (M, 3, 3)), g.uniform(0.05, 0.5, (M, 3))))


def _poses(n):
    return raster.poses_tensor([S.pose_pack(np.eye(3), [0.01 * v, -0.008 * v, 0.02 * v]) for v in range(n)])


def _targets(n):
    g = np.random.default_rng(5)
    return G.to_dev(g.uniform(0, 1, 3 * n)), G.to_dev(g.uniform(1, 3, n))


def _close(a, b):
    a, b = a.double().reshape(-1), b.double().reshape(-1)
    return float((a - b).norm()) <= 1e-5 * float(b.norm())


def test_segments_of_several_chunks_against_single_views():
    sc, p, P = _scene(), _poses(VIEWS), INTR.width * INTR.height
    tc, td = _targets(VIEWS * P)
    rast = raster.Rasterizer(sc, [INTR] * VIEWS, raster.Params())
    print(f"[segments] {VIEWS} views together", flush=True)
    k = rast.fit(p)
    rast.bin_and_sort(p)
    color = torch.empty(3 * P * VIEWS, device="cuda")
    got = rast.train_l1(p, tc, td, color=color)
    ones, total = [], None
    for v in range(VIEWS):
        print(f"[segments] view {v}", flush=True)
        one = raster.Rasterizer(sc, [INTR], raster.Params())
        q = p.reshape(VIEWS, 12)[v:v + 1].contiguous()
        ones.append(one.fit(q))
        one.bin_and_sort(q)
        c = torch.empty(3 * P, device="cuda")
        out = one.train_l1(q, tc[3 * P * v:3 * P * (v + 1)].contiguous(), td[P * v:P * (v + 1)].contiguous(), color=c)
        assert torch.equal(c, color[3 * P * v:3 * P * (v + 1)])
        assert _close(got[3].reshape(VIEWS, 6)[v], out[3])
        total = [x.double() for x in out[:3]] if total is None else [a + x.double() for a, x in zip(total, out[:3])]
        del one, out
    assert k == sum(ones) and k > 0
    for nm, a, b in zip(NAMES, got, total):
        assert float(b.abs().max()) > 0 and _close(a, b), nm


@pytest.mark.parametrize("views", [1, VIEWS])
def test_a_count_leaves_the_binning(views):
    """One view of 2.8M faces and eight of 350,000 (the order of the 12 tiles and the dense visible list
    are read after the count; an indexed mesh, so that the faces need not be stored eight times)."""
    P = INTR.width * INTR.height
    sc, p = _scene(), _poses(views)
    if views == 1:
        n = sc.n_vertices
        faces = torch.arange(n, dtype=torch.int32, device="cuda").reshape(-1, 3).repeat(VIEWS, 1).contiguous()
        sc = raster.DeviceScene(sc.pos, sc.col, sc.opa, faces, None)
    tc, td = _targets(views * P)
    rast = raster.Rasterizer(sc, [INTR] * views, raster.Params())
    k = rast.fit(p)
    for sched in ((0, 0, 0), (0, 1, 0), (1, 1, 64)):
        print(f"[count] {views} views, schedule {sched}", flush=True)
        res = []
        for counted in (False, True):
            rast.bin_and_sort(p)
            if counted:
                assert rast.count(p) == k
            loss, color = torch.zeros(views, device="cuda"), torch.empty(3 * P * views, device="cuda")
            res.append([x.clone() for x in rast.train_l1(p, tc, td, color=color, loss=loss, schedule=sched)] + [loss, color])
        for a, b in zip(*res):
            assert float(a.abs().max()) > 0 and _close(b, a)
        assert torch.equal(res[0][5], res[1][5])
    rast.bin_and_sort(p)
    a = [x.clone() for x in rast.forward(p)] + [x.clone() for x in rast.face_stats(p)]
    rast.bin_and_sort(p)
    rast.count(p)
    for x, y in zip(a, list(rast.forward(p)) + list(rast.face_stats(p))):
        assert torch.equal(x, y)
