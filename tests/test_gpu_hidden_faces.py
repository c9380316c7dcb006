"""Faces behind the point where every pixel has stopped are not visited: whatever their colours are
(infinite, not a number), images and the other faces' gradients are those without them."""
import numpy as np
import pytest
import torch

from paper_2605_31419_amd import raster
from paper_2605_31419_amd import scenes as S
from tests import gpu_util as G
from tests.helpers import IDENTITY

pytestmark = pytest.mark.gpu

W, H = 208, 176
INTR = S.Intrinsics(W, H, 200.0, 200.0, 103.5, 87.5)


def _scene(n, value):
    """One opaque face over the whole image, and n faces behind it around the middle tile."""
    g = S.rng(n)
    front = np.array([[(-30.0, -20.0, 1.0), (30.0, -20.0, 1.0), (0.0, 35.0, 1.0)]])
    c = np.stack([g.uniform(-0.2, 0.2, n), g.uniform(-0.2, 0.2, n), g.uniform(2.0, 3.0, n)], 1)
    t1, t2 = S._tangents(S._random_unit(g, n) * 0.3 + np.array([0.0, 0.0, 1.0]))
    verts = np.concatenate([front, S._triangles_around(g, c, g.uniform(0.3, 0.8, n), t1, t2)]) if n else front
    col = np.full((n + 1, 3, 3), value)
    col[0] = S.rng(0).uniform(0, 1, (3, 3))
    return S._pack_soup(verts, col, np.ones((n + 1, 3)))


@pytest.mark.parametrize("value", [np.nan, np.inf], ids=str)
@pytest.mark.parametrize("n", [1, 2, 64, 200])
@pytest.mark.parametrize("views", [1, 2])
def test_hidden_faces(value, n, views):
    print(f"[hidden] {value} n={n} views={views}", flush=True)
    res = []
    for k in (0, n):
        rast, p = G.make(_scene(k, value), [INTR] * views, [IDENTITY] * views, t_min=0.5)
        rast.bin_and_sort(p)
        if k:
            ranges = G.binning_arrays(rast)[2].astype(np.int64)
            assert (ranges[:, 1] - ranges[:, 0]).max() == n + 1
        P = rast.total_pixels
        img = [x.clone() for x in rast.forward(p)]
        assert float(img[2].max()) < 0.5
        out = []
        for sched in ((0, 0, 0), (0, 1, 0)):
            color = torch.empty(3 * P, device="cuda")
            g = rast.train_l1(p, torch.zeros(3 * P, device="cuda"), torch.ones(P, device="cuda"), color=color, schedule=sched)
            assert torch.equal(color, img[0])
            out.append([x.clone() for x in g])
        res.append((img, out))
    for a, b in zip(res[0][0], res[1][0]):
        assert bool(torch.isfinite(a).all()) and torch.equal(a, b)
    for a, b in zip(res[0][1], res[1][1]):                # of the front face (its neighbours' own are 0 * value)
        for x, y in zip(a[:2], b[:2]):
            assert torch.allclose(y.reshape(3, -1)[:, :3], x.reshape(3, -1), rtol=1e-5)
