"""A seed that is not a number reaches the gradients of the faces that some pixel of its 8x8 quadrant
blends, and no others: not a face that the quadrant lists but that covers none of its pixels, and not
the face that stands in where a quadrant has an odd number of faces to visit (the first of the list)."""
import numpy as np
import pytest
import torch

from paper_2605_31419_amd import raster
from paper_2605_31419_amd import scenes as S
from tests import gpu_util as G
from tests.helpers import IDENTITY, plain_scene

pytestmark = pytest.mark.gpu

INTR = S.Intrinsics(16, 16, 20.0, 20.0, 7.5, 7.5)
PIX = (12, 12)                                     # in the last quadrant
FACES = {                                          # pixel coordinates of the corners, depth
    "other": ([(1.0, 1.0), (6.0, 1.5), (2.0, 6.0)], 1.0),             # in the first quadrant only
    "between": ([(9.55, 9.15), (14.55, 14.15), (9.65, 9.05)], 1.5),   # between the pixels' diagonals
    "seen": ([(9.0, 9.5), (15.0, 10.0), (11.0, 15.0)], 2.0),
}


def _scene(names):
    v = []
    for n in names:
        corners, z = FACES[n]
        v.append([((x - INTR.cx) / INTR.fx * z, (y - INTR.cy) / INTR.fy * z, z) for x, y in corners])
    return plain_scene(np.asarray(v, np.float32))


@pytest.mark.parametrize("names", [("other", "seen"), ("other", "between", "seen")], ids="+".join)
@pytest.mark.parametrize("views", [1, 2])
@pytest.mark.parametrize("mode", [dict(sigma=1.0), dict(sigma=0.5), dict(sigma=0.8, perspective=True)], ids=str)
@pytest.mark.parametrize("channel", ["colour", "depth", "trans"])
def test_nan_seed(names, views, mode, channel):
    print(f"[nan] {names} {views} {mode} {channel}", flush=True)
    dev = raster.DeviceScene.from_numpy(_scene(names))
    rast = raster.Rasterizer(dev, [INTR] * views, raster.Params(**mode))
    p = raster.poses_tensor([IDENTITY] * views)
    rast.fit(p)
    rast.bin_and_sort(p)
    ranges = G.binning_arrays(rast)[2]
    assert (ranges[:, 1] - ranges[:, 0] == len(names)).all()
    rast.forward(p)
    g = np.random.default_rng(1)
    seeds = [g.normal(size=(views, ch, 16, 16)).astype(np.float32) for ch in (3, 1, 1)]
    k = ("colour", "depth", "trans").index(channel)

    def grads(value):
        s = [x.copy() for x in seeds]
        s[k][0, 0, PIX[1], PIX[0]] = value
        out = rast.backward(p, *[G.to_dev(x) for x in s])[:3]
        pos, col = (x.cpu().numpy().reshape(3, len(names), 3) for x in out[:2])
        return pos, col, out[2].cpu().numpy().reshape(len(names), 3)

    for i, (a, b) in enumerate(zip(grads(0.0), grads(np.nan))):
        a, b = np.moveaxis(a, -2, 0), np.moveaxis(b, -2, 0)        # by face
        assert np.isfinite(a).all() and np.abs(a[0]).max() > 0
        assert i > 0 or np.isnan(b[-1]).any()                      # (positions: every kind of seed reaches them)
        assert np.allclose(b[:-1], a[:-1], rtol=1e-6, atol=0.0)
        if "between" in names:
            assert not b[1].any()
