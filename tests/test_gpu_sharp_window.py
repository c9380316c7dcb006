"""An infinite window exponent leaves a face its incentre alone: 3-4-5 triangles whose incentre is a pixel,
where every edge function is exactly 1, so the window is 1 whatever the exponent."""
import numpy as np
import pytest
import torch

from paper_2605_31419_amd import raster
from paper_2605_31419_amd import scenes as S
from tests.helpers import IDENTITY, plain_scene, unit_cam

pytestmark = pytest.mark.gpu

SCALES = [(2, 1, 1), (3, 10, 2), (4, 20, 14)]          # inradius, first corner


@pytest.mark.parametrize("per_face", [False, True])
@pytest.mark.parametrize("views", [1, 2])
def test_infinite_exponent(per_face, views):
    print(f"[sharp] per_face={per_face} views={views}", flush=True)
    v = [[(x, y, 1.0), (x + 4 * s, y, 1.0), (x, y + 3 * s, 1.0)] for s, x, y in SCALES]
    sc = plain_scene(v, opa=np.full(9, 0.5))
    if per_face:
        sc = S.Scene(sc.pos, sc.col, sc.opa, None, np.full(3, np.inf, np.float32))
    w, h = 48, 32
    rast = raster.Rasterizer(raster.DeviceScene.from_numpy(sc), [unit_cam(w, h)] * views,
                             raster.Params(sigma=1.0 if per_face else float("inf")))
    p = raster.poses_tensor([IDENTITY] * views)
    rast.fit(p)
    rast.bin_and_sort(p)
    color = rast.forward(p)[0].cpu().numpy().reshape(views, 3, h, w)
    want = np.zeros((h, w))
    for s, x, y in SCALES:
        want[y + s, x + s] = 0.5
    assert np.allclose(color, want, atol=1e-6)
    ones = torch.ones(3 * h * w * views, device="cuda")
    grads = rast.backward(p, ones, torch.zeros(h * w * views, device="cuda"))
    assert all(bool(torch.isfinite(g).all()) for g in grads)
    # dL/do_F = 3 (the three channels) a view, a third of it to each vertex
    assert np.allclose(grads[2].cpu().numpy(), views, atol=1e-5)
