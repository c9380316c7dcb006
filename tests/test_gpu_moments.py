"""Accuracy of the colour gradients' sums for large faces whose tiles are split between two workgroups:
a face of a hundred pixels takes some two hundred FP32 additions per plane moment, from tiles all
around it.  The reference is the same backward, one tile's seeds at a time (a gradient is linear in its
seeds, and every other tile then adds zeros), summed in 64 bits: the two differ by the rounding of
the sums alone.  An emulation of the sums in this scene (FP32 additions in random order, seeds 1 to 3)
gives relative errors of 4.8e-7 to 5.2e-7 with moments about the corner of a face's rectangle and whole
tiles, 6.7e-7 to 6.8e-7 with every tile split, and 2.6e-7 to 3.7e-7 about the middle, whole or split;
the bound lies between the last two kinds."""
import numpy as np
import pytest

from paper_2605_31419_amd import scenes as S
from tests import gpu_util as G
from tests.helpers import IDENTITY

pytestmark = pytest.mark.gpu

W, H = 208, 176                       # 13 x 11 tiles: enough for a single view to split
INTR = S.Intrinsics(W, H, 200.0, 200.0, 103.5, 87.5)
TOL = 4.3e-7


def _large_faces(seed, n=260):
    """Faint fronto-parallel faces of 100 to 160 pixels radius all over the image, squeezed to 0.3 to 1."""
    g = S.rng(seed)
    c = np.stack([g.uniform(0, W, n), g.uniform(0, H, n)], 1)
    r, squeeze, rot = np.exp(g.uniform(np.log(100), np.log(160), n)), g.uniform(0.3, 1, n), g.uniform(0, 2 * np.pi, n)
    ang = g.uniform(0, 2 * np.pi, n)[:, None] + 2 * np.pi / 3 * np.arange(3)
    x, y = r[:, None] * np.cos(ang), (r * squeeze)[:, None] * np.sin(ang)
    co, si = np.cos(rot)[:, None], np.sin(rot)[:, None]
    u, v = c[:, :1] + x * co - y * si, c[:, 1:] + x * si + y * co
    z = g.uniform(1, 3, n)[:, None] * np.ones(3)
    verts = np.stack([(u - INTR.cx) / INTR.fx * z, (v - INTR.cy) / INTR.fy * z, z], -1)
    return S._pack_soup(verts, g.uniform(0, 1, (n, 3, 3)), g.uniform(0.002, 0.02, (n, 3)))


def _grad_col(out):
    return out[1].cpu().numpy().astype(np.float64).reshape(-1)


@pytest.mark.parametrize("fused", [False, True])
def test_colour_gradients_of_split_tiles(fused):
    errs = []
    tile = (np.arange(H) // 16)[:, None] * 13 + (np.arange(W) // 16)[None, :]
    for seed in (1, 2, 3):
        print(f"[moments] fused {fused}, seed {seed}", flush=True)
        rast, p = G.make(_large_faces(seed), [INTR], [IDENTITY])
        rast.bin_and_sort(p)
        _, _, ranges, _, _ = G.binning_arrays(rast)
        assert ((ranges[:, 1].astype(np.int64) - ranges[:, 0]) > 128).sum() >= 40
        img, zero = rast.forward(p)[0].cpu().numpy().reshape(3, H, W), G.to_dev(np.zeros(W * H))
        gc = np.random.default_rng(seed).uniform(0.5, 1.5, size=(3, H, W)).astype(np.float32)

        def grad(mask):
            if not fused:
                return _grad_col(rast.backward(p, G.to_dev(gc * mask), zero))
            # L1 seeds: w_color / (3 W H) where the target lies below the image, 0 where it is the image
            return _grad_col(rast.train_l1(p, G.to_dev(np.where(mask, -1.0, img)), zero, schedule=(0, 1, 0)))

        whole = grad(np.ones((H, W), bool))
        parts = sum(grad(tile == t) for t in range(143))
        errs.append(np.linalg.norm(whole - parts) / np.linalg.norm(parts))
    print(f"[moments] fused {fused}: {errs}", flush=True)
    assert np.mean(errs) <= TOL, errs
