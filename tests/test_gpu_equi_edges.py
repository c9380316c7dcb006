"""Equilateral regulariser at the sizes where its launches change shape: one face, full and partial
workgroups of 256 faces, and as many workgroups as make the loss sum's threads take one more than
1,024 or 4,096 partial sums; soups with vertices past the faces' last, written and added to."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
gpu = pytest.mark.gpu

from paper_2605_31419_amd import raster


def _reference(pos, weight):
    """Loss and gradient of eq. 14 in FP64 by autograd (pos: [3, 3M] float32)."""
    v = pos.double().reshape(3, -1, 3).permute(1, 2, 0).clone().requires_grad_(True)      # [M, corner, axis]
    e = v.roll(-1, 1) - v
    h = e / e.norm(dim=2, keepdim=True)
    c = -(h * h.roll(1, 1)).sum(2)               # towards the next corner and towards the previous one
    loss = ((c - 0.5) ** 2).mean(1).mean()
    (float(np.float32(weight)) * loss).backward()      # the weight crosses the C interface as a float
    return float(loss.detach()), v.grad.permute(2, 0, 1).reshape(3, -1)


@gpu
@pytest.mark.parametrize("accumulate", [False, True], ids=["write", "add"])
@pytest.mark.parametrize("faces", [1, 255, 256, 257, 1024 * 256 + 1, 4096 * 256 + 1])
def test_equilateral_sizes(faces, accumulate):
    print(f"[equi] faces={faces} accumulate={accumulate}", flush=True)
    extra = 2
    g = np.random.default_rng(faces)
    n = 3 * faces + extra
    pos = g.uniform(-1, 1, (3, n)).astype(np.float32)
    scene = raster.DeviceScene(torch.from_numpy(pos).cuda(), torch.zeros(3, n, device="cuda"),
                               torch.zeros(n, device="cuda"), None)
    assert scene.n_faces == faces
    m3 = 3 * faces
    before = torch.from_numpy(g.normal(size=(3, n)).astype(np.float32)).cuda() if accumulate else None
    grad = before.clone() if accumulate else None
    loss, grad = raster.equilateral(scene, weight=1.2, grad=grad, accumulate=accumulate)
    torch.cuda.synchronize()
    ref_loss, ref_grad = _reference(torch.from_numpy(pos[:, :m3]), 1.2)
    # the loss is one FP32 rounding of an FP64 sum
    assert abs(float(loss) - ref_loss) <= 1.2e-7 * abs(ref_loss)
    got, add = grad.cpu().double(), torch.zeros(3, n, dtype=torch.float64)
    add[:, :m3] = ref_grad
    ref = add + before.cpu().double() if accumulate else add
    # an FP32 rounding of the gradient, and where it is added one of the sum; the FP64 evaluation
    # itself is off by some 1e-15 of the largest term (a short edge divides it)
    tol = 6.1e-8 * (add.abs() + (ref.abs() if accumulate else 0)) + 1e-9 * float(add.abs().max())
    assert ((got - ref).abs() <= tol).all()
