"""The fused step under every kind of tile schedule, with and without the longest-first order that tiles
are split in, on a view whose tiles list nothing, a few faces, and more than a split tile's 128: the
separate backward of the same seeds has the same gradients up to the order of the FP32 sums."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2605_31419_amd import scenes as S
from tests import gpu_util as G
from tests import test_gpu_parity as PAR
from tests.helpers import IDENTITY
from tests.test_gpu_walk_edges import NAMES, PIX, SHIFTED, WIDE, _tile

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [0, 3, 150, 300])
@pytest.mark.parametrize("views", [1, 2])
def test_schedules_with_empty_tiles(n, views):
    print(f"[sparse] n={n} views={views}", flush=True)
    few = _tile(5, True)
    sc = few
    if n:
        t = _tile(n, True)
        sc = S.Scene(np.concatenate([few.pos, t.pos], 1), np.concatenate([few.col, t.col], 1), np.concatenate([few.opa, t.opa]), None)
    poses = [IDENTITY, SHIFTED][:views]
    rast, p = G.make(sc, [WIDE] * views, poses)
    c, d, _ = G.render(rast, p)
    ranges = G.binning_arrays(rast)[2].astype(np.int64)
    assert (ranges[:, 1] == ranges[:, 0]).any() and ((ranges[:, 1] - ranges[:, 0]).max() > 128) == (n > 128)
    tcs, tds, seeds = [], [], []
    for v in range(views):
        cv, dv = G.per_view(rast, c, 3)[v], G.per_view(rast, d, 1)[v]
        tc, td, _ = PAR._nudged_targets(cv, dv, 10 * n + v, None)
        tcs.append(tc.reshape(-1))
        tds.append(td.reshape(-1))
        seeds.append(O.l1_seeds(cv, dv, tc, td, PIX))
    sep = rast.backward(p, G.to_dev(np.concatenate([s[1].reshape(-1) for s in seeds])),
                        G.to_dev(np.concatenate([s[2].reshape(-1) for s in seeds])), None)
    loss, color = torch.zeros(views, device="cuda"), torch.empty(3 * PIX * views, device="cuda")
    for sched in ((0, 0, 0), (0, 1, 0), (1, 0, 64), (1, 1, 64), (1, 1, 4096)):
        out = rast.train_l1(p, G.to_dev(np.concatenate(tcs)), G.to_dev(np.concatenate(tds)), color=color, loss=loss,
                            schedule=sched)
        torch.cuda.synchronize()
        assert np.array_equal(color.cpu().numpy(), c)
        assert np.allclose(loss.cpu().numpy(), [float(s[0]) for s in seeds], rtol=1e-5), sched
        for nm, a, b in zip(NAMES, out, sep):
            a, b = a.cpu().numpy().astype(np.float64), b.cpu().numpy().astype(np.float64)
            assert np.linalg.norm(b) > 0 and np.linalg.norm(a - b) <= 1e-5 * np.linalg.norm(b), (sched, nm)
