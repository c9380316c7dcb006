"""The walks take only entries of the tile order that are tiles: with an order that holds none, which no
binning leaves, no tile is walked and every gradient is zero."""
import pytest
import torch

from paper_2605_31419_amd import raster
from paper_2605_31419_amd import scenes as S
from tests import gpu_util as G
from tests.helpers import IDENTITY, tiny_scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("views", [1, 2])
@pytest.mark.parametrize("sched", [(0, 1, 0), (1, 1, 64)])
def test_entries_that_are_no_tiles_are_passed_over(views, sched):
    print(f"[order] {views} views, schedule {sched}", flush=True)
    intr = S.Intrinsics(208, 176, 250.0, 250.0, 103.5, 87.5)
    sc, _ = tiny_scene(3, n_faces=200, w=208, h=176, f=250.0)
    rast, p = G.make(sc, [intr] * views, [IDENTITY] * views)
    n = rast.total_pixels
    tc, td = torch.rand(3 * n, device="cuda"), torch.full((n,), 2.0, device="cuda")
    b = rast.binning()
    nbytes = 4 * b.n_tiles
    # the order ends where the last blended faces start, both on 256-byte boundaries
    at = b.last_face - rast.ws.data_ptr() - (nbytes + 255) // 256 * 256
    order = rast.ws[at:at + nbytes].view(torch.int32)
    rast.bin_and_sort(p)
    torch.cuda.synchronize()
    assert sorted(order.tolist()) == list(range(b.n_tiles))
    got = rast.train_l1(p, tc, td, schedule=sched)
    assert all(float(x.abs().max()) > 0 for x in got)
    order[0::2], order[1::2] = -1, b.n_tiles
    got = rast.train_l1(p, tc, td, schedule=sched)
    torch.cuda.synchronize()
    assert all(float(x.abs().max()) == 0 for x in got)
