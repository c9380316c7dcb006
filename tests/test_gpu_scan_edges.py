"""Binning of views whose tile tables are on both sides of the one-launch scan's round (10,240 tiles),
with an empty last chunk entry and a partial one: lists and ranges against the oracle binner, and an
overflow, which leaves every range empty and is reported."""
import numpy as np
import pytest

from paper_2605_31419_amd import scenes as S
from tests import gpu_util as G
from tests import test_gpu_parity as PAR
from tests.helpers import IDENTITY, tiny_scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h", [(2048, 1280), (2048, 1281), (16384, 176), (16, 16384), (3000, 2000)])
def test_tile_tables_of_several_chunks(w, h):
    print(f"[scan] {w}x{h}", flush=True)
    f = 1.2 * min(w, h) if min(w, h) > 16 else 400.0
    sc, _ = tiny_scene(5, n_faces=60, w=64, h=48, f=60.0)
    intrs = [S.Intrinsics(w, h, f, f, (w - 1) / 2, (h - 1) / 2)]
    rast, p = G.make(sc, intrs, [IDENTITY])
    rast.bin_and_sort(p)
    k = PAR._assert_bins_equal(rast, sc, [IDENTITY], intrs)
    assert k > 0
    # too little room: every range empty, the true total reported
    small, p = G.make(sc, intrs, [IDENTITY], fit=False)
    small.ensure_capacity(1)
    if k > small.capacity:
        small.bin_and_sort(p, check_capacity=False)
        kk, _, ranges, _, overflow = G.binning_arrays(small)
        assert kk == k and int(np.asarray(overflow).reshape(-1)[0]) == 1
        assert not np.asarray(ranges).any()
