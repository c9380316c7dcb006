"""Tile lists at the lengths where the workgroup merge sort changes shape: the last and first lengths
of its two sizes (2,048 and 4,096 keys), partial runs, and lists of several chunks whose last one is
shorter than a run or has a few keys over it."""
import pytest

from paper_2605_31419_amd import scenes as S
from tests import gpu_util as G
from tests import test_gpu_parity as PAR
from tests.helpers import IDENTITY

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1500, 1537, 2047, 2048, 2049, 2561, 4095, 4096 + 300, 4096 + 513, 8193])
def test_long_tile_lists(n):
    print(f"[tile sort] one tile of {n} faces", flush=True)
    sc = PAR._one_tile_scene(n, seed=n)
    intrs = [S.Intrinsics(16, 16, 20.0, 20.0, 7.5, 7.5)]
    rast, p = G.make(sc, intrs, [IDENTITY])
    rast.bin_and_sort(p)
    assert PAR._assert_bins_equal(rast, sc, [IDENTITY], intrs) == n
