"""Scratch sizes against the bounds that the public header states."""
import ctypes as C

import pytest

from paper_2605_31419_amd import _lib


@pytest.mark.parametrize("size,views,faces", [((16, 16), 1, 1), ((1200, 680), 1, 1_000_000), ((1200, 680), 8, 500_000),
                                              ((333, 251), 1, 60_001), ((481, 269), 3, 120_001), ((2048, 1281), 2, 7)])
def test_mapping_scratch(size, views, faces):
    lib = _lib.load()
    sc = _lib.TsrScene(1, 1, 1, None, 3 * faces, faces, None, None)
    arr = (_lib.TsrIntrinsics * views)(*[_lib.TsrIntrinsics(*size, 100.0, 100.0, 8.0, 8.0)] * views)
    dssim, mapping = C.c_size_t(), C.c_size_t()
    assert lib.tsr_dssim_scratch_size(arr, views, C.byref(dssim)) == 0
    assert lib.tsr_mapping_scratch_size(C.byref(sc), arr, views, C.byref(mapping)) == 0
    tiles = views * ((size[0] + 15) // 16) * ((size[1] + 15) // 16)
    # the D-SSIM scratch + 32 per face + 128 per tile + 3.25 KB
    assert mapping.value <= dssim.value + 32 * faces + 128 * tiles + 3328


def test_workspace_of_several_views_has_no_room_for_split_tiles():
    """Only a single view's tiles are split: per pixel and face, a second view costs what any other does."""
    lib = _lib.load()
    sc = _lib.TsrScene(1, 1, 1, None, 30, 10, None, None)

    def size(n):
        arr = (_lib.TsrIntrinsics * n)(*[_lib.TsrIntrinsics(1024, 512, 100.0, 100.0, 8.0, 8.0)] * n)
        out = C.c_size_t()
        assert lib.tsr_workspace_size(C.byref(sc), arr, n, 0, C.byref(out)) == 0
        return out.value

    tiles, pixels = 64 * 32, 1024 * 512
    # 48 bytes of tables a tile (16 of loss sums, 16 of counters, 4 + 4 of lists, 8 of ranges), 8 of
    # state a pixel, and 4 KB of sums and faces
    assert size(3) - size(2) <= 48 * tiles + 8 * pixels + 24576
