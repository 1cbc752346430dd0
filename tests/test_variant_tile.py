"""wave_variant_tile: the tile a workgroup of each variant covers."""
import ctypes
import os

import pytest

from paper_2404_04441_amd import _lib as L


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(L.LIB_PATH):
        from paper_2404_04441_amd.build import build
        build()
    return L.lib()


def test_tiles_hold_the_nodes_of_their_lanes(lib):
    info, tile = (ctypes.c_int32 * 5)(), (ctypes.c_int32 * 2)()
    widths = set()
    for v in range(lib.wave_variant_count()):
        assert lib.wave_variant_info(v, info) == 0 and lib.wave_variant_tile(v, tile) == 0
        fam, by, ry, _, vec = list(info)
        nodes = tile[0] * tile[1]
        if fam in (1, 2):
            assert list(tile) == [64, by]
        elif v < 20:
            assert list(tile) == [64 * vec, by * ry]
        elif v < 29:
            assert nodes == 64 * by * ry * vec
        else:  # padded forms: the tile of the shape, whose vec they don't report
            assert nodes in (64 * by * ry, 128 * by * ry, 256 * by * ry)
        widths.add(tile[0])
    assert {64, 128, 192, 256, 320} <= widths
    assert lib.wave_variant_tile(lib.wave_variant_count(), tile) == L.WAVE_EINVAL
    assert lib.wave_variant_tile(-1, tile) == L.WAVE_EINVAL
    assert lib.wave_variant_tile(0, None) == L.WAVE_EINVAL
