"""Where the row statistics of a folded stack come in pieces that its projections leave, and by which tiles (host code: no GPU needed)."""
import ctypes as C

import pytest

from paper_2605_17633_amd import binding as B
from test_gpu_row_statistics import CASES


def parts(D, images, g, density):
    tiles = (C.c_int * 4)()
    form = B.lib().ssam_parts_tiles(C.c_int(images * g * g), C.c_int(images * B.ssam_keep_count(g * g, density)), C.c_int(D), C.c_int(4 * D), tiles)
    return form, tuple(tiles)


def test_the_gpu_tests_reach_their_tiles():
    for D, images, g, density, form, tiles, kv in CASES:
        assert parts(D, images, g, density) == (form, tiles), (D, images, g, density)
    assert {c[4] for c in CASES} == {1, 3} and {c[6] for c in CASES if c[4] == 3} == {True, False}


@pytest.mark.parametrize("D,g,images,density", [(1024, 36, 8, 0.2), (768, 48, 6, 0.2), (768, 48, 3, 0.4), (768, 32, 7, 0.4)])
def test_fc2_keeps_its_tile(D, g, images, density):
    """Where qkv reads no pieces fc2 leaves none: 96x96 is its fastest tile (23.1 to 29.1 us; of those that leave pieces 128x128, 23.7 to 32.3)."""
    form, tiles = parts(D, images, g, density)
    kept = images * B.ssam_keep_count(g * g, density)
    assert form == 1 and tiles[3] == 2 == B.lib().ssam_linear_wide_form(*(C.c_int(v) for v in (kept, D, 4 * D, 2, 1, 0)), C.c_size_t(32 << 20))
