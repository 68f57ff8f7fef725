"""Where the row statistics of a folded stack come in pieces that its projections leave, and by which tiles (host code: no GPU needed)."""
import ctypes as C

import pytest

from paper_2605_17633_amd import binding as B
from test_gpu_row_statistics import CASES


def parts(D, images, g, density, Dm=None):
    tiles = (C.c_int * 4)()
    form = B.lib().ssam_parts_tiles(C.c_int(images * g * g), C.c_int(images * B.ssam_keep_count(g * g, density)), C.c_int(D), C.c_int(Dm or 4 * D), tiles)
    return form, tuple(tiles)


def reached(form, tiles):
    """What leaves or reads pieces: (contraction, tile)."""
    qkv, proj, fc1, fc2 = tiles
    return {1: {("proj", proj), ("fc1", fc1)}, 3: {("qkv", qkv), ("proj", proj), ("fc1", fc1), ("fc2", fc2)}}.get(form, set())


def test_the_gpu_tests_reach_every_tile():
    tested = set()
    for D, images, g, density, form, tiles, kv in CASES:
        assert parts(D, images, g, density) == (form, tiles), (D, images, g, density)
        tested |= reached(form, tiles)
    taken = set()
    for D in (512, 768, 1024):                    # the widths that fold LN1 (3 D % 256 == 0) in at most 16 pieces and at least five slabs
        for images in range(1, 17):
            for g in range(8, 65):
                if images * g * g % 128 == 0:
                    for density in (0.1, 0.2, 0.3, 0.4, 0.5, 0.6, 0.75, 0.9, 1.0):
                        taken |= reached(*parts(D, images, g, density))
    assert taken <= tested, sorted(taken - tested)
    assert {c[4] for c in CASES} == {1, 3} and {c[6] for c in CASES if c[4] == 3} == {True, False}


@pytest.mark.parametrize("D,g,images,density", [(1024, 36, 8, 0.2), (768, 48, 6, 0.2), (768, 48, 3, 0.4), (768, 32, 7, 0.4), (1024, 24, 6, 0.6)])
def test_fc2_keeps_its_tile(D, g, images, density):
    """No tile that leaves pieces is as fast for fc2 as 96x96 here (23.1 to 29.1 us; 128x128 23.7 to 32.3), by more than what qkv could save."""
    form, tiles = parts(D, images, g, density)
    kept = images * B.ssam_keep_count(g * g, density)
    assert form < 3 and tiles[3] == 2 == B.lib().ssam_linear_wide_form(*(C.c_int(v) for v in (kept, D, 4 * D, 2, 1, 0)), C.c_size_t(32 << 20))


# us a block of the stack, without pieces and with pieces for fc1: 166.4, 168.8; 163.2, 164.1
@pytest.mark.parametrize("D,g,images,density", [(768, 64, 3, 0.2), (768, 40, 8, 0.2)])
def test_none_where_they_cost_more_than_a_launch(D, g, images, density):
    assert parts(D, images, g, density)[0] == 0


# the same, and with all pieces: 76.8, 73.6; 118.2, 113.4; 84.3, 78.7; 103.3, 100.1
@pytest.mark.parametrize("D,g,images,density", [(768, 40, 2, 0.4), (1024, 64, 1, 0.4), (768, 48, 2, 0.2), (1024, 24, 6, 0.4)])
def test_both_launches_saved_where_that_pays(D, g, images, density):
    assert parts(D, images, g, density)[0] == 3
