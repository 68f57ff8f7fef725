"""Where the row statistics of folded stacks of width 1280 come in pieces, and by which tiles (host code: no GPU needed)."""
import ctypes as C

import pytest

from paper_2605_17633_amd import binding as B
from test_gpu_row_statistics_long import CASES, WIDTHS
from test_parts_forms import parts, reached


def test_the_gpu_tests_reach_every_tile():
    tested = set()
    for D, images, g, density, form, tiles, kv in CASES:
        assert parts(D, images, g, density) == (form, tiles), (D, images, g, density)
        tested |= reached(form, tiles)
    taken = set()
    for images in range(1, 17):
        for g in range(8, 65):
            if images * g * g % 128 == 0:
                for density in (0.1, 0.2, 0.3, 0.4, 0.5, 0.6, 0.75, 0.9, 1.0):
                    taken |= reached(*parts(1280, images, g, density))
    assert taken <= tested, sorted(taken - tested)


# us a block of the stack, without pieces and with them: 204.7, 208.9; 823, 830
@pytest.mark.parametrize("images,g,density", [(2, 64, 0.2), (8, 64, 0.4)])
def test_none_where_they_cost_more_than_a_launch(images, g, density):
    assert parts(1280, images, g, density)[0] == 0


# the same: 223.0, 218.8; 229.6, 219.6; 94.2, 90.8; 129.3, 126.7
@pytest.mark.parametrize("images,g,density", [(2, 64, 0.3), (3, 48, 0.4), (2, 32, 0.2), (1, 64, 0.2)])
def test_both_launches_saved_where_that_pays(images, g, density):
    assert parts(1280, images, g, density)[0] == 3


def test_the_gpu_tests_of_other_widths_take_what_they_name():
    for D, images, g, density, form, tiles, kv, Dm in WIDTHS:
        assert parts(D, images, g, density, Dm) == (form, tiles), (images, g, density, Dm)


def mlp_tiles(rows, kept, D, Dm, form, split_bytes):
    tiles = (C.c_int * 2)()
    B.lib().ssam_mlp_tiles(*(C.c_int(v) for v in (rows, kept, D, Dm, form)), C.c_size_t(split_bytes), tiles)
    return tuple(tiles)


@pytest.mark.parametrize("D", [512, 768, 1024, 1280])
def test_the_launches_take_what_the_form_was_decided_by(D):
    """With the scratch that is left beside the pieces.  (fc2 leaves none in form 1, and takes what it likes.)"""
    whole, other = 32 << 20, 0
    for Dm in (256, 768, 1024, 1536, 2048, 2560, 3840, 4096, 5120, 6144, 8704, 10240, 16384):
        for rows in (128, 640, 1024, 2176, 2304, 2816, 3456, 4096, 7168, 9216, 16384):
            for kept in (rows // 10, rows * 3 // 10, rows // 2, rows * 3 // 4, rows):
                if not kept:
                    continue
                split_bytes, tiles = C.c_size_t(), (C.c_int * 4)()
                sizes = [C.c_int(v) for v in (rows, kept, D, Dm)]
                form = B.lib().ssam_parts_tiles(*sizes, tiles)
                assert B.lib().ssam_parts_plan(*sizes, C.byref(split_bytes)) == form
                if not form:
                    assert split_bytes.value == whole
                    continue
                got = mlp_tiles(rows, kept, D, Dm, form, split_bytes.value)
                assert got[0] == tiles[2] and (form == 1 or got[1] == tiles[3] >= 0), (rows, kept, Dm, form)
                other += form == 3 and got != mlp_tiles(rows, kept, D, Dm, form, whole)
    assert (other > 0) == (D == 1280)        # (the shorter rows' kernels that read or leave pieces cut no K)


# us a block of a stack, without and with pieces: 64.2, 66.7; 83.6, 85.7; 62.2, 64.5; 51.5, 53.8; 536.6, 553.8
@pytest.mark.parametrize("images,g,density,Dm", [(1, 32, 0.3, 2560), (7, 16, 0.2, 2560), (3, 16, 1.0, 1280), (10, 8, 0.4, 768), (4, 48, 1.0, 7680)])
def test_none_for_an_mlp_that_loses_more_than_the_launches(images, g, density, Dm):
    assert parts(1280, images, g, density, Dm)[0] == 0


# kept rows 1280 to 1536 in one round of 256x128 (us a block of a stack with it, with the large tile: 143.4, 151.1; 125.9, 135.8; 132.6, 140.8), 3276 not in two of 192x192 (205.3, 198.9)
@pytest.mark.parametrize("images,g,density,fc1", [(1, 64, 0.35, 7), (2, 40, 0.4, 7), (12, 16, 0.5, 7), (4, 32, 0.8, -1), (1, 64, 0.8, -1)])
def test_fc1_reads_pieces_in_the_faster_tile(images, g, density, fc1):
    assert parts(1280, images, g, density)[1][2] == fc1


# 200.7 us by the wide kernel, 196.4 by the large tile; 160.3, 158.4
@pytest.mark.parametrize("images,g,density", [(5, 32, 0.6), (6, 24, 0.75)])
def test_qkv_reads_pieces_in_the_faster_tile(images, g, density):
    form, tiles = parts(1280, images, g, density)
    assert form == 3 and tiles[0] == -1


@pytest.mark.parametrize("D", [1152, 1280])
def test_every_row_of_pieces_has_what_its_readers_request(D):
    """128 bytes and, above 16 pieces, 32 more: the last row's lie inside the workspace.  (Blocks whose qkv folds its LayerNorm have no width between 1024 and 1280.)"""
    rows, split_bytes = 2048, C.c_size_t()
    assert B.lib().ssam_parts_plan(*(C.c_int(v) for v in (rows, rows // 2, D, 4 * D)), C.byref(split_bytes)) == 3
    assert split_bytes.value == (32 << 20) - 256 - 160 * rows
