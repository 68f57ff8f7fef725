"""Row statistics in the 20 pieces of rows of 1280: left by the wide contraction, read by it and by the large tiles (-1) with their left-over forms
(which are taken where is checked without a GPU, in test_parts_forms_long.py)."""
import pytest

import test_gpu_row_statistics as short

pytestmark = pytest.mark.gpu

# as in test_gpu_row_statistics.py
CASES = [
    (1280, 6, 8, 0.9, 3, (4, 0, 4, 0), True),
    (1280, 14, 8, 0.9, 3, (4, 1, 6, 1), False),
    (1280, 7, 16, 0.75, 3, (7, 4, 7, 3), False),
    (1280, 10, 16, 1.0, 3, (10, 4, -1, 4), False),     # fc1: 400 large tiles
    (1280, 2, 32, 0.6, 3, (7, 4, 7, 3), True),
    (1280, 7, 16, 0.9, 1, (7, 4, 8, 2), True),
    (1280, 7, 16, 1.0, 3, (7, 4, 10, 4), True),
    (1280, 13, 16, 1.0, 3, (-1, 6, -1, 6), True),      # fc1: left-over tiles with K cut, and their sum
    (1280, 14, 16, 1.0, 3, (-1, 6, -1, 6), False),     # fc1: left-over tiles in one piece; padding rows behind the large tiles of qkv
    (1280, 2, 24, 0.3, 3, (6, 1, 4, 0), True),
    (1280, 1, 48, 0.2, 3, (8, 4, 4, 0), True),
    (1280, 2, 40, 0.1, 3, (9, 4, 4, 0), True),
    (1280, 5, 32, 1.0, 3, (-1, 7, -1, 7), True),       # fc1: whole rounds
    (1280, 7, 32, 1.0, 3, (-1, 9, -1, 9), False),
    (1280, 4, 48, 0.1, 3, (-1, 9, 6, 1), True),
]


@pytest.mark.parametrize("D,images,g,density,form,tiles,kv", CASES)
def test_row_statistics_in_twenty_pieces(D, images, g, density, form, tiles, kv):
    short.test_row_statistics_in_pieces(D, images, g, density, form, tiles, kv)


# with MLPs that are not four times as wide: the large tile's forms that D * 4 does not reach, as kept rows x Dm here
WIDTHS = [
    (1280, 16, 4, 0.1, 1, (0, 0, -1, -1), True, 10240),     # 40 tiles, all of them left over: K cut in a launch of its own, and their sum; 16 rows
    (1280, 3, 16, 0.02, 1, (4, 0, -1, -1), False, 10240),   # the same, ragged rows
    (1280, 1, 64, 0.4, 1, (-1, 6, -1, 2), False, 10240),    # a round and left-over tiles with K cut
    (1280, 2, 32, 0.9, 1, (7, 4, -1, -1), True, 10240),     # a round and left-over tiles in one piece
    (1280, 2, 64, 0.75, 1, (-1, 9, 7, -1), False, 1280),
    (1280, 1, 64, 1.0, 3, (-1, 6, 5, 6), False, 1536),
    (1280, 8, 32, 0.75, 3, (-1, 9, 9, 7), True, 2048),
    (1280, 11, 16, 0.75, 3, (10, 4, -1, 4), True, 9216),    # fc2 would take the large tile with all of the scratch, and leaves pieces beside them
]


@pytest.mark.parametrize("D,images,g,density,form,tiles,kv,Dm", WIDTHS)
def test_row_statistics_in_twenty_pieces_of_other_widths(D, images, g, density, form, tiles, kv, Dm):
    short.check_row_statistics_in_pieces(D, images, g, density, form, tiles, kv, Dm)
