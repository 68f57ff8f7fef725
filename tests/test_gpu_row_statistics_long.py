"""Row statistics in the 20 pieces of rows of 1280: left by the wide contraction, read by it and by the large tiles (-1) with their left-over forms
(which are taken where is checked without a GPU, in test_parts_forms_long.py)."""
import pytest

import test_gpu_row_statistics as short

pytestmark = pytest.mark.gpu

# as in test_gpu_row_statistics.py
CASES = [
    (1280, 6, 8, 0.9, 3, (4, 0, 4, 0), True),
    (1280, 14, 8, 0.9, 3, (4, 1, 6, 1), False),
    (1280, 7, 16, 0.75, 3, (7, 4, -1, 3), False),      # fc1: 280 large tiles
    (1280, 2, 32, 0.6, 3, (7, 4, 7, 3), True),
    (1280, 7, 16, 0.9, 1, (7, 4, 8, 2), True),
    (1280, 7, 16, 1.0, 3, (7, 4, 10, 4), True),
    (1280, 13, 16, 1.0, 3, (11, 6, -1, 6), True),      # fc1: left-over tiles with K cut, and their sum
    (1280, 14, 16, 1.0, 3, (-1, 6, -1, 6), False),     # fc1: left-over tiles in one piece; padding rows behind the large tiles of qkv
    (1280, 2, 24, 0.3, 3, (6, 1, 4, 0), True),
    (1280, 1, 48, 0.2, 3, (8, 4, 4, 0), True),
    (1280, 2, 40, 0.1, 3, (9, 4, 4, 0), True),
    (1280, 5, 32, 1.0, 3, (10, 7, -1, 7), True),       # fc1: whole rounds
    (1280, 7, 32, 1.0, 3, (-1, 9, -1, 9), False),
    (1280, 4, 48, 0.1, 3, (-1, 9, 6, 1), True),
]


@pytest.mark.parametrize("D,images,g,density,form,tiles,kv", CASES)
def test_row_statistics_in_twenty_pieces(D, images, g, density, form, tiles, kv):
    short.test_row_statistics_in_pieces(D, images, g, density, form, tiles, kv)
