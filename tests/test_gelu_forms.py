"""Rings against the wide contraction behind a GELU epilogue (host code: no GPU needed)."""
import ctypes as C

import pytest

from paper_2605_17633_amd import binding as B

GELU = 1


def wide(M, N, K, packed):
    return B.lib().ssam_linear_wide_form(*(C.c_int(v) for v in (M, N, K, GELU, packed, 0)), C.c_size_t(32 << 20))


# us of the routed MLP with the ring and with the wide kernel
@pytest.mark.parametrize("kept,width,packed", [
    (2500, 768, 0),        # 47.1, 45.7
    (2500, 768, 1),        # 47.4, 46.0
    (1944, 1024, 0),       # 55.6, 53.6
    (3483, 576, 0),        # 43.4, 42.3
    (1881, 512, 1),        # 29.8, 29.4
])
def test_wide_where_large_rings_were(kept, width, packed):
    assert wide(kept, 4 * width, width, packed) >= 4


@pytest.mark.parametrize("kept,width,packed", [
    (612, 512, 1),         # 23.9, 25.2
    (120, 576, 0),         # 20.7, 21.9
    (256, 768, 1),         # 22.6, 23.5
    (512, 576, 0),         # 24.6, 25.3
])
def test_small_rings_stay(kept, width, packed):
    assert wide(kept, 4 * width, width, packed) == -1


# with gather and LN2 folded in: rows of the residual stream, rows through the MLP; MLPs or, of the last three, stacks, us a block, with the ring and with this tile
FOLDED = [
    (3584, 1792, 512, 4),         # 26.0 -> 25.3
    (13068, 2613, 512, 6),
    (3969, 2976, 512, 6),         # 31.1 -> 30.6
    (3087, 3087, 512, 7),         # 32.8 -> 31.9
    (5000, 2500, 768, 7),
    (5808, 2323, 768, 7),         # 114.3 -> 113.3
    (8100, 1620, 1024, 7),        # 164.4 -> 158.0
    (4232, 1692, 1024, 7),        # 127.7 -> 125.8
]


@pytest.mark.parametrize("rows,kept,width,tile", FOLDED)
def test_wide_where_large_rings_were_with_the_layernorm_folded_in(rows, kept, width, tile):
    assert B.lib().ssam_fold_gelu_wide_form(*(C.c_int(v) for v in (rows, kept, width, 4 * width))) == tile


def test_the_folded_form_takes_the_wide_kernel_wherever_the_plain_one_leaves_a_ring_of_128_rows():
    """Of the tiles from 128x128; below them the plain form asks both layouts of the weights, the folded one has one."""
    other = []
    for width in (512, 768, 1024):
        for kept in range(900, 3600, 7):
            plain = wide(kept, 4 * width, width, 1)
            folded = B.lib().ssam_fold_gelu_wide_form(*(C.c_int(v) for v in (2 * kept, kept, width, 4 * width)))
            if (plain >= 4 or folded >= 4) and plain != folded:
                other.append((width, kept, plain, folded))
    assert not other
