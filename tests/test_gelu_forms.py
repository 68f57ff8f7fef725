"""Rings against the wide contraction behind a GELU epilogue (host code: no GPU needed).  us: the routed MLP, measured with the ring and with the wide kernel."""
import ctypes as C

import pytest

from paper_2605_17633_amd import binding as B

GELU = 1


def wide(M, N, K, packed):
    return B.lib().ssam_linear_wide_form(*(C.c_int(v) for v in (M, N, K, GELU, packed, 0)), C.c_size_t(32 << 20))


@pytest.mark.parametrize("kept,width,packed,us", [(2500, 768, 0, (47.1, 45.7)), (2500, 768, 1, (47.4, 46.0)), (1944, 1024, 0, (55.6, 53.6)), (3483, 576, 0, (43.4, 42.3)), (1881, 512, 1, (29.8, 29.4))])
def test_wide_where_large_rings_were(kept, width, packed, us):
    assert us[1] < us[0] and wide(kept, 4 * width, width, packed) >= 4


@pytest.mark.parametrize("kept,width,packed,us", [(612, 512, 1, (23.9, 25.2)), (120, 576, 0, (20.7, 21.9)), (256, 768, 1, (22.6, 23.5)), (512, 576, 0, (24.6, 25.3))])
def test_small_rings_stay(kept, width, packed, us):
    assert us[0] < us[1] and wide(kept, 4 * width, width, packed) == -1
