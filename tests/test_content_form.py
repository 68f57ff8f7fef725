"""Which kernel makes the content-aware tables (host code: no GPU needed)."""
import ctypes as C

import pytest

from paper_2605_17633_amd import binding as B


@pytest.mark.parametrize("w,groups,count,sort", [
    (4, 6400, 9.6, 7.4), (8, 1600, 9.8, 6.9), (8, 12800, 57.4, 17.1), (10, 800, 10.8, 8.0), (14, 525, 14.0, 10.4), (14, 800, 19.1, 10.8), (14, 12800, 235, 48.1),
    (16, 3200, 72.7, 16.8), (24, 400, 29.1, 18.3), (32, 200, 33.0, 16.5), (64, 50, 80.4, 40.4), (128, 16, 297.9, 161.9),
    (4, 25, 2.9, 4.2), (8, 200, 3.7, 6.2), (14, 25, 3.6, 9.4), (14, 200, 7.1, 9.4), (24, 50, 6.6, 15.6), (32, 50, 11.4, 16.2), (50, 2, 6.0, 38), (64, 1, 7.5, 39.7),
    (64, 8, 17, 40), (128, 1, 26.0, 160.9), (128, 4, 83.9, 163.4)])
def test_the_faster_form_is_taken(w, groups, count, sort):
    """count, sort: measured us."""
    assert B.lib().ssam_content_tables_form(C.c_long(groups), C.c_int(w)) == (count < sort)


def test_a_counting_launch_stays_within_the_launch_limit():
    """blocks * threads has to stay below 2^32; the sort launches at most 1024 threads a group, 64 for the smallest ones."""
    for w in (1, 2, 3, 4, 8, 14, 32, 64, 128):
        for groups in (1 << 16, 1 << 20, 1 << 24):
            assert not B.lib().ssam_content_tables_form(C.c_long(groups), C.c_int(w))
