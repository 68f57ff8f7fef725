"""Where the row statistics of folded stacks of width 1280 come in pieces, and by which tiles (host code: no GPU needed)."""
import pytest

from test_gpu_row_statistics_long import CASES
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


@pytest.mark.parametrize("images,g,density,us", [(2, 64, 0.2, (204.7, 208.9)), (8, 64, 0.4, (823, 830))])
def test_none_where_they_cost_more_than_a_launch(images, g, density, us):
    """us: a block of the stack, measured without pieces and with them."""
    assert parts(1280, images, g, density)[0] == 0


@pytest.mark.parametrize("images,g,density,us", [(2, 64, 0.3, (223.0, 218.8)), (3, 48, 0.4, (229.6, 219.6)), (2, 32, 0.2, (94.2, 90.8)), (1, 64, 0.2, (129.3, 126.7))])
def test_both_launches_saved_where_that_pays(images, g, density, us):
    assert parts(1280, images, g, density)[0] == 3
