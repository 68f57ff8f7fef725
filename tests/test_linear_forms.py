"""Which kernel the library takes for a contraction (host code: no GPU needed)."""
import ctypes as C

import pytest

from paper_2605_17633_amd import binding as B
from test_gpu_linear_small import FOLDED, FORM_CASES, MLP

WS = 32 << 20


def form(M, N, K, epi=0, packed=False, folded=False, ws=WS):
    return B.lib().ssam_linear_form(*(C.c_int(int(v)) for v in (M, N, K, epi, packed, folded)), C.c_size_t(ws))


@pytest.mark.parametrize("M,N,K,epi,packed,us", [
    (42, 1560, 5120, 0, False, (17.3, 32.1)), (318, 1280, 5120, 2, False, (24.5, 31.8)), (384, 1024, 4096, 2, False, (22.4, 26.0)),
    (62, 576, 2304, 1, False, (13.0, 16.3)), (427, 3824, 4560, 1, False, (44.1, 54.0)), (1230, 2008, 3688, 2, False, (48.6, 55.2)),
    (399, 1280, 5120, 2, False, (26.2, 31.8)), (429, 1408, 5312, 0, True, (26.4, 31.4)), (489, 1280, 5120, 3, True, (25.8, 29.6)),
    (40, 5504, 3712, 1, True, (20.7, 24.8)), (378, 1024, 4096, 0, True, (20.9, 23.7))])
def test_few_rows_and_a_long_k_keep_the_k_split(M, N, K, epi, packed, us):
    """us: measured, K cut over many workgroups | a ring of 64x64 tiles that walks all of K."""
    assert form(M, N, K, epi, packed) < 16


@pytest.mark.parametrize("M,N,K,epi,packed,us", [
    (313, 768, 3072, 2, True, (17.1, 8.9)), (65, 1024, 4096, 3, True, (16.0, 13.6)), (784, 2304, 768, 3, True, (21, 7.7)),
    (1638, 768, 3072, 2, True, (25.9, 20.1)), (1638, 1280, 1280, 2, True, (22.2, 15.1)), (4096, 768, 768, 2, False, (17.8, 11.6)),
    (8192, 576, 2304, 2, False, (45, 32)), (3357, 128, 384, 0, True, (8.3, 4.4))])
def test_small_problems_take_the_small_kernels(M, N, K, epi, packed, us):
    """us: measured, large tiles | the kernel taken."""
    assert form(M, N, K, epi, packed) >= 16


def test_large_problems_take_the_large_tiles():
    for M in (16384, 32768):
        for N, K in ((2304, 768), (3840, 1280), (5120, 1280), (1280, 5120)):
            assert form(M, N, K, 0, True) < 16 and form(M, N, K, 0, False) < 16
    assert form(32768, 3840, 1280, 3, True, folded=True) == 4


def test_the_gpu_tests_reach_every_small_kernel():
    for f, packed, epi, M, N, K in FORM_CASES:
        assert form(M, N, K, epi, packed, ws=0) == f, (f, packed, epi, M, N, K)
    for f, M, N, K in FOLDED:
        assert form(M, N, K, 3, True, folded=True) == f, (f, M, N, K)
    for f, rows, Dm, D in MLP:
        assert form(rows, Dm, D, 1, True) == f, (f, rows, Dm, D)
