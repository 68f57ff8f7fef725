"""Which contractions take one large workgroup per CU, and which of its tiles (host code: no GPU needed)."""
import ctypes as C

import pytest

from paper_2605_17633_amd import binding as B
from test_gpu_linear_small import FOLDED as SMALL_FOLDED, FORM_CASES, MLP as SMALL_MLP
from test_gpu_linear_wide import CASES, FOLDED, MLP, STRIDED


def wide(M, N, K, epi=0, packed=False, folded=False, ws=32 << 20):
    return B.lib().ssam_linear_wide_form(*(C.c_int(int(v)) for v in (M, N, K, epi, packed, folded)), C.c_size_t(ws))


def test_the_gpu_tests_reach_every_tile():
    for tile, packed, epi, M, N, K in CASES:
        assert wide(M, N, K, epi, packed, ws=0) == tile, (tile, packed, epi, M, N, K)
    for tile, M, N, K in FOLDED:
        assert wide(M, N, K, 3, True, folded=True) == tile, (tile, M, N, K)
    for tile, rows, Dm, D in MLP:
        assert wide(rows, Dm, D, 1, True) == tile, (tile, rows, Dm, D)
    assert {c[:3] for c in CASES} == {(t, p, e) for t in range(12) for p in (False, True) for e in range(4)}
    assert {c[0] for c in FOLDED} == {c[0] for c in MLP} == set(range(12))


def test_the_small_kernels_keep_the_shapes_they_are_tested_with():
    for _, packed, epi, M, N, K in FORM_CASES:
        assert wide(M, N, K, epi, packed, ws=0) == -1, (packed, epi, M, N, K)
    for _, M, N, K in SMALL_FOLDED:
        assert wide(M, N, K, 3, True, folded=True) == -1, (M, N, K)
    for _, rows, Dm, D in SMALL_MLP:
        assert wide(rows, Dm, D, 1, True) == -1, (rows, Dm, D)


@pytest.mark.parametrize("M,N,K", [(1000, 768, 768 + 8), (1000, 768, 256), (1 << 20, 1280, 1280)])
def test_what_is_left_to_the_others(M, N, K):
    """A ragged last slab, fewer than five slabs, many rounds."""
    assert wide(M, N, K) == -1


@pytest.mark.parametrize("epi", [0, 1, 2, 3])
def test_two_chains_whatever_the_layout(epi):
    """Tiles below 128x128 (two chains over K) are taken with both layouts of the weights or with neither."""
    for M in range(33, 3000, 97):
        for N, K in ((768, 768), (768, 3072), (1280, 1280), (3072, 768), (256, 1024)):
            a, b = wide(M, N, K, epi, False), wide(M, N, K, epi, True)
            assert a == b or not (0 <= a < 4 or 0 <= b < 4), (M, N, K, a, b)


def wide_ld(M, N, K, epi, packed, lda, ldw, ws=32 << 20):
    return B.lib().ssam_linear_wide_form_ld(*(C.c_int(int(v)) for v in (M, N, K, epi, packed, False)), C.c_size_t(ws), C.c_int(lda), C.c_int(ldw))


def test_row_strides_reach_the_kernel():
    for tile, packed, epi, M, N, K, pa, pw, _ in STRIDED:
        assert wide_ld(M, N, K, epi, packed, K + pa, K + pw, ws=0) == tile, (tile, packed, epi, M, N, K, pa, pw)
    assert {t < 4 for t, *_ in STRIDED} == {True, False}


@pytest.mark.parametrize("M,N,K,epi,us", [(130, 864, 4096, 1, (18.4, 21.1)), (34, 3016, 3072, 0, (18.8, 21.1)), (439, 328, 4224, 1, (19.5, 22.6)),
                                          (123, 2096, 3712, 1, (21.6, 29.3))])
def test_rows_that_tear_lines_are_charged(M, N, K, epi, us):
    """us: measured with rows of A and W that do not begin on 128 bytes, the others and this kernel."""
    assert wide_ld(M, N, K, epi, False, K + 8, K + 8) == -1
    assert wide_ld(M, N, K, epi, False, K + 64, K + 64) == wide(M, N, K, epi) >= 0


@pytest.mark.parametrize("M,N,K,epi,packed,us", [(22, 1088, 3456, 0, False, (14.1, 16.9)), (177, 984, 5120, 1, False, (20.0, 26.4)), (158, 272, 4224, 2, False, (16.0, 19.9)),
                                                 (34, 2888, 4032, 1, False, (16.3, 20.6)), (57, 4224, 4800, 1, True, (21.6, 25.5))])
def test_few_rows_and_a_long_k_keep_the_k_split(M, N, K, epi, packed, us):
    """us: measured with weights from memory, K cut over many workgroups and this kernel."""
    assert wide(M, N, K, epi, packed) == -1
