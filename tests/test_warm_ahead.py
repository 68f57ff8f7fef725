"""Which weights a launch with idle compute units reads ahead (host code: no GPU needed)."""
import ctypes as C

import pytest

from paper_2605_17633_amd import binding as B

NAMES = ("wqkv", "wproj", "w1", "w2")


def pieces(ws, D, Dm, now, groups, most):
    at, nbytes = (C.c_void_p * 3)(), (C.c_uint32 * 3)()
    k = B.lib().ssam_warm_pieces(ws, C.c_int(len(ws)), C.c_int(D), C.c_int(Dm), C.c_int(now), C.c_int(groups), C.c_double(most), at, nbytes)
    assert 0 <= k <= 3
    return [(at[i], nbytes[i]) for i in range(k)]


def stack(blocks, D, Dm, base=1 << 40):
    """Blocks whose weights lie one behind the other, 4 KB between them."""
    ws, spans = (B.BlockWeights * blocks)(), []
    for i in range(blocks):
        for name, size in zip(NAMES, (6 * D * D, 2 * D * D, 2 * D * Dm, 2 * D * Dm)):
            setattr(ws[i], name, base)
            spans.append((base, size))
            base += size + 4096
    return ws, spans


@pytest.mark.parametrize("D,Dm,blocks,most", [(768, 3072, 3, 1e12), (128, 128, 2, 1e12), (1024, 4096, 2, 3e6), (1280, 5120, 2, 8191.0), (1280, 5120, 2, 0.0)])
def test_pieces_lie_inside_the_next_weights_and_none_is_read_twice(D, Dm, blocks, most):
    ws, spans = stack(blocks, D, Dm)
    seen = {}
    for now in range(4 * blocks):
        total = 0
        for at, n in pieces(ws, D, Dm, now, 32, most):
            i = next(j for j, (b, size) in enumerate(spans) if b <= at < b + size)
            assert now < i <= now + 2 and n > 0 and n % 16 == 0
            assert at - spans[i][0] == seen.get(i, 0) and at + n <= spans[i][0] + spans[i][1]
            seen[i] = seen.get(i, 0) + n
            total += n
        assert total <= most
    if most == 1e12:
        assert seen == {i: size for i, (_, size) in enumerate(spans) if i > 0}


def test_missing_and_misaligned_weights_are_left_to_the_contraction():
    ws, _ = stack(2, 256, 1024)
    ws[0].w1 = None
    ws[1].wproj = ws[1].wproj + 8
    assert len(pieces(ws, 256, 1024, 0, 32, 1e12)) == 1      # wproj, not the missing w1
    assert pieces(ws, 256, 1024, 1, 32, 1e12) == []
    assert len(pieces(ws, 256, 1024, 2, 32, 1e12)) == 2      # w2 and the next wqkv
    assert pieces(ws, 256, 1024, 3, 32, 1e12) == []          # not the misaligned wproj


def stack_of_two_kinds(flags, D, Dm, base=1 << 40):
    ws, spans = (B.BlockWeights * len(flags))(), []
    for i, f in enumerate(flags):
        for name, size in zip(NAMES, (6 * D * D, 2 * D * D, 2 * D * Dm[f], 2 * D * Dm[f])):
            setattr(ws[i], name, base)
            spans.append((base, size))
            base += size + 4096
    return ws, spans


@pytest.mark.parametrize("Dm", [(4096, 1024), (1024, 4096), (2048, 2048)])
@pytest.mark.parametrize("flags", [(0, 1, 0, 1), (1, 0, 0, 1, 1), (1, 1), (0, 0)])
def test_a_block_of_either_kind_has_its_own_width(flags, Dm):
    """Windowed blocks of one MLP width, global ones of another: every piece inside the weight that it is of, and all of them read."""
    D = 512
    ws, spans = stack_of_two_kinds(flags, D, Dm)
    cfg = [B.make_cfg(1, 16, D, D // 64, Dm[f], 0 if f else 14, 128 if f else 32, 100, 0.4) if f in flags else None for f in (0, 1)]
    seen = {}
    for now in range(4 * len(flags)):
        at, nbytes = (C.c_void_p * 3)(), (C.c_uint32 * 3)()
        k = B.lib().ssam_warm_pieces_of_stack(ws, (C.c_uint8 * len(flags))(*flags), C.c_int(len(flags)), *(c and C.byref(c) for c in cfg),
                                              C.c_int(now), C.c_int(32), C.c_double(1e12), at, nbytes)
        assert 0 <= k <= 3
        for j in range(k):
            i = next(j2 for j2, (b, size) in enumerate(spans) if b <= at[j] < b + size)
            assert at[j] - spans[i][0] == seen.get(i, 0)
            seen[i] = seen.get(i, 0) + nbytes[j]
            assert seen[i] <= spans[i][1], (now, i)
    assert seen == {i: size for i, (_, size) in enumerate(spans) if i > 0}


def budget(tiles, fills, us, blocks=12):
    most = C.c_double()
    return B.lib().ssam_warm_budget(C.c_int(blocks), C.c_int(tiles), C.c_int(fills), C.c_double(us), C.byref(most)), most.value


@pytest.mark.parametrize("tiles,us", [(240, 13.4), (504, 54.0), (760, 91.0), (1000, 130.0), (512 + 64, 80.0)])
def test_a_launch_reads_in_its_last_round(tiles, us):
    """A CU without a tile in the last of several rounds has tiles until then: no more than it can read from there on, at 30 KB a microsecond."""
    groups, most = budget(tiles, 0, us)
    assert 8 <= groups <= -tiles % 256
    assert 0 < most <= groups * 30e3 * us / -(-tiles // 256) * (1 + 1e-12)


@pytest.mark.parametrize("us", [20.0, 31.3])
@pytest.mark.parametrize("tiles,fills", [(256, 51), (512, 102), (250, 51), (192, 51), (192, 0), (192, 100), (64, 400)])
def test_padding_rows_are_no_tiles(tiles, fills, us):
    """Workgroups of padding rows behind the tiles: they open no round, and take some of the idle CUs' time."""
    groups, most = budget(tiles, fills, us)
    alone, most_alone = budget(tiles, 0, us)
    assert groups in (0, alone) and most <= most_alone
    assert (groups > 0) == (most > 0)
    if alone:
        assert most < most_alone or not fills
    if (tiles, fills) == (192, 51):
        assert most > 0.8 * most_alone


@pytest.mark.parametrize("tiles", [8, 64, 184, 200, 248, 256, 300, 500])
def test_few_workgroups_read(tiles):
    """More than 64 stand in the way of the tiles; fewer than 8 CUs are not worth a launch's while."""
    idle = -tiles % 256
    assert budget(tiles, 0, 12.0)[0] == (min(idle, 64) if idle >= 8 else 0)


@pytest.mark.parametrize("tiles", [64, 192, 240, 504])
def test_a_block_by_itself_reads_nothing(tiles):
    """Its weights are where its last call left them."""
    assert budget(tiles, 0, 12.0, blocks=1) == (0, 0.0) and budget(tiles, 0, 12.0, blocks=2)[0] >= 8


@pytest.mark.parametrize("D,Dm", [(16384, 131072), (16384, 131072 - 128), (8192, 131072), (32768, 4096)])
def test_a_piece_of_a_huge_weight_keeps_its_offsets_in_32_bits(D, Dm):
    """A thread reads 16 bytes at offsets up to a piece's end and one stride of all workgroups (256 of 8 KB, four times) past it."""
    ws, spans = stack(3, D, Dm)
    seen = {}
    for now in range(12):
        for at, n in pieces(ws, D, Dm, now, 32, 1e13):
            i = next(j for j, (b, size) in enumerate(spans) if b <= at < b + size)
            assert 0 < n <= 2 ** 30 and n % 16 == 0
            assert at - spans[i][0] >= seen.get(i, 0) and at + n <= spans[i][0] + spans[i][1]
            seen[i] = at + n - spans[i][0]
