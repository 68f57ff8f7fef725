"""Keep-set and content-aware tables where their kernels change form: 4 / 16 / 64 keys per thread in the selection, ranking
by counting or by sorting for the tables."""
import numpy as np
import pytest
import torch

import oracle
from helpers import announce
from paper_2605_17633_amd import binding as B
from paper_2605_17633_amd import inputs

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("n,K", [(1, 1), (3, 2), (4095, 1000), (4096, 4096), (4097, 1), (16384, 9000), (16385, 16385), (65533, 30000), (65536, 1)])
@pytest.mark.parametrize("kind", ["spread", "ties", "extremes"])
def test_select_sizes(n, K, kind):
    announce("select", n, K, kind)
    rng = np.random.default_rng(n + K)
    if kind == "spread":
        s = rng.normal(size=(2, n))
    elif kind == "ties":                       # a handful of values, zeros of both signs among them
        s = rng.choice([-1.0, -0.0, 0.0, 0.5, 2.0], size=(2, n))
    else:
        s = rng.choice([np.inf, -np.inf, np.nan, 3e38, -3e38, 1e-42, -1e-42, 0.0], size=(2, n))
    s = s.astype(np.float32)
    keep = B.ssam_select_tokens(torch.from_numpy(s).to(DEV), K).cpu().numpy()
    for b in range(2):
        assert np.array_equal(keep[b], oracle.select_tokens(s[b], K))


@pytest.mark.parametrize("Bn,g,ws,levels", [(1, 14, 14, 0), (2, 30, 14, 3), (1, 5, 2, 0), (1, 50, 0, 4), (9, 128, 0, 50),
                                            (1, 6, 2, 0), (3, 12, 6, 2), (2, 90, 2, 3), (1, 230, 8, 5), (20, 70, 14, 0), (40, 70, 14, 7)])
def test_content_tables_forms(Bn, g, ws, levels):
    """levels > 0: only that many different scores, so that most pairs are decided by the cell index.  Windows of 2 x 2 and 64
    cells or more in few and in many groups, on both sides of the point where the tables are sorted instead of counted."""
    announce("content tables", Bn, g, ws, levels)
    rng = np.random.default_rng(g + ws)
    s = rng.integers(0, levels, size=(Bn, g * g)).astype(np.float32) if levels else inputs.lognormal_scores(rng, Bn, g * g)
    if not levels:
        s[0, :3] = [np.nan, -np.inf, -0.0]
    table, sigma = B.ssam_build_content_tables(torch.from_numpy(s).to(DEV), g, ws, 4)
    table, sigma = table.cpu().numpy(), sigma.cpu().numpy()
    w = ws or g
    nws, S = -(-g // w), w * w
    for b in range(Bn):
        for win in range(nws * nws):
            row, col = (win // nws) * w + np.arange(S) // w, (win % nws) * w + np.arange(S) % w
            inside = (row < g) & (col < g)
            v = np.where(inside, s[b, np.where(inside, row * g + col, 0)], -np.inf)
            v = np.where(np.isnan(v), -np.inf, v) + 0.0
            pi = np.lexsort((np.arange(S), -v))
            order = pi.reshape(S // 4, 4).T.reshape(-1)
            assert np.array_equal(sigma[b * nws * nws + win], order), (b, win)
            cell = np.where(inside, row * g + col, -1)[order]
            assert np.array_equal(table[b, win * S:(win + 1) * S], cell), (b, win)


def test_content_tables_of_millions_of_windows():
    """Windows of one cell: the tables name the cells in window order."""
    announce("content tables, one cell a window")
    g = 2900
    s = torch.randn(1, g * g, device=DEV)
    table, sigma = B.ssam_build_content_tables(s, g, 1, 1)
    assert torch.equal(table.reshape(-1), torch.arange(g * g, dtype=torch.int32, device=DEV)) and not sigma.any()


@pytest.mark.parametrize("gh,gw,D", [(1, 1, 8), (4, 4, 768), (5, 3, 520), (3, 18, 1024), (17, 6, 1032), (13, 9, 1544), (2, 31, 2048), (4, 5, 2056)])
def test_scores_in_one_launch(gh, gw, D):
    """Edges of the 4 x 4 tiles, of a wave's loads of a row, and a row too wide for them: the bits of the form with two launches,
    which a batch of more than 28 MB takes, and the sums of 64 bits up to the rounding of D additions in 32."""
    announce("scores", gh, gw, D)
    n = 28_000_000 // (gh * gw * D * 2) + 1
    gen = torch.Generator(device=DEV).manual_seed(gh * gw + D)
    x = torch.randn(1, gh, gw, D, generator=gen, device=DEV).bfloat16()
    got = B.ssam_score_tokens(x)
    two = B.ssam_score_tokens(x.expand(n, -1, -1, -1).contiguous())
    assert torch.equal(got.expand(n, -1), two)
    c = torch.nn.functional.pad(x[0].double().sum(-1), (1, 1, 1, 1))
    at = lambda r, k: c[1 + r:1 + r + gh, 1 + k:1 + k + gw]
    gx = at(-1, 1) - at(-1, -1) + 2 * (at(0, 1) - at(0, -1)) + at(1, 1) - at(1, -1)
    gy = at(1, -1) - at(-1, -1) + 2 * (at(1, 0) - at(-1, 0)) + at(1, 1) - at(-1, 1)
    bound = 12 * 2.0 ** -24 * D * float(x.float().abs().max())           # twelve sums of D terms weigh into a score
    assert float((got[0].double() - torch.sqrt(gx * gx + gy * gy).reshape(-1)).abs().max()) <= bound


@pytest.mark.parametrize("B_,gh,gw,D", [(70000, 1, 2, 8), (65536, 1, 1, 16), (1024, 2, 2, 8), (1025, 2, 2, 8), (1, 262145, 1, 8), (1, 4096, 1, 8), (2, 300000, 1, 16), (3, 9, 6, 768)])
def test_scores_of_many_images_and_tall_grids(B_, gh, gw, D):
    """More images, or more rows of tiles, than a grid's second and third dimension hold, the most that one launch takes, and images that differ."""
    announce("scores", B_, gh, gw, D)
    gen = torch.Generator(device=DEV).manual_seed(B_ + gh)
    x = torch.randn(B_, gh, gw, D, generator=gen, device=DEV).bfloat16()
    got = B.ssam_score_tokens(x)
    c = torch.nn.functional.pad(x.double().sum(-1), (1, 1, 1, 1))
    at = lambda r, k: c[:, 1 + r:1 + r + gh, 1 + k:1 + k + gw]
    gx = at(-1, 1) - at(-1, -1) + 2 * (at(0, 1) - at(0, -1)) + at(1, 1) - at(1, -1)
    gy = at(1, -1) - at(-1, -1) + 2 * (at(1, 0) - at(-1, 0)) + at(1, 1) - at(-1, 1)
    bound = 12 * 2.0 ** -24 * D * float(x.float().abs().max())           # as above
    assert float((got.double() - torch.sqrt(gx * gx + gy * gy).reshape(B_, -1)).abs().max()) <= bound


def test_calls_go_to_the_current_stream():
    """The binding asks for the raw handle of the current device's current stream: the one that torch.cuda.current_stream() wraps."""
    side = torch.cuda.Stream()
    assert (B._stream().value or 0) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert B._stream().value == side.cuda_stream
    assert (B._stream().value or 0) == torch.cuda.current_stream().cuda_stream
