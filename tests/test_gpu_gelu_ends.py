"""The GELU epilogue at the ends of its range, through every family of contraction kernels: infinities, NaN, the largest and smallest
finite pre-activations.  With A = 0 the pre-activation is the bias."""
import math

import pytest
import torch

from helpers import announce
from paper_2605_17633_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda"
INF, NAN = math.inf, math.nan
PRE = [INF, -INF, NAN, 0.0, -0.0, 3.4e38, -3.4e38, 1e30, -1e30, 100.0, -100.0, 16.5, -16.5, 15.5, -15.5, 6.0, -6.0, 3.0, -3.0, 0.7, -0.7, 1e-3, -1e-3, 1e-30, -1e-30]

# (packed, M, N, K, tile, workspace): forced large tiles, a K-split and its reduce, rings of 64x64, 128x64 and 128x128, the direct kernel, the wide
# kernel with one chain over K and with two
CASES = [(False, 300, 264, 64, t, False) for t in (1, 2, 3, 4)] + [(True, 300, 256, 64, t, False) for t in (1, 3, 4)] + [
    (False, 42, 1560, 5120, 0, True), (True, 31, 1280, 5120, 0, True), (False, 63, 72, 136, 0, False), (False, 4097, 200, 136, 0, False),
    (False, 2500, 776, 136, 0, False), (True, 65, 3072, 192, 0, False), (True, 4097, 256, 128, 0, False), (True, 4097, 768, 128, 0, False), (True, 31, 128, 832, 0, False),
    (False, 38, 72, 576, 0, False), (False, 8566, 200, 448, 0, False), (True, 70, 2816, 768, 0, False), (True, 1414, 2176, 512, 0, False)]


@pytest.mark.parametrize("packed,M,N,K,tile,split", CASES)
def test_linear(packed, M, N, K, tile, split):
    """erfc is held to 1.5e-7, half of that times |t| up to 6 where it matters, and the result is rounded to bf16 once."""
    announce("gelu ends", packed, M, N, K, tile, split)
    b = torch.tensor(PRE, device=DEV).repeat(-(-N // len(PRE)))[:N].contiguous()
    W = torch.zeros(N, K, dtype=torch.bfloat16, device=DEV)
    ws = torch.empty(B.ssam_linear_workspace_bytes(), dtype=torch.uint8, device=DEV) if split else None
    got = B.ssam_linear_ld(torch.zeros(M, K, dtype=torch.bfloat16, device=DEV), B.ssam_pack_weight(W) if packed else W, b, epilogue=1, w_packed=packed, tile=tile,
                           workspace=ws).double()
    assert bool((got.view(torch.int64) == got[:1].view(torch.int64)).all())
    got, want = got[0], torch.nn.functional.gelu(b.double())
    want[b == -INF] = 0.0                     # its limit; the formula gives -inf * 0
    nan, big = b.isnan(), b.abs() > 3.39e38           # the largest bf16 is 3.39e38
    assert bool(got[nan].isnan().all()) and not bool(got[~nan].isnan().any())
    assert bool((got[b == INF] == INF).all()) and bool((got[b == -INF] == 0).all()) and bool((got[big & (b < 0)] == 0).all())
    ok = ~(nan | big)
    assert bool(((got - want)[ok].abs() <= 2.0 ** -8 * want[ok].abs() + 5e-7).all()), ((got - want)[ok].abs().max())


@pytest.mark.parametrize("form", ["row-major", "packed", "folded"])
@pytest.mark.parametrize("rows,Dm,D", [(31, 128, 256), (97, 256, 384), (131, 1664, 640), (781, 3840, 512), (4097, 256, 128)])
def test_routed_mlp(rows, Dm, D, form):
    """Hidden activations of +inf, -inf and NaN through fc2 with positive weights: inf, the bias alone, NaN."""
    announce("gelu ends, routed mlp", rows, Dm, D, form)
    x = torch.randn(1, rows + 9, D, device=DEV).to(torch.bfloat16)
    keep = torch.arange(4, rows + 4, dtype=torch.int32, device=DEV)[None].contiguous()
    w1, w2 = torch.zeros(Dm, D, dtype=torch.bfloat16, device=DEV), torch.ones(D, Dm, dtype=torch.bfloat16, device=DEV)
    one, zero = torch.ones(D, device=DEV), torch.zeros(D, device=DEV)
    for pre, add in ((INF, INF), (-INF, 1.0), (NAN, NAN)):
        b1, b2 = torch.full((Dm,), pre, device=DEV), torch.ones(D, device=DEV)
        if form == "folded":
            wf, colsum, _ = B.ssam_fold_ln_weight(w1, torch.zeros(Dm, device=DEV), one, zero)
            got = B.ssam_routed_mlp_folded(x.clone(), keep, 1e-6, B.ssam_pack_weight(wf), colsum, b1, B.ssam_pack_weight(w2), b2)
        elif form == "packed":
            got = B.ssam_routed_mlp_packed(x.clone(), keep, one, zero, 1e-6, B.ssam_pack_weight(w1), b1, B.ssam_pack_weight(w2), b2)
        else:
            got = B.ssam_routed_mlp(x.clone(), keep, one, zero, 1e-6, w1, b1, w2, b2)
        want = x.clone()
        want[:, 4:rows + 4] = (x[:, 4:rows + 4].float() + add).to(torch.bfloat16)
        assert torch.equal(got.nan_to_num(nan=7e4), want.nan_to_num(nan=7e4)), (pre, form)
