"""The contraction on problems of at most one round of small workgroups (tile chosen by the library): edges of the 32x32, 64x64,
128x64 and 128x128 tiles, one to three slabs of K and ragged ones, every epilogue, both weight layouts, the folded LayerNorm."""
import numpy as np
import pytest
import torch

from helpers import announce, assert_close
from paper_2605_17633_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _operands(M, N, K):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(M + N + K)
    A = torch.randn(M, K, generator=gen, device=DEV).to(torch.bfloat16)
    W = (torch.randn(N, K, generator=gen, device=DEV) / K ** 0.5).to(torch.bfloat16)
    return A, W, torch.randn(N, generator=gen, device=DEV), gen


@pytest.mark.parametrize("epi", [0, 1, 2, 3])
@pytest.mark.parametrize("M,N,K", [(1, 8, 8), (64, 64, 64), (65, 72, 136), (63, 56, 200), (129, 200, 192), (784, 768, 768),
                                   (1640, 776, 328), (1638, 1536, 384), (3001, 1544, 128), (2500, 3064, 136), (2433, 3072, 128),
                                   (31, 128, 64), (33, 256, 128), (313, 768, 1536), (97, 2048, 192)])
@pytest.mark.parametrize("packed", [False, True])
def test_small_problems(M, N, K, epi, packed):
    """Element-wise within one bf16 rounding of the result and the fp32 summation error of a dot product of unit-variance terms."""
    if packed and (N % 128 or K % 64):
        pytest.skip("packed weights are whole blocks")
    announce("small linear", M, N, K, epi, packed)
    A, W, b, gen = _operands(M, N, K)
    ref = A.double() @ W.double().t() + b.double()
    Wx = B.ssam_pack_weight(W) if packed else W
    if epi < 2:
        got = B.ssam_linear_ld(A, Wx, b, epilogue=epi, w_packed=packed)
        want = torch.nn.functional.gelu(ref) if epi else ref
    else:
        rows = M + 5
        dst = torch.randperm(rows, generator=gen, device=DEV)[:M].to(torch.int32)
        if M > 3:
            dst[M // 2] = -1
        x = torch.randn(rows, N, generator=gen, device=DEV).to(torch.bfloat16)
        got = x.clone()
        B.ssam_linear_ld(A, Wx, b, got, epilogue=epi, row_map=dst, rows_per_batch=M, map_batch_stride=0, dst_rows_per_batch=rows, w_packed=packed)
        want = x.double()
        ok = dst >= 0
        to = dst[ok].long()
        want[to] = ref[ok] + want[to] if epi == 2 else ref[ok]
    err = (got.double() - want).abs()
    assert bool((err <= 2.0 ** -8 * want.abs() + 2e-5).all()), float((err / (want.abs() + 1e-2)).max())


@pytest.mark.parametrize("M,N,K", [(128, 256, 64), (256, 768, 768), (2048, 2304, 128), (1024, 3840, 1280)])
def test_small_folded_ln(M, N, K):
    announce("small folded ln", M, N, K)
    A, W, b, gen = _operands(M, N, K)
    gamma, beta = 1 + 0.1 * torch.randn(K, generator=gen, device=DEV), 0.1 * torch.randn(K, generator=gen, device=DEV)
    stats = B.ssam_ln_stats(A, 1e-6)
    Wf, colsum, bf = B.ssam_fold_ln_weight(W, b, gamma, beta)
    dst = torch.randperm(M, generator=gen, device=DEV).to(torch.int32)
    out = torch.empty(M, N, dtype=torch.bfloat16, device=DEV)
    B.ssam_linear_ln(A, stats, B.ssam_pack_weight(Wf), colsum, bf, out, dst, M, 0, M)
    ln = torch.nn.functional.layer_norm(A.double(), (K,), gamma.double(), beta.double(), 1e-6)
    want = ln @ W.double().t() + b.double()
    assert_close(out.float().cpu().numpy()[dst.cpu().numpy()], want.cpu().numpy(), "small folded ln", tol=1e-2)
