"""The contraction on problems of at most one round of small workgroups (kernel chosen by the library): edges of the 32x32, 64x64,
128x64 and 128x128 tiles, one to three slabs of K and ragged ones, every epilogue, both weight layouts, the folded LayerNorm
with and without gather, row maps per batch item."""
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


SHAPES = [(1, 8, 8), (64, 64, 64), (65, 72, 136), (63, 56, 200), (129, 200, 192), (784, 768, 768), (1640, 776, 328), (1638, 1536, 384), (3001, 1544, 128),
          (2500, 3064, 136), (2433, 3072, 128), (31, 128, 64), (33, 256, 128), (313, 768, 1536), (97, 2048, 192)]
PACKED = [s for s in SHAPES if s[1] % 128 == 0 and s[2] % 64 == 0]      # packed weights are whole blocks

# (kernel, packed, epilogues, shapes that take it without a workspace): 16 to 18 the rings of 128x128, 128x64 and 64x64 tiles, 19 the
# direct kernel, with one, two, three and more slabs of K where they take such; test_linear_forms.py asserts that they do
FORMS = [(16, False, (1, 2), [(2500, 776, 72), (2500, 776, 136), (2500, 776, 200)]), (16, False, (0, 3), [(5000, 776, 1032)]),
         (17, False, (0, 1, 2, 3), [(4097, 200, 72), (4097, 200, 136), (4097, 200, 200)]), (18, False, (0, 1, 2, 3), [(1, 72, 56), (63, 72, 136), (65, 136, 200)]),
         (16, True, (1, 2), [(3001, 768, 64), (4097, 768, 128), (4097, 768, 192)]), (17, True, (0, 1, 2, 3), [(4097, 256, 64), (4097, 256, 128), (4097, 256, 192)]),
         (18, True, (0, 1, 2, 3), [(1, 128, 64), (63, 128, 128), (65, 3072, 192)]), (19, True, (0, 1, 2, 3), [(1, 128, 192), (31, 128, 832), (33, 256, 1536), (65, 128, 960)])]
FORM_CASES = [(form, packed, epi, *shape) for form, packed, epis, shapes in FORMS for epi in epis for shape in shapes]
FOLDED = [(16, 1408, 1536, 64), (16, 1408, 2304, 128), (16, 1408, 2304, 192), (17, 1408, 768, 64), (17, 1408, 768, 128), (17, 1408, 768, 192),
          (18, 128, 256, 64), (18, 128, 256, 128), (18, 128, 2304, 192), (19, 128, 256, 192), (19, 128, 256, 832)]
MLP = [(16, 4097, 768, 128), (17, 4097, 256, 128), (18, 65, 3072, 128), (19, 31, 128, 256), (19, 97, 256, 384)]        # kept rows, hidden width, width


def _check(M, N, K, epi, packed, per_batch=None):
    """Element-wise within one bf16 rounding of the result and the fp32 summation error of a dot product of unit-variance terms.
    per_batch: rows of a batch item, each with a row map of its own (the mapped epilogues)."""
    A, W, b, gen = _operands(M, N, K)
    ref = A.double() @ W.double().t() + b.double()
    Wx = B.ssam_pack_weight(W) if packed else W
    if epi < 2:
        got = B.ssam_linear_ld(A, Wx, b, epilogue=epi, w_packed=packed)
        want = torch.nn.functional.gelu(ref) if epi else ref
    else:
        per = per_batch or M
        items, rows = -(-M // per), per + 5
        maps = torch.stack([torch.randperm(rows, generator=gen, device=DEV)[:per] for _ in range(items)]).to(torch.int32)
        if per > 3:
            maps[:, per // 2] = -1
            maps[:, per // 3] = rows                # past the end: dropped as well
        x = torch.randn(items * rows, N, generator=gen, device=DEV).to(torch.bfloat16)
        got = x.clone()
        B.ssam_linear_ld(A, Wx, b, got, epilogue=epi, row_map=maps, rows_per_batch=per, map_batch_stride=per, dst_rows_per_batch=rows, w_packed=packed)
        want = x.double()
        dst = maps.reshape(-1)[:M].long()
        ok = (dst >= 0) & (dst < rows)
        to = (dst + torch.arange(M, device=DEV) // per * rows)[ok]
        want[to] = ref[ok] + want[to] if epi == 2 else ref[ok]
    err = (got.double() - want).abs()
    assert bool((err <= 2.0 ** -8 * want.abs() + 2e-5).all()), float((err / (want.abs() + 1e-2)).max())


@pytest.mark.parametrize("epi", [0, 1, 2, 3])
@pytest.mark.parametrize("packed,M,N,K", [(False, *s) for s in SHAPES] + [(True, *s) for s in PACKED])
def test_small_problems(packed, M, N, K, epi):
    announce("small linear", M, N, K, epi, packed)
    _check(M, N, K, epi, packed)


@pytest.mark.parametrize("form,packed,epi,M,N,K", FORM_CASES)
def test_every_small_kernel(form, packed, epi, M, N, K):
    """Every kernel for small problems with every epilogue it is taken for; mapped ones with a map per batch item."""
    announce("small linear, by kernel", form, packed, epi, M, N, K)
    _check(M, N, K, epi, packed, per_batch=max(1, M // 3 + 1))


@pytest.mark.parametrize("form,rows,Dm,D", MLP)
def test_folded_gather_by_kernel(form, rows, Dm, D):
    """fc1 of the routed MLP with gather and LayerNorm folded in, two images."""
    announce("folded fc1", form, rows, Dm, D)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(rows + Dm)
    images = 1 if rows % 2 else 2
    keep_n, tokens = rows // images, rows // images + 37
    x = torch.randn(images, tokens, D, generator=gen, device=DEV).to(torch.bfloat16)
    keep = torch.stack([torch.randperm(tokens, generator=gen, device=DEV)[:keep_n].sort()[0] for _ in range(images)]).to(torch.int32)
    g, b = 1 + 0.1 * torch.randn(D, generator=gen, device=DEV), 0.1 * torch.randn(D, generator=gen, device=DEV)
    w1, w2 = ((torch.randn(n, k, generator=gen, device=DEV) / k ** 0.5).to(torch.bfloat16) for n, k in ((Dm, D), (D, Dm)))
    b1, b2 = torch.randn(Dm, generator=gen, device=DEV), torch.randn(D, generator=gen, device=DEV)
    wf, colsum, bf = B.ssam_fold_ln_weight(w1, b1, g, b)
    got = B.ssam_routed_mlp_folded(x.clone(), keep, 1e-6, B.ssam_pack_weight(wf), colsum, bf, B.ssam_pack_weight(w2), b2)
    want = torch.zeros(images, tokens, D, dtype=torch.float64, device=DEV)
    for i in range(images):
        k = keep[i].long()
        h = torch.nn.functional.layer_norm(x[i, k].double(), (D,), g.double(), b.double(), 1e-6) @ w1.double().t() + b1.double()
        want[i, k] = torch.nn.functional.gelu(h) @ w2.double().t() + b2.double()
    x, got = x.double(), got.double()
    assert_close((got - x).cpu().numpy(), want.cpu().numpy(), f"folded fc1 {rows} x {Dm} x {D}", stored=((x + want).cpu().numpy(),))


@pytest.mark.parametrize("M,N,K", [(256, 768, 768), (2048, 2304, 128), (1024, 3840, 1280)] + [f[1:] for f in FOLDED])
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
