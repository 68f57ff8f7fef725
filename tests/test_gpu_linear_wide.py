"""The contraction with one large workgroup per CU (gemm_wide.h): every tile with every epilogue and weight layout at its edges (ragged
rows and columns, the fewest slabs, one more than the ring holds, a row map per batch item), the folded LayerNorm with and
without gather.  test_wide_forms.py asserts that these shapes take these tiles."""
import pytest
import torch

from helpers import announce, assert_close
from paper_2605_17633_amd import binding as B
from test_gpu_linear_small import _check, _operands, test_folded_gather_by_kernel as folded_gather

pytestmark = pytest.mark.gpu
DEV = "cuda"

# (tile, packed, epilogue, M, N, K), tiles in the order of gemm.hip's wide_tiles
CASES = [
    (0, False, 0, 35, 176, 448), (0, False, 0, 95, 88, 512), (0, False, 1, 38, 72, 576), (0, False, 2, 42, 304, 512),
    (0, False, 2, 44, 72, 448), (0, False, 3, 44, 144, 448), (0, False, 3, 50, 80, 512), (0, True, 0, 71, 2944, 512),
    (0, True, 1, 70, 2816, 768), (0, True, 2, 70, 2816, 576), (0, True, 3, 66, 2944, 576), (1, False, 0, 8682, 80, 320),
    (1, False, 0, 8691, 72, 320), (1, False, 1, 8229, 72, 384), (1, False, 1, 8633, 72, 384), (1, False, 2, 8225, 72, 384),
    (1, False, 2, 8326, 72, 448), (1, False, 3, 8428, 72, 320), (1, False, 3, 8883, 72, 384), (1, True, 0, 333, 2816, 448),
    (1, True, 0, 580, 1664, 448), (1, True, 1, 450, 2176, 768), (1, True, 2, 390, 2432, 768), (1, True, 3, 327, 2816, 512),
    (1, True, 3, 335, 2816, 448), (2, False, 0, 4691, 392, 448), (2, False, 0, 6584, 264, 512), (2, False, 1, 6729, 264, 320),
    (2, False, 1, 6774, 264, 320), (2, False, 2, 8281, 136, 1280), (2, False, 3, 6801, 264, 448), (2, False, 3, 6951, 264, 448),
    (2, True, 0, 651, 3072, 512), (2, True, 0, 714, 2816, 448), (2, True, 1, 651, 3072, 448), (2, True, 1, 777, 2560, 448),
    (2, True, 2, 769, 2560, 1280), (2, True, 3, 653, 3072, 448), (2, True, 3, 657, 3072, 448), (3, False, 0, 4978, 264, 576),
    (3, False, 1, 6388, 208, 1280), (3, False, 2, 6382, 200, 1280), (3, False, 3, 6198, 200, 576), (3, True, 0, 504, 2816, 1280),
    (3, True, 1, 491, 2944, 1280), (3, True, 2, 99, 8320, 960), (3, True, 3, 518, 2816, 1280), (4, False, 0, 8319, 200, 320), (4, False, 0, 8325, 200, 384),
    (4, False, 1, 8566, 200, 448), (4, False, 1, 8697, 200, 448), (4, False, 2, 8248, 200, 384), (4, False, 2, 8250, 200, 320),
    (4, False, 3, 8333, 200, 320), (4, False, 3, 8398, 200, 320), (4, True, 0, 712, 2816, 320), (4, True, 0, 782, 2560, 384),
    (4, True, 1, 1414, 2176, 512), (4, True, 2, 1154, 1792, 512), (4, True, 2, 1481, 1408, 512), (4, True, 3, 771, 2560, 320),
    (4, True, 3, 774, 2560, 320), (5, False, 0, 8070, 648, 320), (5, False, 0, 8137, 648, 320), (5, False, 1, 8082, 2200, 384),
    (5, False, 1, 8179, 656, 448), (5, False, 2, 6258, 920, 768), (5, False, 3, 8170, 680, 320), (5, False, 3, 8188, 656, 384),
    (5, True, 0, 1924, 3072, 448), (5, True, 0, 2114, 2816, 384), (5, True, 1, 2137, 2816, 768), (5, True, 2, 1946, 3072, 1280),
    (5, True, 3, 1928, 3072, 384), (5, True, 3, 2129, 2816, 384), (6, False, 0, 8260, 400, 384), (6, False, 0, 8287, 392, 320),
    (6, False, 1, 7179, 520, 320), (6, False, 1, 7287, 520, 320), (6, False, 2, 7249, 520, 320), (6, False, 2, 8206, 456, 384),
    (6, False, 3, 8330, 400, 320), (6, False, 3, 8472, 392, 320), (6, True, 0, 1537, 2560, 384), (6, True, 0, 1547, 2560, 320),
    (6, True, 1, 1537, 2560, 384), (6, True, 1, 2051, 2944, 320), (6, True, 2, 1283, 3072, 384), (6, True, 2, 1558, 2560, 320),
    (6, True, 3, 1417, 2816, 320), (6, True, 3, 1557, 2560, 320), (7, False, 0, 6955, 792, 320), (7, False, 0, 8554, 648, 320),
    (7, False, 1, 6409, 2320, 320), (7, False, 1, 7239, 2072, 384), (7, False, 2, 6404, 2328, 320), (7, False, 2, 8267, 1800, 320),
    (7, False, 3, 6956, 776, 384), (7, False, 3, 8370, 648, 320), (7, True, 0, 8211, 896, 384), (7, True, 0, 8346, 896, 448),
    (7, True, 1, 7172, 2176, 384), (7, True, 1, 7173, 2176, 320), (7, True, 2, 7221, 2176, 320), (7, True, 2, 8193, 1920, 320),
    (7, True, 3, 2188, 2816, 448), (7, True, 3, 8203, 896, 384), (8, False, 0, 7218, 1040, 384), (8, False, 0, 7275, 1032, 320),
    (8, False, 1, 7241, 1032, 320), (8, False, 1, 8346, 912, 320), (8, False, 2, 7170, 1048, 384), (8, False, 2, 8201, 904, 384),
    (8, False, 3, 6550, 1160, 320), (8, False, 3, 8216, 920, 320), (8, True, 0, 3337, 2432, 320), (8, True, 0, 3340, 2432, 384),
    (8, True, 1, 3205, 2560, 320), (8, True, 1, 3339, 2432, 320), (8, True, 2, 3329, 2432, 384), (8, True, 2, 3333, 2432, 384),
    (8, True, 3, 3338, 2432, 320), (8, True, 3, 3356, 2432, 320), (9, False, 0, 5898, 1928, 384), (9, False, 0, 8715, 2696, 320),
    (9, False, 1, 6444, 1736, 384), (9, False, 1, 6472, 1736, 320), (9, False, 2, 6411, 1776, 320), (9, False, 2, 6427, 1744, 320),
    (9, False, 3, 6516, 1736, 320), (9, False, 3, 6533, 1736, 384), (9, True, 0, 6413, 1792, 448), (9, True, 0, 6443, 1792, 448),
    (9, True, 1, 6409, 1792, 512), (9, True, 1, 6443, 1792, 512), (9, True, 2, 6018, 2048, 320), (9, True, 2, 6024, 2048, 320),
    (9, True, 3, 6401, 1792, 512), (9, True, 3, 6411, 1792, 448), (10, False, 0, 8227, 976, 320), (10, False, 0, 8234, 968, 384),
    (10, False, 1, 8206, 968, 320), (10, False, 1, 8206, 984, 320), (10, False, 2, 7221, 1032, 320), (10, False, 2, 8329, 976, 384),
    (10, False, 3, 6930, 1160, 320), (10, False, 3, 6935, 1160, 320), (10, True, 0, 8194, 1024, 320), (10, True, 0, 8198, 1024, 384),
    (10, True, 1, 8263, 1024, 320), (10, True, 1, 8265, 1024, 320), (10, True, 2, 3590, 2304, 320), (10, True, 2, 8194, 1024, 384),
    (10, True, 3, 8201, 1024, 320), (10, True, 3, 8203, 1024, 320), (11, False, 0, 8193, 2904, 448), (11, False, 0, 8227, 1360, 768),
    (11, False, 1, 5050, 2312, 320), (11, False, 1, 7502, 1544, 384), (11, False, 2, 7221, 1544, 320), (11, False, 2, 8302, 1352, 320),
    (11, False, 3, 7688, 3120, 384), (11, False, 3, 8295, 1352, 512), (11, True, 0, 8200, 2944, 448), (11, True, 0, 8206, 2944, 384),
    (11, True, 2, 8241, 2944, 320), (11, True, 2, 8285, 2944, 320), (11, True, 3, 5016, 2432, 1280), (11, True, 1, 1567, 7552, 1792)]
# (tile, M, N, K): qkv with LN1 folded in
FOLDED = [(0, 128, 2304, 576), (1, 384, 2816, 512), (2, 640, 3328, 512), (3, 128, 8448, 768), (4, 640, 3328, 320), (5, 1792, 3328, 384), (6, 5504, 768, 320),
          (7, 1664, 3840, 448), (8, 5504, 1536, 320), (9, 6528, 1792, 448), (10, 8320, 1024, 320), (11, 1408, 8448, 1280)]
# (tile, kept rows, hidden width, width): fc1 with gather and LN2 folded in
MLP = [(0, 131, 1664, 640), (1, 270, 3328, 640), (2, 513, 3712, 512), (3, 385, 3456, 1280), (4, 781, 3840, 512),
       (5, 1734, 3328, 640), (6, 1161, 3328, 384), (7, 6540, 2432, 384), (8, 2326, 3456, 384), (9, 6438, 1792, 512),
       (10, 2314, 3712, 384), (11, 1567, 7552, 1792)]

# (tile, packed, epilogue, M, N, K, elements past the end of a row of A, of W, of C)
STRIDED = [(0, False, 2, 42, 304, 512, 64, 64, 8), (1, False, 2, 8326, 72, 448, 8, 8, 16), (2, False, 0, 6584, 264, 512, 8, 64, 24), (2, True, 2, 769, 2560, 1280, 8, 0, 8),
           (3, False, 0, 4978, 264, 576, 8, 8, 16), (4, False, 3, 8333, 200, 320, 64, 64, 8), (4, True, 0, 782, 2560, 384, 8, 0, 8), (5, True, 2, 1946, 3072, 1280, 8, 0, 16),
           (6, False, 0, 8260, 400, 384, 8, 8, 16), (7, False, 1, 6409, 2320, 320, 8, 8, 8), (10, False, 2, 7221, 1032, 320, 64, 64, 24), (11, True, 0, 8200, 2944, 448, 8, 0, 8)]


@pytest.mark.parametrize("tile,packed,epi,M,N,K,pa,pw,pc", STRIDED)
def test_row_strides(tile, packed, epi, M, N, K, pa, pw, pc):
    """Rows of A, W and C with elements between them, which are not read and not written."""
    announce("wide linear, row strides", tile, packed, epi, M, N, K, pa, pw, pc)
    A, W, b, gen = _operands(M, N, K)
    far = lambda t, pad: torch.cat([t, torch.full((t.shape[0], pad), 7.0, dtype=t.dtype, device=DEV)], 1)[:, :t.shape[1]]
    to = {"row_map": torch.randperm(M, generator=gen, device=DEV).to(torch.int32), "rows_per_batch": M, "map_batch_stride": M, "dst_rows_per_batch": M} if epi >= 2 else {}
    x = torch.randn(M, N, generator=gen, device=DEV).to(torch.bfloat16)
    C = torch.full((M, N + pc), 3.0, dtype=torch.bfloat16, device=DEV)
    C[:, :N] = x
    B.ssam_linear_ld(far(A, pa), B.ssam_pack_weight(W) if packed else far(W, pw), b, C[:, :N], epilogue=epi, w_packed=packed, **to)
    assert bool((C[:, N:] == 3.0).all())
    want = A.double() @ W.double().t() + b.double()
    want = torch.nn.functional.gelu(want) if epi == 1 else want
    if epi >= 2:
        back = to["row_map"].long().argsort()
        want = want[back] + (x.double() if epi == 2 else 0.0)
    err = (C[:, :N].double() - want).abs()
    assert bool((err <= 2.0 ** -8 * want.abs() + 2e-5).all()), float((err / (want.abs() + 1e-2)).max())


@pytest.mark.parametrize("tile,packed,epi,M,N,K", CASES)
def test_every_tile(tile, packed, epi, M, N, K):
    announce("wide linear", tile, packed, epi, M, N, K)
    _check(M, N, K, epi, packed, per_batch=max(1, M // 3 + 1))


@pytest.mark.parametrize("tile,rows,Dm,D", MLP)
def test_folded_gather(tile, rows, Dm, D):
    folded_gather(tile, rows, Dm, D)


@pytest.mark.parametrize("tile,M,N,K", FOLDED)
def test_folded_ln(tile, M, N, K):
    announce("wide folded ln", tile, M, N, K)
    A, W, b, gen = _operands(M, N, K)
    gamma, beta = 1 + 0.1 * torch.randn(K, generator=gen, device=DEV), 0.1 * torch.randn(K, generator=gen, device=DEV)
    stats = B.ssam_ln_stats(A, 1e-6)
    Wf, colsum, bf = B.ssam_fold_ln_weight(W, b, gamma, beta)
    dst = torch.randperm(M, generator=gen, device=DEV).to(torch.int32)
    out = torch.empty(M, N, dtype=torch.bfloat16, device=DEV)
    B.ssam_linear_ln(A, stats, B.ssam_pack_weight(Wf), colsum, bf, out, dst, M, 0, M)
    want = torch.nn.functional.layer_norm(A.double(), (K,), gamma.double(), beta.double(), 1e-6) @ W.double().t() + b.double()
    assert_close(out.float().cpu().numpy()[dst.cpu().numpy()], want.cpu().numpy(), "wide folded ln", tol=1e-2)
