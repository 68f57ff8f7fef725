"""Window attention at the edges of its kernels: every window side, a last tile of one to thirty-two keys, one to seven active blocks,
both kernels on either side of the line between them, biases past the range of fp16, any softmax scale, rows far apart."""
import ctypes as C

import numpy as np
import pytest
import torch

from helpers import announce, assert_close, to_np
from paper_2605_17633_amd import binding as B
from paper_2605_17633_amd import inputs
from test_gpu_block import dev_bf16, dev_i32, run_attention_case

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("d", [16, 32, 64, 80])
@pytest.mark.parametrize("groups,w,h,r", [(1, 1, 3, 1.0), (9, 2, 1, 0.5), (2, 5, 2, 0.4), (3, 6, 1, 0.9), (1, 8, 5, 0.6), (2, 9, 1, 0.34), (1, 11, 2, 1.0),
                                          (2, 12, 1, 0.2), (1, 13, 3, 0.5), (1, 14, 1, 0.1), (5, 14, 3, 0.75), (3, 14, 2, 1.0)])
def test_window_sides(groups, w, h, r, d):
    announce("window attention", groups, w, h, r, d)
    got, ref = run_attention_case(groups, w, h, d, 32, r, G=4 if w % 2 == 0 else 1, rel_scale=0.3)
    assert_close(got, ref, f"window {w} x {w} d={d} r={r}")


def _case(groups, w, h, d, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    qkv = (torch.randn(groups, w * w, 3, h, d, generator=gen, device=DEV) * 0.7).bfloat16()
    rel = [(torch.randn(2 * w - 1, d, generator=gen, device=DEV) * 0.1).bfloat16() for _ in range(2)]
    return qkv, rel, dev_i32(B.ssam_build_perm(w, w, 4 if w % 2 == 0 else 1)[0])


@pytest.mark.parametrize("w", [8, 14])
@pytest.mark.parametrize("r", [0.2, 0.4, 1.0])
@pytest.mark.parametrize("groups,own", [(26, False), (120, False), (120, True)])
def test_both_kernels_of_d80(groups, own, r, w):
    """26 and 120 windows of 16 heads loop over persistent workgroups, five of them run a wave to a tile: the same bits, with an
    order for all windows and with one for each."""
    announce("d = 80", groups, own, r, w)
    qkv, rel, sigma = _case(groups, w, 16, 80, groups)
    if own:
        sigma = torch.stack([torch.randperm(w * w, generator=torch.Generator().manual_seed(g)) for g in range(groups)]).int().to(DEV)
    many = B.ssam_sparse_attention(qkv, *rel, sigma, w, 32, r)
    for g in range(0, groups, 5):
        few = B.ssam_sparse_attention(qkv[g:g + 5].contiguous(), *rel, sigma[g:g + 5].contiguous() if own else sigma, w, 32, r)
        assert torch.equal(few, many[g:g + 5]), g


@pytest.mark.parametrize("own", [False, True])
@pytest.mark.parametrize("d,w,r,groups", [(64, 10, 0.4, 132), (64, 11, 0.75, 132), (80, 9, 0.4, 66), (80, 10, 1.0, 260), (80, 12, 0.2, 196)])
def test_both_kernels_by_side(d, w, r, groups, own):
    """Windows of 16 heads, just enough for the persistent workgroups, and five of them a wave to a tile: the same bits."""
    announce("window, both kernels", d, w, r, groups, own)
    qkv, rel, sigma = _case(groups, w, 16, d, groups)
    if own:
        sigma = torch.stack([torch.randperm(w * w, generator=torch.Generator().manual_seed(g)) for g in range(groups)]).int().to(DEV)
    many = B.ssam_sparse_attention(qkv, *rel, sigma, w, 32, r)
    for g in range(0, groups - 4, 41):
        few = B.ssam_sparse_attention(qkv[g:g + 5].contiguous(), *rel, sigma[g:g + 5].contiguous() if own else sigma, w, 32, r)
        assert torch.equal(few, many[g:g + 5]), g


@pytest.mark.parametrize("d", [64, 80])
def test_rows_far_apart(d):
    """A window whose rows span more than 32-bit byte offsets: the bits of the compact call."""
    announce("rows far apart", d)
    w, h, S, stride = 14, 2, 196, 11_100_000
    qkv, rel, sigma = _case(1, w, h, d, 5)
    want = B.ssam_sparse_attention(qkv, *rel, sigma, w, 32, 0.6)
    far = torch.empty(S, stride, dtype=torch.bfloat16, device=DEV)
    far[:, :3 * h * d] = qkv.reshape(S, 3 * h * d)
    got = torch.empty_like(want)
    ptr = [C.c_void_p(far.data_ptr() + 2 * i * h * d) for i in range(3)]
    rc = B.lib().ssam_sparse_attention(*ptr, C.c_long(stride), C.c_void_p(rel[0].data_ptr()), C.c_void_p(rel[1].data_ptr()), C.c_void_p(sigma.data_ptr()),
                                       C.c_long(0), C.c_void_p(got.data_ptr()), None, C.c_int(1), C.c_int(S), C.c_int(w), C.c_int(h), C.c_int(d), C.c_int(32),
                                       C.c_double(0.6), C.c_float(d ** -0.5), C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    assert torch.equal(got, want)


@pytest.mark.parametrize("groups", [1, 500])
@pytest.mark.parametrize("d", [16, 64, 80])
@pytest.mark.parametrize("scale,bias", [(1e-3, -120.0), (1e-3, 150.0), (1e-4, 1000.0), (0.125, -16384.0), (0.125, 3000.0)])
def test_bias_past_fp16(scale, bias, d, groups):
    """Bias / scale past the range of fp16, up and down, against 64 bits: the tables carry a power of two, so that logits up to the
    range of fp16 in units of log 2 keep their values and what lies below takes no weight."""
    announce("window bias past fp16", scale, bias, d, groups)
    w, S, r, rng = 14, 196, 1.0, np.random.default_rng(d)
    sigma = np.ascontiguousarray(B.ssam_build_perm(w, w, 4)[0])
    qkv = rng.normal(size=(1, S, 3, 1, d)).astype(np.float32)
    qkv[:, :, 0, :, 0] = 4.0
    qkv = inputs.bf16_round(qkv)
    rel = [inputs.bf16_round(rng.normal(0, 0.02, size=(2 * w - 1, d)).astype(np.float32)) for _ in range(2)]
    rel[0][w + 2:], rel[0][w + 2:, 0] = 0.0, bias / 4
    got = to_np(B.ssam_sparse_attention(dev_bf16(np.repeat(qkv, groups, 0)), dev_bf16(rel[0]), dev_bf16(rel[1]), dev_i32(sigma), w, 32, r, scale=scale))
    q, k, v = (qkv[0, :, i, 0].astype(np.float64) for i in range(3))
    logit = scale * (q @ k.T)
    for t, c in zip(rel, (sigma // w, sigma % w)):
        logit += np.take_along_axis(q @ t.T.astype(np.float64), c[:, None] - c[None, :] + w - 1, axis=1)
    p = np.exp(logit - logit.max(1, keepdims=True))
    assert np.array_equal(got, np.repeat(got[:1], groups, 0))
    assert_close(got[0], p @ v / p.sum(1, keepdims=True), f"window bias past fp16 d={d} scale={scale} bias={bias}")


def _one_head(groups, d, seed, scale, mag):
    """A window of 14 x 14 whose queries are of size `mag`, with biases of 18 to 30 on the keys some rows above a query, against 64 bits."""
    w, S, rng = 14, 196, np.random.default_rng(seed)
    sigma = np.ascontiguousarray(B.ssam_build_perm(w, w, 4)[0])
    qkv = rng.normal(size=(1, S, 3, 1, d)).astype(np.float32)
    qkv[:, :, 0, :, 0] = 4.0
    qkv[:, :, 0] *= mag
    qkv = inputs.bf16_round(qkv)
    rel = [rng.normal(0, 0.2, size=(2 * w - 1, d)).astype(np.float32) for _ in range(2)]
    rel[0][w + 2:], rel[0][w + 2:, 0] = 0.0, (18 + 4 * (np.arange(w - 3) % 4)) / 4
    rel = [inputs.bf16_round((t / np.float32(mag)).astype(np.float32)) for t in rel]
    got = B.ssam_sparse_attention(dev_bf16(np.repeat(qkv, groups, 0)), dev_bf16(rel[0]), dev_bf16(rel[1]), dev_i32(sigma), w, 32, 1.0, scale=scale)
    q, k, v = (qkv[0, :, i, 0].astype(np.float64) for i in range(3))
    logit = float(np.float32(scale)) * (q @ k.T)
    for t, c in zip(rel, (sigma // w, sigma % w)):
        logit += np.take_along_axis(q @ t.T.astype(np.float64), c[:, None] - c[None, :] + w - 1, axis=1)
    p = np.exp(logit - logit.max(1, keepdims=True))
    return got, p @ v / p.sum(1, keepdims=True)


@pytest.mark.parametrize("groups", [1, 500])
@pytest.mark.parametrize("d", [16, 64, 80])
@pytest.mark.parametrize("scale", [1e-44, 1e-30, 1e-8, 1.9e-5, 2.3e-5, 0.6, 300.0, 400.0, 5e6, 7e6, 1e30])
def test_any_scale(scale, d, groups):
    """Queries of the size that gives logits of a few units at this scale: what the scale splits into (ones of fp16, the queries) is exact."""
    announce("window scale", scale, d, groups)
    mag = 2.0 ** np.clip(np.round(-np.log2(scale * d ** 0.5)), -116, 100)
    got, want = _one_head(groups, d, 7, scale, mag)
    assert bool((got == got[:1]).all())
    assert_close(to_np(got)[0], want, f"window scale {scale} d={d}")


@pytest.mark.parametrize("d", [16, 64, 80])
@pytest.mark.parametrize("scale", [1e-44, 3e-39, 1e-30, 1e-8, 1e-6])
def test_small_scale_keeps_the_bias(scale, d):
    """Queries of size 1: the logits are the biases."""
    announce("window bias alone", scale, d)
    got, want = _one_head(3, d, 8, scale, 1.0)
    assert_close(to_np(got)[0], want, f"window bias alone, scale {scale} d={d}")


@pytest.mark.parametrize("groups", [1, 500])
@pytest.mark.parametrize("d", [16, 64, 80])
@pytest.mark.parametrize("e", [5, 16, 40, 100])
def test_powers_of_two(e, d, groups):
    """Queries 2^e times larger, tables and scale 2^e times smaller: the same bits."""
    announce("window, powers of two", e, d, groups)
    qkv, rel, sigma = _case(groups, 14, 1, d, 3)
    want = B.ssam_sparse_attention(qkv, *rel, sigma, 14, 32, 0.6, scale=d ** -0.5)
    far = qkv.clone()
    far[:, :, 0] *= 2.0 ** e
    got = B.ssam_sparse_attention(far, *[t * 2.0 ** -e for t in rel], sigma, 14, 32, 0.6, scale=d ** -0.5 * 2.0 ** -e)
    assert torch.equal(got, want)
