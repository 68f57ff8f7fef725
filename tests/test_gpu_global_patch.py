"""Global attention on power-of-two grids in the position-only order (pipelined path): the shortest and longest lists of key
blocks, every head size, and logits that grow along the scan order, so that the exponent reference moves again and again
while probabilities are still waiting for their product."""
import numpy as np
import pytest

import oracle
from helpers import announce, assert_close
from paper_2605_17633_amd import binding as B
from paper_2605_17633_amd import inputs
from test_gpu_block import dev_bf16, dev_i32, run_attention_case, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,d,r", [(16, 2, 16, 0.3), (16, 1, 64, 0.6), (32, 3, 16, 0.1), (32, 1, 80, 0.1), (32, 1, 32, 1.0),
                                     (32, 9, 64, 0.5), (64, 1, 80, 0.02), (128, 1, 16, 0.01), (128, 1, 80, 0.01)])
def test_block_lists(w, h, d, r):
    announce("global patch", w, h, d, r)
    got, ref = run_attention_case(1, w, h, d, 128, r)
    assert_close(got, ref, f"global attention w={w} d={d} r={r}")


@pytest.mark.parametrize("w,h,d,r", [(17, 1, 80, 0.5), (31, 1, 64, 0.2), (33, 2, 80, 0.3), (63, 1, 16, 0.1), (63, 1, 80, 0.02), (65, 1, 64, 0.05),
                                     (72, 1, 80, 0.03), (127, 1, 16, 0.01)])
def test_any_grid(w, h, d, r):
    """Sides around 32 and 64, where the bias table changes from 32 to 64 entries and to look-ups, ragged last tiles."""
    announce("global general", w, h, d, r)
    got, ref = run_attention_case(1, w, h, d, 128, r, G=1)
    assert_close(got, ref, f"global attention w={w} d={d} r={r}")


@pytest.mark.parametrize("d", [16, 32, 64, 80])
@pytest.mark.parametrize("grow", [40.0, -40.0])
def test_growing_logits(d, grow):
    announce("global patch, growing logits", d, grow)
    w, h, r = 32, 2, 0.5
    S, rng = w * w, np.random.default_rng(d)
    sigma, _ = oracle.grid_sigma(w, 4)
    ramp = np.linspace(0.0, 1.0, S) if grow > 0 else np.linspace(1.0, 0.0, S)
    q = np.abs(rng.normal(size=(S, h, d))) * 0.3 + 0.7
    k = rng.normal(size=(S, h, d)) * 0.05 + (abs(grow) / np.sqrt(d)) * ramp[:, None, None]     # logits 0 .. about 40
    v = rng.normal(size=(S, h, d))
    scan = inputs.bf16_round(np.stack([q, k, v], 1).astype(np.float32))                         # [S,3,h,d], scan order
    rel = [inputs.bf16_round(rng.normal(0, 0.1, size=(2 * w - 1, d)).astype(np.float32)) for _ in range(2)]
    got = to_np(B.ssam_sparse_attention(dev_bf16(scan[None]), dev_bf16(rel[0]), dev_bf16(rel[1]), dev_i32(B.ssam_build_perm(w, w, 4)[0]),
                                        w, 128, r)).reshape(S, h, d)
    spatial = np.empty_like(scan)
    spatial[sigma] = scan
    o = oracle.attention(*(np.ascontiguousarray(spatial[:, i].transpose(1, 0, 2)) for i in range(3)), *rel, w, 4, 128, r)
    assert_close(got, o.transpose(1, 0, 2)[sigma], f"growing logits d={d}")


@pytest.mark.parametrize("w,d,order,scale", [(20, 64, "row", 1e-3), (31, 16, "row", 1e-5), (32, 80, "row", 1e-3), (50, 64, "row", 0.125), (50, 80, "position", 1e-3),
                                             (64, 32, "row", 1e-3), (64, 80, "row", 1e-5), (72, 64, "position", 1e-3), (72, 80, "row", 1e-5),
                                             (16, 64, "position", 0.125), (32, 16, "position", 1e-5), (64, 80, "position", 1e-3), (64, 32, "position", 1e-3)])
def test_bias_past_fp16(w, d, order, scale):
    """Bias / scale, what the kernel's tables hold, past the range of fp16: a bias of -120 at scales of 1e-3 and 1e-5, of -16384 at
    1/8.  The keys concerned get no weight (exp(-120) of what the others have at most), the query's other keys what they
    would have without.  Some queries meet nothing else in their first 64 keys."""
    announce("bias past fp16", w, d, order, scale)
    S, rng, r = w * w, np.random.default_rng(w + d), 0.4
    sigma = np.arange(S, dtype=np.int32) if order == "row" else np.ascontiguousarray(B.ssam_build_perm(w, w, 4 if w % 2 == 0 else 1)[0])
    qkv = rng.normal(size=(1, S, 3, 1, d)).astype(np.float32)                                   # scan order
    qkv[:, :, 0, :, 0] = 4.0
    qkv = inputs.bf16_round(qkv)
    rel = [inputs.bf16_round(rng.normal(0, 0.02, size=(2 * w - 1, d)).astype(np.float32)) for _ in range(2)]
    far = np.r_[w + 2, w - 1 + w // 2:2 * w - 1]                                              # three rows, and half the grid or more, above the query
    rel[0][far], rel[0][far, 0] = 0.0, -30.0 if scale < 0.1 else -4096.0
    got = to_np(B.ssam_sparse_attention(dev_bf16(qkv), dev_bf16(rel[0]), dev_bf16(rel[1]), dev_i32(sigma), w, 128, r, scale=scale))[0]
    q, k, v = (qkv[0, :, i, 0].astype(np.float64) for i in range(3))
    row, col = sigma // w, sigma % w
    logit = scale * (q @ k.T)
    for t, c in zip(rel, (row, col)):
        logit += np.take_along_axis(q @ t.T.astype(np.float64), c[:, None] - c[None, :] + w - 1, axis=1)
    tile = np.arange(S) // 128
    logit[~((tile[None, :] < int(r * (tile[-1] + 1) + 1e-6)) | (tile[None, :] == tile[:, None]))] = -np.inf
    p = np.exp(logit - logit.max(1, keepdims=True))
    assert_close(got, p @ v / p.sum(1, keepdims=True), f"bias past fp16 w={w} d={d} {order} scale={scale}")


def exact_global(qkv, rel, sigma, w, r):
    """Attention of one group over tiles of 128, in 64 bits, for any table of cells."""
    S, (_, _, nh, d) = w * w, qkv.shape
    tile, row, col = np.arange(S) // 128, sigma // w, sigma % w
    off = ~((tile[None, :] < int(r * (tile[-1] + 1) + 1e-6)) | (tile[None, :] == tile[:, None]))
    want = np.empty((S, nh, d))
    for h in range(nh):
        q, k, v = (qkv[:, i, h].astype(np.float64) for i in range(3))
        logit = d ** -0.5 * (q @ k.T)
        for t, c in zip(rel, (row, col)):
            logit += np.take_along_axis(q @ t.T.astype(np.float64), c[:, None] - c[None, :] + w - 1, axis=1)
        logit[off] = -np.inf
        p = np.exp(logit - logit.max(1, keepdims=True))
        want[:, h] = p @ v / p.sum(1, keepdims=True)
    return want


@pytest.mark.parametrize("w,d,r,shared", [(1, 16, 1.0, True), (2, 80, 0.5, False), (3, 64, 0.4, False), (8, 80, 1.0, False), (11, 32, 0.4, False), (12, 64, 0.4, False),
                                          (16, 80, 0.5, True), (23, 16, 1.0, False), (32, 64, 0.3, False), (32, 80, 1.0, True), (33, 32, 0.2, False),
                                          (45, 80, 1.0, False), (64, 16, 0.1, True), (64, 64, 0.2, False), (64, 80, 0.1, True)])
def test_any_order(w, d, r, shared):
    """Two groups with tables of their own (or one table, which on a power-of-two grid goes through the check for patches first): a random order,
    and entries that repeat and begin and end at the corners.  Less than a tile, ragged last blocks, blocks past the end, and sides where the
    tables change from 32 to 64 entries.  The bound: a bf16 rounding is 2^-8 / sqrt(3) * sqrt(0.54) = 1.66e-3 of a value in the root mean square (over
    mantissas spread evenly in their logarithm), the probabilities' and the output's together 2.34e-3 where no key dominates.  The tables' fp16 adds
    2^-11 / sqrt(3) * b of a probability for a bias b, 0.1 * sqrt(80) = 0.9 and up to three times that where it gives a key its weight: both
    tables' together up to 1.0e-3.  2.55e-3 in all."""
    announce("global, any order", w, d, r, shared)
    S, rng = w * w, np.random.default_rng(100 * w + d)
    sigma = np.stack([rng.permutation(S) for _ in range(2)]).astype(np.int32)
    sigma[0, :1], sigma[0, -1:] = S - 1, 0
    if S > 8:
        sigma[0, 3:6] = sigma[0, 2]
    if shared:
        sigma[1] = sigma[0]
    qkv = inputs.bf16_round(rng.normal(size=(2, S, 3, 2, d)).astype(np.float32))
    rel = [inputs.bf16_round(rng.normal(0, 0.1, size=(2 * w - 1, d)).astype(np.float32)) for _ in range(2)]
    got = to_np(B.ssam_sparse_attention(dev_bf16(qkv), dev_bf16(rel[0]), dev_bf16(rel[1]), dev_i32(sigma[0] if shared else sigma), w, 128, r)).reshape(2, S, 2, d)
    want = np.stack([exact_global(qkv[g], rel, sigma[g], w, r) for g in range(2)])
    err = np.linalg.norm(got - want) / np.linalg.norm(want)
    print("error", err)
    assert err < 2.6e-3


@pytest.mark.parametrize("w,d,r,shared", [(4, 64, 1.0, True), (5, 16, 1.0, False), (7, 80, 1.0, False), (8, 32, 1.0, True), (12, 80, 1.0, False), (12, 64, 0.5, True), (20, 64, 1.0, True),
                                          (20, 80, 0.3, False), (23, 32, 1.0, False), (28, 16, 1.0, True), (28, 80, 0.4, False), (36, 64, 0.2, False), (36, 80, 1.0, True), (60, 16, 0.1, False), (60, 32, 0.1, True),
                                          (44, 80, 0.1, False)])
def test_short_last_tile(w, d, r, shared):
    """At most 64 keys in the last tile: its two blocks are the only ones, or come behind whole tiles, one or many."""
    test_any_order(w, d, r, shared)


@pytest.mark.parametrize("d", [16, 32, 64, 80])
@pytest.mark.parametrize("w,r,order", [(32, 0.2, "position"), (64, 0.4, "position"), (28, 0.4, "position"), (50, 0.5, "row")])
def test_error_where_one_key_dominates(w, r, order, d):
    """Rounding to bf16 alone: the output's (2^-9 of a value at most, 1.2e-3 of it in the root mean square) and the probabilities',
    which is the same for each key and cancels as far as one dominates: together 1.2e-3 * sqrt(2) = 1.7e-3 and some.  A largest
    probability that is not exactly 1, over a sum of unrounded ones, gives 2.35e-3."""
    announce("peaky softmax", w, r, order, d)
    S, rng = w * w, np.random.default_rng(w + d)
    sigma = np.arange(S, dtype=np.int32) if order == "row" else np.ascontiguousarray(B.ssam_build_perm(w, w, 4)[0])
    qkv = rng.normal(size=(1, S, 3, 2, d)).astype(np.float32)
    qkv[:, :, :2] *= 2.0
    qkv = inputs.bf16_round(qkv)
    rel = [inputs.bf16_round(rng.normal(0, 0.1, size=(2 * w - 1, d)).astype(np.float32)) for _ in range(2)]
    got = to_np(B.ssam_sparse_attention(dev_bf16(qkv), dev_bf16(rel[0]), dev_bf16(rel[1]), dev_i32(sigma), w, 128, r))[0].reshape(S, 2, d)
    tile, row, col = np.arange(S) // 128, sigma // w, sigma % w
    off = ~((tile[None, :] < int(r * (tile[-1] + 1) + 1e-6)) | (tile[None, :] == tile[:, None]))
    want = np.empty((S, 2, d))
    for h in range(2):
        q, k, v = (qkv[0, :, i, h].astype(np.float64) for i in range(3))
        logit = d ** -0.5 * (q @ k.T)
        for t, c in zip(rel, (row, col)):
            logit += np.take_along_axis(q @ t.T.astype(np.float64), c[:, None] - c[None, :] + w - 1, axis=1)
        logit[off] = -np.inf
        p = np.exp(logit - logit.max(1, keepdims=True))
        want[:, h] = p @ v / p.sum(1, keepdims=True)
    err = np.linalg.norm(got - want) / np.linalg.norm(want)
    print("error", err)
    assert err < 2.0e-3
