"""Row statistics that the projections of a folded stack leave in pieces of 64 columns, instead of a launch for them: every tile of the wide contraction that
leaves or reads them (which ones the library takes is checked without a GPU, in test_parts_forms.py)."""
import pytest
import torch

from helpers import announce
from paper_2605_17633_amd import binding as B
from paper_2605_17633_amd import inputs

pytestmark = pytest.mark.gpu
DEV = "cuda"

# width, images, grid, density; the form (1: proj leaves pieces and fc1 reads them, 3: fc2 and qkv too) and the tiles of qkv, proj, fc1, fc2; key and value
# biases folded: without, padding rows are written behind the qkv tiles of every block
CASES = [
    (768, 2, 16, 0.75, 3, (4, 0, 4, 0), True),
    (1024, 6, 16, 0.75, 3, (6, 1, 6, 1), False),
    (768, 11, 16, 0.75, 3, (7, 4, 7, 3), True),
    (768, 8, 28, 0.6, 3, (11, 6, 10, 4), False),       # no padding
    (768, 11, 16, 1.0, 1, (7, 4, 8, 2), False),
    (768, 1, 64, 0.5, 3, (10, 4, 5, 3), False),
    (1024, 3, 32, 1.0, 3, (8, 4, 9, 4), True),
    (1024, 2, 40, 1.0, 3, (10, 4, 11, 4), False),
    (768, 14, 24, 0.75, 3, (8, 6, 8, 6), True),
    (768, 11, 32, 0.1, 1, (-1, 9, 4, 0), True),
]


def device_weights(gen, D, w, Dm=None):
    Dm = Dm or 4 * D
    n = lambda *s, std=0.02, dtype=torch.float32: (torch.randn(*s, generator=gen, device=DEV) * std).to(dtype)
    bf = torch.bfloat16
    # a strong output projection: the rows that fc1 reads then have statistics of their own, not those of the block's input
    return {"ln1_g": 1 + n(D), "ln1_b": n(D), "wqkv": n(3 * D, D, dtype=bf), "bqkv": n(3 * D), "rel_h": n(2 * w - 1, 64, dtype=bf), "rel_w": n(2 * w - 1, 64, dtype=bf),
            "wproj": n(D, D, std=0.1, dtype=bf), "bproj": n(D), "ln2_g": 1 + n(D), "ln2_b": n(D), "w1": n(Dm, D, dtype=bf), "b1": n(Dm),
            "w2": n(D, Dm, dtype=bf), "b2": n(D)}


def close(got, want, start, what):
    """The same block with the statistics of its rows from another order of sums.  A few units of 2^-24 in them move 2^-14 of the hidden values across a bf16
    rounding, by 2^-8 of themselves: 2^-15 of the update in the root mean square.  Where x + update is stored, a shift of d moves a value by its unit
    u = 2^-8 |x| with probability d / u, in the root mean square sqrt(d u) = 2^-11.5 sqrt(|update| |x|); x is at most about 16 updates here: 2^-9.5."""
    err = float((got.double() - want.double()).norm() / (want.double() - start.double()).norm())
    print(what, "error of the update", err)
    assert err < 2.0 ** -9.5, what


@pytest.mark.parametrize("D,images,g,density,form,tiles,kv", CASES)
def test_row_statistics_in_pieces(D, images, g, density, form, tiles, kv):
    check_row_statistics_in_pieces(D, images, g, density, form, tiles, kv, 4 * D)


def check_row_statistics_in_pieces(D, images, g, density, form, tiles, kv, Dm):
    announce("row statistics in pieces", D, images, g, density, form, tiles, kv, Dm)
    gen = torch.Generator(device=DEV).manual_seed(D + images * g)
    n, ws = g * g, 14
    K = B.ssam_keep_count(n, density)
    flags = [False, True, False]
    base = [device_weights(gen, D, g if f else ws, Dm) for f in flags]
    fold = dict(fold_ln1=True, fold_kv_bias=kv)
    wts = [B.pack_block_weights(w, fold_ln2=True, **fold) for w in base]
    structs = [B.block_weights_struct(w) for w in wts]
    cfg_l = B.make_cfg(images, g, D, D // 64, Dm, ws, 32, K, 0.4)
    cfg_g = B.make_cfg(images, g, D, D // 64, Dm, 0, 128, K, 0.4)
    dev = lambda a: torch.from_numpy(a).to(DEV)
    wtab, wsig, gtab = dev(B.ssam_build_window_table(g, ws, 4)), dev(B.ssam_build_perm(ws, ws, 4)[0]), dev(B.ssam_build_perm(g, g, 4)[0])
    x0 = torch.randn(images, n, D, generator=gen, device=DEV).bfloat16()
    scores, keep = torch.empty(images, n, device=DEV), torch.empty(images, K, dtype=torch.int32, device=DEV)
    workspace = torch.full((B.ssam_encoder_workspace_bytes(cfg_l, cfg_g),), 0xff, dtype=torch.uint8, device=DEV)      # NaN wherever nothing was written

    def block(x, s, f=False):
        x = x.clone()
        B.ssam_encoder_block(x, s, cfg_g if f else cfg_l, gtab if f else wtab, gtab if f else wsig, keep)
        return x

    # a stack, whose qkv reads what fc2 and proj left, is the same bits as its blocks one by one, whose qkv reads a launch's
    got = x0.clone()
    B.ssam_encoder_forward(got, structs, flags, cfg_l, cfg_g, wtab, wsig, gtab, gtab, scores, keep, workspace)
    one = x0
    for s, f in zip(structs, flags):
        one = block(one, s, f)
    assert torch.isfinite(got).all() and torch.equal(got, one)

    # proj's pieces in fc1: the block's second half against the routed MLP, which has a launch for them
    nothing = dict(w2=torch.zeros_like(wts[0]["w2"]), b2=torch.zeros_like(wts[0]["b2"]))
    mid = block(x0, B.block_weights_struct({**wts[0], **nothing}))
    want = mid.clone()
    w = wts[0]
    B.ssam_routed_mlp_folded(want, keep, 1e-6, w["w1"], w["fc1_colsum"], w["b1_folded"], w["w2"], w["b2"])
    close(block(x0, structs[0]), want, mid, "fc1")

    # qkv: the block's first half against one whose LN2 is not folded, which takes no pieces at all
    plain = B.pack_block_weights(base[0], **fold)
    close(mid, block(x0, B.block_weights_struct({**plain, **nothing})), x0, "qkv")

    # and what the first comparison would see: the update with the statistics of the rows before proj
    rows = keep[0, :256].long()
    ln = lambda v, of: (v - of.mean(-1, keepdim=True)) / torch.sqrt(of.var(-1, unbiased=False, keepdim=True) + 1e-6) * base[0]["ln2_g"] + base[0]["ln2_b"]
    a, b = mid[0, rows].float(), x0[0, rows].float()
    mlp = lambda t: torch.nn.functional.gelu(t @ base[0]["w1"].float().t() + base[0]["b1"]) @ base[0]["w2"].float().t()
    right, stale = mlp(ln(a, a)), mlp(ln(a, b))
    assert float((stale - right).norm() / right.norm()) > 10 * 2.0 ** -9.5
