"""The keep-set and the tables that a stack makes in front of its first block: the same as of the calls that make them one by one."""
import pytest
import torch

from helpers import announce
from paper_2605_17633_amd import binding as B
from test_gpu_row_statistics import device_weights

pytestmark = pytest.mark.gpu
DEV = "cuda"


# images, grid, blocks (global or not), layout; the keep-set of up to 4096 and 16384 tokens in the tables' launch, above in its own; no padding at 28 x 28
@pytest.mark.parametrize("images,g,flags,fold,content", [
    (3, 16, [False, True], True, False), (2, 16, [False, True], True, True), (1, 28, [False], False, False), (2, 66, [False, True], False, False),
    (1, 130, [False], False, False), (1, 2, [True], False, False)])
def test_stack_tables(images, g, flags, fold, content):
    announce("stack tables", images, g, flags, fold, content)
    D, ws, n = 256, 14, g * g
    gen = torch.Generator(device=DEV).manual_seed(images * g)
    K = B.ssam_keep_count(n, 0.4)
    wts = [device_weights(gen, D, g if f else ws) for f in flags]
    if fold:
        wts = [B.pack_block_weights(w, fold_ln1=True, fold_kv_bias=True, fold_ln2=True) for w in wts]
    structs = [B.block_weights_struct(w) for w in wts]
    cfg = [B.make_cfg(images, g, D, D // 64, 4 * D, w, m, K, 0.4, content_order=content, stripe=4) for w, m in ((ws, 32), (0, 128))]
    x0 = torch.randn(images, n, D, generator=gen, device=DEV).bfloat16()
    scores = B.ssam_score_tokens(x0.view(images, g, g, D))
    if content:
        wtab, wsig = B.ssam_build_content_tables(scores, g, ws, 4)
        gtab, gsig = B.ssam_build_content_tables(scores, g, 0, 4)
    else:
        dev = lambda a: torch.from_numpy(a).to(DEV)
        wtab, wsig = dev(B.ssam_build_window_table(g, ws, 4)), dev(B.ssam_build_perm(ws, ws, 4)[0])
        gtab = gsig = dev(B.ssam_build_perm(g, g, 4)[0])
    workspace = torch.full((B.ssam_encoder_workspace_bytes(*cfg),), 0xff, dtype=torch.uint8, device=DEV)
    keep = torch.full((images, K), -1, dtype=torch.int32, device=DEV)
    got = x0.clone()
    tables = [t.clone() for t in (wtab, wsig, gtab, gsig)]
    B.ssam_encoder_forward(got, structs, flags, *cfg, *tables, torch.empty_like(scores), keep, workspace)
    assert torch.equal(keep, B.ssam_select_tokens(scores, K))
    want = x0.clone()
    for s, f in zip(structs, flags):
        B.ssam_encoder_block(want, s, cfg[1] if f else cfg[0], gtab if f else wtab, gsig if f else wsig, keep)
    assert torch.isfinite(got).all() and torch.equal(got, want)
