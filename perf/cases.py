"""The work that the library's speed is judged on: calls of its public entry points, as a user's program makes them.

A case is a dict of plain values.  Its ``path`` says which part of the library it stands for:

  encoder    the whole stack of SAM ViT blocks on a batch of token grids (``ssam_encoder_forward``), with ``ends`` also
             the patch embedding in front and the neck behind: pixels in, embedding out
  block      one encoder block (``ssam_encoder_block``), windowed (``window`` = 14) or global (``window`` = 0)
  attention  Stripe-Sort attention alone on a packed q/k/v tensor, windows of a grid or whole grids
  mlp        the Residual-Consistency MLP alone: keep-set given, gather, LayerNorm, fc1, GELU, fc2, scatter-add
  select     what an image costs before its first block: token scores, keep-set and, with the content-aware order, the
             scan tables of its windows and of its grid

``weights`` is how the program laid its weights out at load time: ``rows`` (row-major, the default of the library),
``packed`` (MFMA fragment order) or ``folded`` (packed, with the LayerNorms and the key and value biases folded into the
contractions wherever the library has the folded form for the shape).  ``order`` is the scan order of attention:
``position`` (tables made once per grid size) or ``content`` (tables made from every image's scores).  ``density`` is the
attention density and the keep ratio of the MLP.

Weights and tokens follow the library's input recipe (``paper_2605_17633_amd/inputs.py``), drawn on the GPU: Linear
weights, biases and rel-pos tables N(0, 0.02), LayerNorm gains around 1, tokens of a few low-frequency waves and noise.
"""
import math

import torch

from paper_2605_17633_amd import binding as B
from paper_2605_17633_amd import inputs

DEV = "cuda"
STRIPE = 4            # G of the stripe interleave
WINDOW = 14           # SAM's window side
PATCH, NECK = 16, 256  # pixels per token side; channels of the embedding
BF = torch.bfloat16


def listed():
    return [
        # before the first block of a single image, content-aware order: the smallest call, bound by latency and launches
        dict(name="select_b1", path="select", batch=1, grid=64, width=768, density=0.4, order="content"),
        # one windowed block on a small grid, batch 1: the unit that a program tries first
        dict(name="block_vit_b_28x28_b1", path="block", model="vit_b", batch=1, grid=28, window=WINDOW, density=0.4, weights="packed"),
        # interactive use: one 1024x1024 image through the base and the large encoder
        dict(name="encoder_vit_b_b1", path="encoder", model="vit_b", batch=1, grid=64, density=0.4, order="position", weights="folded", ends=False),
        dict(name="encoder_vit_l_b1", path="encoder", model="vit_l", batch=1, grid=64, density=0.3, order="position", weights="folded", ends=False),
        # pixels in, embedding out on images that are not 1024x1024 (grid 50: ragged rows, tiles and windows), by a program
        # that hands its weights over as they are
        dict(name="image_vit_b_800px_b2", path="encoder", model="vit_b", batch=2, grid=50, density=0.5, order="position", weights="rows", ends=True),
        # throughput: the huge encoder on a batch, and a small batch of it with the content-aware order
        dict(name="encoder_vit_h_b8", path="encoder", model="vit_h", batch=8, grid=64, density=0.4, order="position", weights="folded", ends=False),
        dict(name="encoder_vit_h_content_b2", path="encoder", model="vit_h", batch=2, grid=64, density=0.3, order="content", weights="folded", ends=False),
        # one global block at density 1: the dense model through the same kernels
        dict(name="block_vit_h_global_dense_b4", path="block", model="vit_h", batch=4, grid=64, window=0, density=1.0, weights="folded"),
        # attention by itself: global at a large batch, and the windows of a batch
        dict(name="attention_global_b16", path="attention", batch=16, grid=64, window=0, heads=16, dim=80, density=0.4, order="position"),
        dict(name="attention_windows_b4", path="attention", batch=4, grid=64, window=WINDOW, heads=16, dim=64, density=0.4, order="position"),
        # the routed MLP by itself: huge-encoder width at a large batch, and a stage of a hierarchical encoder, whose
        # widths are not multiples of 128
        dict(name="mlp_1280_b16", path="mlp", batch=16, grid=64, width=1280, hidden=5120, density=0.4, weights="folded"),
        dict(name="mlp_576_b4", path="mlp", batch=4, grid=64, width=576, hidden=2304, density=0.5, weights="rows"),
    ]


# ------------------------------------------------------------------ sizes
def _model(case):
    return inputs.SHAPES[case["model"]]


def _tiles(S, mask_block, r):
    """Active tiles of the A-shape mask."""
    T = -(-S // mask_block)
    pre = min(T, int(math.floor(r * T + 1e-6)))
    return pre * T + (T - pre)


def _attention_flops(groups, S, heads, dim, mask_block, r):
    return 4.0 * mask_block * mask_block * dim * _tiles(S, mask_block, r) * heads * groups


def _windows(g, w):
    return (-(-g // w)) ** 2


def _keep(n, density):
    return B.ssam_keep_count(n, density)


def _block_work(shape, batch, g, window, density):
    """Flops of one block and the bytes of its weights."""
    n, D, Dm = g * g, shape.D, shape.Dm
    w = window or g
    groups = batch * (_windows(g, w) if window else 1)
    flops = 2.0 * batch * n * D * 4 * D + 4.0 * batch * _keep(n, density) * D * Dm
    flops += _attention_flops(groups, w * w, shape.heads, shape.d, 32 if window else 128, density)
    return flops, 2.0 * (4 * D * D + 2 * D * Dm + 2 * (2 * w - 1) * shape.d) + 4.0 * (9 * D + Dm)


def work(case):
    """Bytes (inputs, weights and outputs once) and flops of one pass."""
    path, batch, g = case["path"], case["batch"], case["grid"]
    n = g * g
    if path == "encoder":
        shape = _model(case)
        flops, nbytes = 0.0, 0.0
        for i in range(shape.depth):
            f, b = _block_work(shape, batch, g, 0 if i in shape.global_blocks else shape.ws, case["density"])
            flops, nbytes = flops + f, nbytes + b
        tokens = 2.0 * batch * n * shape.D
        if case["ends"]:
            kp = 3 * PATCH * PATCH
            flops += 2.0 * batch * n * (shape.D * kp + NECK * shape.D + 9 * NECK * NECK)
            nbytes += 2.0 * (shape.D * kp + n * shape.D + NECK * shape.D + 9 * NECK * NECK)
            return {"bytes": nbytes + 2.0 * batch * n * (kp + NECK), "flops": flops}
        return {"bytes": nbytes + 2 * tokens, "flops": flops}
    if path == "block":
        flops, nbytes = _block_work(_model(case), batch, g, case["window"], case["density"])
        return {"bytes": nbytes + 2 * 2.0 * batch * n * _model(case).D, "flops": flops}
    if path == "attention":
        w = case["window"] or g
        groups = batch * (_windows(g, w) if case["window"] else 1)
        return {"bytes": 2.0 * groups * w * w * 4 * case["heads"] * case["dim"],
                "flops": _attention_flops(groups, w * w, case["heads"], case["dim"], 32 if case["window"] else 128, case["density"])}
    if path == "mlp":
        k, D, Dm = _keep(n, case["density"]), case["width"], case["hidden"]
        return {"bytes": 2.0 * (2 * batch * k * D + 2 * D * Dm), "flops": 4.0 * batch * k * D * Dm}
    # select: the tokens are read, scores, keep-set and the tables of both kinds of block written
    out = 4.0 * batch * (n + _keep(n, case["density"]))
    if case["order"] == "content":
        out += 8.0 * batch * (_windows(g, WINDOW) * WINDOW * WINDOW + n)
    return {"bytes": 2.0 * batch * n * case["width"] + out, "flops": float(batch * n * case["width"])}


#: no drawn case is more work than the largest listed one
_MOST_FLOPS = max(work(c)["flops"] for c in listed())


def _between(rng, lo, hi):
    """A whole number, spread evenly over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: batches 1 to 16, grids 16x16 to 64x64 (even sides: the stripe interleave of a
    whole grid needs them; attention alone also larger ones), densities 0.2 to 1, all orders, layouts and widths."""
    while True:
        path = rng.choice(["encoder", "encoder", "encoder", "block", "attention", "mlp", "select"])
        case = dict(path=path, batch=_between(rng, 1, 8), grid=rng.choice([64, 2 * _between(rng, 8, 32)]),
                    density=rng.choice([0.2, 0.3, 0.4, 0.5, 0.6, 1.0]))
        if path == "encoder":
            case.update(model=rng.choice(["vit_b", "vit_l", "vit_h"]), order=rng.choice(["position", "position", "content"]),
                        weights=rng.choice(["folded", "folded", "packed", "rows"]), ends=rng.random() < 0.3)
        elif path == "block":
            case.update(model=rng.choice(["vit_b", "vit_l", "vit_h"]), window=rng.choice([WINDOW, 0]),
                        weights=rng.choice(["folded", "packed", "rows"]))
        elif path == "attention":
            case.update(batch=_between(rng, 1, 16), grid=rng.choice([64, 2 * _between(rng, 8, 48)]), window=rng.choice([WINDOW, 0]),
                        order=rng.choice(["position", "content"]))
            case["heads"], case["dim"] = rng.choice([(12, 64), (16, 64), (16, 80)])
        elif path == "mlp":
            case["batch"] = _between(rng, 1, 16)
            if rng.random() < 0.4:         # stages of a hierarchical encoder: token grid and width go together
                case["grid"], case["width"] = rng.choice([(256, 144), (128, 288), (64, 576), (32, 1152)])
                case["batch"] = min(case["batch"], 8)
                case["weights"] = "rows"
            else:
                case["width"], case["weights"] = rng.choice([768, 1024, 1280]), rng.choice(["folded", "packed", "rows"])
            case["hidden"] = 4 * case["width"]
        else:
            case.update(batch=_between(rng, 1, 16), width=rng.choice([768, 1024, 1280]), order=rng.choice(["position", "content"]))
        if work(case)["flops"] <= _MOST_FLOPS:
            return case


# ------------------------------------------------------------------ inputs
def _normal(gen, *shape, std=0.02, dtype=torch.float32):
    return (torch.randn(*shape, generator=gen, device=DEV) * std).to(dtype).contiguous()


def _tokens(gen, batch, g, D):
    """[batch, g*g, D]: per image 8 low-frequency waves mixed into the channels, plus noise."""
    line = torch.arange(g, device=DEV, dtype=torch.float32) / g
    mix = (0.5 + torch.randn(8, D, generator=gen, device=DEV)) / math.sqrt(8.0)
    x = torch.empty((batch, g * g, D), dtype=BF, device=DEV)
    for b in range(batch):
        u, v = torch.rand(2, 8, 1, 1, generator=gen, device=DEV) * 6 - 3
        phase = torch.rand(8, 1, 1, generator=gen, device=DEV) * 2 * math.pi
        waves = torch.sin(2 * math.pi * (u * line[None, :, None] + v * line[None, None, :]) + phase).reshape(8, g * g)
        x[b] = waves.t() @ mix + 0.3 * torch.randn(g * g, D, generator=gen, device=DEV)
    return x


def _block_weights(gen, shape, w, layout, rows):
    """Device weights of one block whose attention groups are w x w, laid out as a program lays them out at load time."""
    D, Dm = shape.D, shape.Dm
    wt = {
        "ln1_g": 1 + _normal(gen, D), "ln1_b": _normal(gen, D), "wqkv": _normal(gen, 3 * D, D, dtype=BF), "bqkv": _normal(gen, 3 * D),
        "rel_h": _normal(gen, 2 * w - 1, shape.d, dtype=BF), "rel_w": _normal(gen, 2 * w - 1, shape.d, dtype=BF),
        "wproj": _normal(gen, D, D, dtype=BF), "bproj": _normal(gen, D), "ln2_g": 1 + _normal(gen, D), "ln2_b": _normal(gen, D),
        "w1": _normal(gen, Dm, D, dtype=BF), "b1": _normal(gen, Dm), "w2": _normal(gen, D, Dm, dtype=BF), "b2": _normal(gen, D),
    }
    if layout == "rows":
        return wt
    fold = layout == "folded"
    fold1 = fold and rows % 128 == 0          # the folded qkv contraction exists for whole tiles of 128 rows
    return B.pack_block_weights(wt, fold_ln1=fold1, fold_kv_bias=fold1, fold_ln2=fold)


def _host_table(a):
    return torch.from_numpy(a).to(DEV)


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    return {"case": case, **_PREPARE[case["path"]](case, gen)}


def _prepare_encoder(case, gen):
    shape, batch, g = _model(case), case["batch"], case["grid"]
    n = g * g
    k = _keep(n, case["density"])
    content = case["order"] == "content"
    flags = [i in shape.global_blocks for i in range(shape.depth)]
    wts = [_block_weights(gen, shape, g if f else shape.ws, case["weights"], batch * n) for f in flags]
    structs = [B.block_weights_struct(w) for w in wts]
    cfg_l = B.make_cfg(batch, g, shape.D, shape.heads, shape.Dm, shape.ws, 32, k, case["density"], content_order=content, stripe=STRIPE)
    cfg_g = B.make_cfg(batch, g, shape.D, shape.heads, shape.Dm, 0, 128, k, case["density"], content_order=content, stripe=STRIPE)
    if content:
        groups, S = _windows(g, shape.ws), shape.ws ** 2
        tables = [torch.empty(s, dtype=torch.int32, device=DEV) for s in ((batch, groups * S), (batch * groups, S), (batch, n), (batch, n))]
    else:
        glob = _host_table(B.ssam_build_perm(g, g, STRIPE)[0])
        tables = [_host_table(B.ssam_build_window_table(g, shape.ws, STRIPE)),
                  _host_table(B.ssam_build_perm(shape.ws, shape.ws, STRIPE)[0]), glob, glob]
    s = {"wts": wts, "structs": structs, "flags": flags, "plan": B.EncoderPlan(structs, flags), "cfg": (cfg_l, cfg_g), "tables": tables,
         "scores": torch.empty((batch, n), device=DEV), "keep": torch.empty((batch, k), dtype=torch.int32, device=DEV),
         "x": torch.empty((batch, n, shape.D), dtype=BF, device=DEV),
         "workspace": torch.empty(B.ssam_encoder_workspace_bytes(cfg_l, cfg_g), dtype=torch.uint8, device=DEV)}
    if case["ends"]:
        side = g * PATCH
        s["image"] = _normal(gen, batch, 3, side, side, std=1.0, dtype=BF)
        s["embed"] = (_normal(gen, shape.D, 3 * PATCH * PATCH, dtype=BF), _normal(gen, shape.D), _normal(gen, n, shape.D, dtype=BF))
        s["neck"] = (_normal(gen, NECK, shape.D, dtype=BF), 1 + _normal(gen, NECK), _normal(gen, NECK),
                     _normal(gen, NECK, 9 * NECK, dtype=BF), 1 + _normal(gen, NECK), _normal(gen, NECK))
        s["out"] = torch.empty((batch, n, NECK), dtype=BF, device=DEV)
        s["embed_ws"] = torch.empty(B.ssam_patch_embed_workspace_bytes(batch, side, side, PATCH), dtype=torch.uint8, device=DEV)
        s["neck_ws"] = torch.empty(B.ssam_neck_workspace_bytes(batch, g, shape.D, NECK), dtype=torch.uint8, device=DEV)
    else:
        s["x0"] = _tokens(gen, batch, g, shape.D)
    return s


def _prepare_block(case, gen):
    shape, batch, g, w = _model(case), case["batch"], case["grid"], case["window"]
    n = g * g
    wt = _block_weights(gen, shape, w or g, case["weights"], batch * n)
    x0 = _tokens(gen, batch, g, shape.D)
    keep = B.ssam_select_tokens(B.ssam_score_tokens(x0.view(batch, g, g, shape.D)), _keep(n, case["density"]))
    cfg = B.make_cfg(batch, g, shape.D, shape.heads, shape.Dm, w, 32 if w else 128, keep.shape[1], case["density"])
    sigma = _host_table(B.ssam_build_perm(w or g, w or g, STRIPE)[0])
    return {"wt": wt, "struct": B.block_weights_struct(wt), "cfg": cfg, "x0": x0, "x": torch.empty_like(x0), "keep": keep, "sigma": sigma,
            "table": _host_table(B.ssam_build_window_table(g, w, STRIPE)) if w else sigma,
            "workspace": torch.empty(B.ssam_encoder_block_workspace_bytes(cfg), dtype=torch.uint8, device=DEV)}


def _prepare_attention(case, gen):
    batch, g, heads, dim = case["batch"], case["grid"], case["heads"], case["dim"]
    w = case["window"] or g
    groups = batch * (_windows(g, w) if case["window"] else 1)
    if case["order"] == "content":
        scores = torch.exp(torch.randn(batch, g * g, generator=gen, device=DEV))
        sigma = B.ssam_build_content_tables(scores, g, case["window"], STRIPE)[1]
    else:
        sigma = _host_table(B.ssam_build_perm(w, w, STRIPE)[0])
    return {"qkv": _normal(gen, groups, w * w, 3, heads, dim, std=0.7, dtype=BF), "sigma": sigma, "w": w,
            "rel": (_normal(gen, 2 * w - 1, dim, dtype=BF), _normal(gen, 2 * w - 1, dim, dtype=BF)),
            "out": torch.empty((groups, w * w, heads * dim), dtype=BF, device=DEV)}


def _prepare_mlp(case, gen):
    batch, n, D, Dm = case["batch"], case["grid"] ** 2, case["width"], case["hidden"]
    scores = torch.exp(torch.randn(batch, n, generator=gen, device=DEV))      # heavy-tailed, as Sobel scores of images are
    keep = B.ssam_select_tokens(scores, _keep(n, case["density"]))
    ln = (1 + _normal(gen, D), _normal(gen, D))
    w1, b1, w2, b2 = _normal(gen, Dm, D, dtype=BF), _normal(gen, Dm), _normal(gen, D, Dm, dtype=BF), _normal(gen, D)
    if case["weights"] == "folded":
        w1, colsum, b1 = B.ssam_fold_ln_weight(w1, b1, *ln)
        weights = (B.ssam_pack_weight(w1), colsum, b1, B.ssam_pack_weight(w2), b2)
    elif case["weights"] == "packed":
        weights = (*ln, 1e-6, B.ssam_pack_weight(w1), b1, B.ssam_pack_weight(w2), b2)
    else:
        weights = (*ln, 1e-6, w1, b1, w2, b2)
    x0 = _normal(gen, batch, n, D, std=1.0, dtype=BF)
    return {"x0": x0, "x": torch.empty_like(x0), "keep": keep, "weights": weights,
            "workspace": torch.empty(B.ssam_routed_mlp_workspace_bytes(batch, keep.shape[1], D, Dm), dtype=torch.uint8, device=DEV)}


def _prepare_select(case, gen):
    batch, g, D = case["batch"], case["grid"], case["width"]
    n = g * g
    groups, S = _windows(g, WINDOW), WINDOW * WINDOW
    s = {"x": _tokens(gen, batch, g, D).view(batch, g, g, D), "scores": torch.empty((batch, n), device=DEV),
         "keep": torch.empty((batch, _keep(n, case["density"])), dtype=torch.int32, device=DEV),
         "workspace": torch.empty(4 * batch * n, dtype=torch.uint8, device=DEV)}
    if case["order"] == "content":
        s["tables"] = [torch.empty(sz, dtype=torch.int32, device=DEV) for sz in ((batch, groups * S), (batch * groups, S), (batch, n), (batch, n))]
    return s


# ------------------------------------------------------------------ passes
def run(state):
    return _RUN[state["case"]["path"]](state, state["case"])


def _run_encoder(s, case):
    # the stack works in place on its tokens: a program has new ones for every call, here the same again
    if case["ends"]:
        B.ssam_patch_embed(s["image"], *s["embed"], PATCH, x=s["x"], workspace=s["embed_ws"])
    else:
        s["x"].copy_(s["x0"])
    B.ssam_encoder_forward(s["x"], s["structs"], s["flags"], *s["cfg"], *s["tables"], s["scores"], s["keep"], s["workspace"], plan=s["plan"])
    if not case["ends"]:
        return {"x": s["x"], "keep": s["keep"]}
    B.ssam_neck(s["x"], *s["neck"], case["grid"], out=s["out"], workspace=s["neck_ws"])
    return {"x": s["x"], "keep": s["keep"], "embedding": s["out"]}


def _run_block(s, case):
    s["x"].copy_(s["x0"])
    return B.ssam_encoder_block(s["x"], s["struct"], s["cfg"], s["table"], s["sigma"], s["keep"], workspace=s["workspace"])


def _run_attention(s, case):
    return B.ssam_sparse_attention(s["qkv"], *s["rel"], s["sigma"], s["w"], 32 if case["window"] else 128, case["density"], out=s["out"])


def _run_mlp(s, case):
    s["x"].copy_(s["x0"])
    if case["weights"] == "folded":
        return B.ssam_routed_mlp_folded(s["x"], s["keep"], 1e-6, *s["weights"], workspace=s["workspace"])
    return B.ssam_routed_mlp(s["x"], s["keep"], *s["weights"], workspace=s["workspace"], w_packed=case["weights"] == "packed")


def _run_select(s, case):
    B.ssam_score_tokens(s["x"], scores=s["scores"], workspace=s["workspace"])
    out = {"scores": s["scores"]}
    if case["order"] == "content":
        t = s["tables"]
        B.ssam_build_content_tables(s["scores"], case["grid"], WINDOW, STRIPE, gather_table=t[0], sigma=t[1])
        B.ssam_build_content_tables(s["scores"], case["grid"], 0, STRIPE, gather_table=t[2], sigma=t[3])
        out["tables"] = t
    B.ssam_select_tokens(s["scores"], s["keep"].shape[1], keep_idx=s["keep"])
    out["keep"] = s["keep"]
    return out


_PREPARE = {"encoder": _prepare_encoder, "block": _prepare_block, "attention": _prepare_attention, "mlp": _prepare_mlp, "select": _prepare_select}
_RUN = {"encoder": _run_encoder, "block": _run_block, "attention": _run_attention, "mlp": _run_mlp, "select": _run_select}


def tolerance(case):
    """What another correct implementation at the same precision may differ by: about four times what was measured.

    attention, mlp: against the same product in 64 bits (rel 2.4e-3 and 1.5e-3, the bf16 roundings of the stored
    intermediates; max 9.6e-3 and 9.7e-3).  block, encoder: the folded against the row-major form, two orders of rounding
    of the same block (rel 1.4e-3 to 3.2e-3 for one block, 8e-3 to 1.5e-2 after 12 to 32 blocks whose residual stream
    is rounded in place twice a block; max 2.2e-2 and 0.12).  select: scores in 32 bits against 64 bits (rel 7e-8, max
    5e-7); a different order of those sums can swap tokens whose scores all but tie, and with them a few indices."""
    return {
        "select": {"rel": 1e-6, "max": 4e-6, "differ": 0.01},
        "attention": {"rel": 0.01, "max": 0.04},
        "mlp": {"rel": 0.006, "max": 0.04},
        "block": {"rel": 0.012, "max": 0.09},
        "encoder": {"rel": 0.03, "max": 0.45, "differ": 0.01},
    }[case["path"]]
