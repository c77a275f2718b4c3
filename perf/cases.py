"""The work that a user of this package has it do, as cases that can be timed.

A ViT backbone on a high-resolution tile calls the package in a fixed order: patch embedding, blocks on
the full patch grid (attention restricted to 3x3 neighbouring windows plus the global tokens, with the
importance scores as a by-product where a pruning stage follows), selection and compaction of the kept
tokens, blocks on the pruned sequence.  The cases take each of these calls through the Python binding, as
a program does: outputs and workspaces are left to the binding.  Sizes are those of the synthetic
workloads (`synth.CONFIGS`), of the tests and of the benchmark: patch grids of 16 to 256 a side, windows
2 to 64, fp32 and bf16, one or several global tokens, contiguous or fused q/k/v.

The selection runs on scores that are part of the inputs and not on the attention's own: its result is a
set of whole numbers, in which two correct roundings of a score next to the k-th one would change places.
For the same reason the stack of blocks is the one without a pruning stage (feature maps for a dense
head), and the pruned half of a backbone stands as a block on a given set of survivors.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2601_12150_amd import binding as nb

HEAD_DIM = 64


def listed():
    return [
        # the smallest calls: one 448-pixel image in fp32 (28 x 28 patches, windows of 7), and one
        # 224-pixel image with 14-pixel patches in bf16 (2 x 2 windows of 8)
        _layer("layer_f32_28_w7", "f32", 1, 28, 28, 7),
        _layer("layer_bf16_16_w8", "bf16", 1, 16, 16, 8),
        # ordinary ones: a batch of four 1024-pixel images, q/k/v as views of the fused projection
        _layer("layer_bf16_64_w8_b4_fused", "bf16", 4, 64, 64, 8, fused=True),
        # 1400-pixel images with 14-pixel patches: a grid that the window does not divide, with the
        # CLS token and four register tokens as global tokens
        _layer("layer_bf16_100_w8_b2_g5", "bf16", 2, 100, 100, 8, n_global=5),
        # 2048-pixel images, the size that the benchmark's step has
        _layer("layer_bf16_128_w8_b2", "bf16", 2, 128, 128, 8),
        # 4096-pixel image, wide windows
        _layer("layer_bf16_256_w16", "bf16", 1, 256, 256, 16),
        # the largest: 3430-pixel image (245 x 245 patches), windows of 64
        _layer("layer_bf16_245_w64", "bf16", 1, 245, 245, 64),
        # ranking from q and k alone (no attention output wanted), two 2048-pixel images
        {"name": "scores_bf16_128_b2", "kind": "scores", "dtype": "bf16", "batch": 2, "heads": 16, "patches": 128 * 128,
         "n_global": 1},
        # selection and compaction of 60 % of the tokens of two 2048-pixel images, with their coordinates
        {"name": "filter_bf16_128_b2", "kind": "filter", "dtype": "bf16", "batch": 2, "patches": 128 * 128, "keep_pct": 60,
         "channels": 1024},
        # pixels to tokens: a 1400-pixel image in 14-pixel patches (588 columns, no multiple of 64)
        {"name": "embed_100_p14", "kind": "embed", "batch": 1, "grid_h": 100, "grid_w": 100, "patch": 14, "dim": 1024},
        # one block of the pruned half of a backbone on a 2048-pixel image: 60 % of the patches are left
        {"name": "block_pruned_128", "kind": "block", "batch": 1, "grid_h": 128, "grid_w": 128, "window": 8, "keep_pct": 60,
         "heads": 16},
        # the first twelve blocks on a 2048-pixel image, with the feature maps a dense head takes
        {"name": "stack_12_128", "kind": "stack", "batch": 1, "grid_h": 128, "grid_w": 128, "window": 8, "heads": 16,
         "layers": 12, "taps": 4},
    ]


def _layer(name, dtype, batch, grid_h, grid_w, window, n_global=1, fused=False, heads=16):
    return {"name": name, "kind": "layer", "dtype": dtype, "batch": batch, "heads": heads, "grid_h": grid_h,
            "grid_w": grid_w, "window": window, "n_global": n_global, "fused": fused}


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        case = _draw_any(rng)
        w = work(case)
        # no more than the largest listed cases take (6 TFLOP of attention in the widest windows, 5 TFLOP of a
        # stack, 0.55 GB; the attention of narrower windows gets less out of each byte and lane)
        if w["flops"] <= (2.4e12 if case["kind"] == "layer" else 4.5e12) and w["bytes"] <= 0.6e9:
            return case


def _draw_any(rng):
    kind = rng.choices(("layer", "scores", "filter", "embed", "block", "stack"), (7, 1, 1, 1, 1, 1))[0]
    if kind == "layer":
        f32 = rng.random() < 0.15
        grid_h = _log_int(rng, 14, 64 if f32 else 256)
        grid_w = grid_h if rng.random() < 0.5 else _log_int(rng, max(14, grid_h // 2), min(64 if f32 else 256, grid_h * 2))
        window = rng.choice((7, 8)) if f32 else rng.choice((2, 4, 7, 8, 8, 8, 16, 16, 32, 64))
        case = _layer("", "f32" if f32 else "bf16", rng.choice((1, 1, 2, 2, 3, 4)), grid_h, grid_w, window,
                      n_global=rng.choice((1, 1, 1, 5)), fused=rng.random() < 0.5, heads=rng.choice((8, 16, 16, 24)))
        del case["name"]
        return case
    if kind == "scores":
        return {"kind": kind, "dtype": rng.choice(("f32", "bf16", "bf16")), "batch": rng.choice((1, 2, 4)),
                "heads": rng.choice((8, 16, 24)), "patches": _log_int(rng, 784, 65536), "n_global": rng.choice((1, 1, 5))}
    if kind == "filter":
        return {"kind": kind, "dtype": rng.choice(("f32", "bf16", "bf16")), "batch": rng.choice((1, 2, 4, 8)),
                "patches": _log_int(rng, 784, 65536), "keep_pct": rng.randint(30, 80),
                "channels": rng.choice((512, 1024, 1024, 1536))}
    if kind == "embed":
        grid = _log_int(rng, 16, 200)
        return {"kind": kind, "batch": rng.choice((1, 1, 2, 4)), "grid_h": grid, "grid_w": rng.randint(max(16, grid // 2), grid),
                "patch": rng.choice((14, 16)), "dim": rng.choice((512, 1024, 1024, 1536))}
    grid = _log_int(rng, 28, 160)
    case = {"kind": kind, "batch": rng.choice((1, 1, 2)), "grid_h": grid, "grid_w": rng.randint(max(16, grid // 2), grid),
            "window": rng.choice((8, 8, 16)), "heads": rng.choice((8, 16, 16, 24))}
    if kind == "block":
        case["keep_pct"] = rng.randint(30, 80)
    else:
        case["layers"] = rng.randint(2, 12)
        case["taps"] = rng.randint(1, 2)
    return case


# ---- inputs


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _background(grid_h, grid_w, fraction, seed):
    """[grid_h, grid_w] bool: rectangles of 8 to 48 patches a side until `fraction` of the grid is covered."""
    rng = np.random.default_rng(seed)
    m = np.zeros((grid_h, grid_w), dtype=bool)
    while m.mean() < fraction:
        h, w = (min(int(rng.integers(8, 49)), max(g // 2, 1)) for g in (grid_h, grid_w))
        r, c = int(rng.integers(0, grid_h - h + 1)), int(rng.integers(0, grid_w - w + 1))
        m[r:r + h, c:c + w] = True
    return m


def _qkv(case, seed, gen, T, background):
    """q, k, v [B,H,T,D]: N(0,1), and the keys and values of background patches one vector per (image, head)
    plus a little noise, as the empty part of a slide gives them."""
    B, H, D = case["batch"], case["heads"], HEAD_DIM
    if case.get("fused"):
        x = torch.randn((B, T, 3, H, D), generator=gen, device="cuda")
        q, k, v = (x[:, :, i].transpose(1, 2) for i in range(3))
    else:
        q, k, v = torch.randn((3, B, H, T, D), generator=gen, device="cuda")
        x = None
    if background is not None:
        idx = torch.from_numpy(np.flatnonzero(background)).cuda() + (T - background.size)
        for t in (k, v):
            shared = torch.randn((B, H, 1, D), generator=gen, device="cuda")
            t[:, :, idx] = shared + 0.01 * torch.randn((B, H, idx.numel(), D), generator=gen, device="cuda")
    dt = _dtype(case)
    if x is not None:
        x = x.to(dt)
        return tuple(x[:, :, i].transpose(1, 2) for i in range(3))
    return q.to(dt).contiguous(), k.to(dt).contiguous(), v.to(dt).contiguous()


def _block_weights(dim, gen):
    """Matrices N(0, 0.02^2) bf16, biases N(0, 0.02^2) fp32, LayerNorm gain 1 and offset 0 plus N(0, 0.1^2)."""
    w = {}
    for name, o, i in (("qkv", 3 * dim, dim), ("proj", dim, dim), ("fc1", 4 * dim, dim), ("fc2", dim, 4 * dim)):
        w["w_" + name] = (0.02 * torch.randn((o, i), generator=gen, device="cuda")).to(torch.bfloat16)
        w["b_" + name] = 0.02 * torch.randn(o, generator=gen, device="cuda")
    for ln in ("ln1", "ln2"):
        w[ln + "_g"] = 1.0 + 0.1 * torch.randn(dim, generator=gen, device="cuda")
        w[ln + "_b"] = 0.1 * torch.randn(dim, generator=gen, device="cuda")
    return w


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    kind, B = case["kind"], case["batch"]
    s = {"case": case}
    if kind == "layer":
        T = case["n_global"] + case["grid_h"] * case["grid_w"]
        s["qkv"] = _qkv(case, seed, gen, T, _background(case["grid_h"], case["grid_w"], 0.4, seed))
    elif kind == "scores":
        T = case["n_global"] + case["patches"]
        bg = np.random.default_rng(seed).permutation(case["patches"]) < 2 * case["patches"] // 5
        s["qkv"] = _qkv(case, seed, gen, T, bg)
    elif kind == "filter":
        N = case["patches"]
        # softmax weights of a global token: the exponentials of roughly normal logits, averaged over heads
        logits = torch.randn((B, 16, N), generator=gen, device="cuda")
        s["scores"] = torch.softmax(logits, dim=2).mean(dim=1).contiguous()
        s["x"] = torch.randn((B, 1 + N, case["channels"]), generator=gen, device="cuda").to(_dtype(case))
        side = int(math.ceil(math.sqrt(N)))
        j = torch.arange(N, device="cuda", dtype=torch.int32)
        s["coords"] = (((j // side) << 16) | (j % side)).repeat(B, 1).contiguous()
        s["k"] = (N * case["keep_pct"] + 99) // 100
    elif kind == "embed":
        dim, p, gh, gw = case["dim"], case["patch"], case["grid_h"], case["grid_w"]
        s["pixels"] = ((torch.rand((B, 3, gh * p, gw * p), generator=gen, device="cuda") - 0.5) / 0.25).to(torch.bfloat16)
        s["w_patch"], s["cls"], s["pos"] = ((0.02 * torch.randn(shape, generator=gen, device="cuda")).to(torch.bfloat16)
                                            for shape in ((dim, 3 * p * p), (dim,), (1 + gh * gw, dim)))
        s["b_patch"] = 0.02 * torch.randn(dim, generator=gen, device="cuda")
    else:
        dim, gh, gw = case["heads"] * HEAD_DIM, case["grid_h"], case["grid_w"]
        N = gh * gw
        if kind == "block":
            # survivors: the tissue, then background patches at random, ascending as a selection gives them
            k = (N * case["keep_pct"] + 99) // 100
            rows = []
            for b in range(B):
                bg = _background(gh, gw, 1.0 - case["keep_pct"] / 100.0, seed + 1000 * b).reshape(-1)
                order = np.argsort(bg + 0.5 * np.random.default_rng(seed + b).random(N), kind="stable")
                j = np.sort(order[:k])
                rows.append(((j // gw) << 16) | (j % gw))
            s["coords"] = torch.from_numpy(np.stack(rows).astype(np.int32)).cuda()
            N = k
        s["weights"] = [_block_weights(dim, gen) for _ in range(case.get("layers", 1))]
        s["x"] = torch.randn((B, 1 + N, dim), generator=gen, device="cuda").to(torch.bfloat16)
    return s


# ---- one pass


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "layer":
        q, k, v = s["qkv"]
        return nb.ns_attn_forward_scores(q, k, v, c["grid_h"], c["grid_w"], c["window"], n_global=c["n_global"])
    if kind == "scores":
        q, k, _ = s["qkv"]
        return nb.cls_scores(q, k, n_global=c["n_global"])
    if kind == "filter":
        return nb.topk_filter(s["scores"], s["k"], x=s["x"], coords=s["coords"])
    if kind == "embed":
        return nb.vit_embed(s["pixels"], s["w_patch"], s["b_patch"], s["cls"], s["pos"], c["patch"])
    if kind == "block":
        return nb.vit_block_forward(s["x"], s["weights"][0], c["grid_h"], c["grid_w"], c["window"], c["heads"],
                                    coords=s["coords"])
    return nb.vit_forward(s["x"], s["weights"], c["grid_h"], c["grid_w"], c["window"], c["heads"], tap_layers=_taps(c))


def _taps(c):
    """Feature maps at evenly spaced depths, the last block among them."""
    return [c["layers"] * (i + 1) // c["taps"] for i in range(c["taps"])]


# ---- what a pass cannot do without


def _pairs(grid_h, grid_w, window):
    """Allowed (query, key) pairs of patches: the 3x3 windows around each query's own, clipped at the edges."""
    n = 1
    for g in (grid_h, grid_w):
        sides = [min(window, g - i) for i in range(0, g, window)]
        n *= sum(a * sum(sides[max(i - 1, 0):i + 2]) for i, a in enumerate(sides))
    return n


def work(case):
    kind, B = case["kind"], case["batch"]
    elt = 4 if case.get("dtype") == "f32" else 2
    if kind == "layer":
        H, D, G, N = case["heads"], HEAD_DIM, case["n_global"], case["grid_h"] * case["grid_w"]
        T = G + N
        pairs = _pairs(case["grid_h"], case["grid_w"], case["window"]) + N * G + G * T
        return {"bytes": 4.0 * B * H * T * D * elt + 4.0 * B * H * G * (T + 1) + 4.0 * B * N, "flops": 4.0 * D * pairs * B * H}
    if kind == "scores":
        H, D, G, N = case["heads"], HEAD_DIM, case["n_global"], case["patches"]
        return {"bytes": float(B * H * (G + N + G) * D * elt + 4 * B * N), "flops": 2.0 * D * G * (G + N) * B * H}
    if kind == "filter":
        N = case["patches"]
        k = (N * case["keep_pct"] + 99) // 100
        return {"bytes": float(B * (4 * N + 12 * k + 2 * (1 + k) * case["channels"] * elt)), "flops": 0.0}
    if kind == "embed":
        K, dim, N = 3 * case["patch"] ** 2, case["dim"], case["grid_h"] * case["grid_w"]
        return {"bytes": 2.0 * (B * N * K + dim * K + (1 + N) * dim + B * (1 + N) * dim), "flops": 2.0 * B * N * K * dim}
    dim, N, layers = case["heads"] * HEAD_DIM, case["grid_h"] * case["grid_w"], case.get("layers", 1)
    keep = case.get("keep_pct", 100) / 100.0
    k = int(math.ceil(N * keep))
    # (survivors of a pruned grid: as if spread evenly, i.e. keep^2 of the full grid's pairs, the least there can be)
    pairs = _pairs(case["grid_h"], case["grid_w"], case["window"]) * keep * keep + 2 * k
    flops = layers * (2.0 * B * (1 + k) * 12 * dim * dim + 4.0 * HEAD_DIM * pairs * B * case["heads"])
    return {"bytes": 2.0 * (layers * 12 * dim * dim + (2 + case.get("taps", 0)) * B * (1 + k) * dim), "flops": flops}


def tolerance(case):
    kind = case["kind"]
    if kind == "filter":
        return "exact"
    if kind == "scores" or case.get("dtype") == "f32":
        return {"rel": 1e-5}          # fp32 sums of exact products, fp32 results
    return {"rel": 1e-2}              # bf16 results (the fp32 by-products are nearer)
