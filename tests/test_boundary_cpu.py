"""Host-side checks of the C-ABI library that need no GPU: it loads, exports every function
the header declares, and rejects bad arguments before launching anything."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "nsattn.h")


@pytest.fixture(scope="module")
def nb():
    from paper_2601_12150_amd import binding
    return binding


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    names = re.findall(r"\b([a-z_][a-z0-9_]*)\s*\([^;{]*\)\s*;", text)
    return sorted(set(names))


def test_library_exports_every_declared_function(nb):
    names = declared_functions()
    assert {"ns_attn_forward", "cls_scores", "topk_filter", "vit_block_forward"} <= set(names)
    raw = ctypes.CDLL(nb.LIB_PATH)
    for n in names:
        assert hasattr(raw, n), "libnsattn.so does not export %s" % n
    assert set(nb.EXPORTS) == set(names)


def good_desc(nb):
    d = nb.ns_attn_desc()
    d.batch, d.heads, d.head_dim = 1, 2, 64
    d.grid_h = d.grid_w = 8
    d.block, d.radius, d.n_global, d.dtype, d.tokens = 4, 1, 1, nb.NS_BF16, 65
    d.scale = 0.125
    d.q_stride_b, d.q_stride_h, d.q_stride_t = 2 * 65 * 64, 65 * 64, 64
    d.out_stride_b, d.out_stride_h, d.out_stride_t = 2 * 65 * 64, 65 * 64, 64
    return d


FAKE = ctypes.c_void_p(0x10000)   # never dereferenced: every call below fails validation first


def attn_call(nb, d, q=FAKE, out=ctypes.c_void_p(0x20000), ws=ctypes.c_void_p(0x30000), ws_bytes=1 << 30):
    return nb.lib.ns_attn_forward(ctypes.byref(d), q, FAKE, FAKE, out, None, None, ws, ws_bytes, None)


def test_descriptor_validation(nb):
    d = good_desc(nb)
    assert nb.lib.ns_attn_workspace_bytes(ctypes.byref(d)) > 0
    cases = [("batch", 0, nb.NS_ERR_INVALID_ARG), ("heads", -1, nb.NS_ERR_INVALID_ARG),
             ("block", 0, nb.NS_ERR_INVALID_ARG), ("dtype", 7, nb.NS_ERR_INVALID_ARG),
             ("tokens", 64, nb.NS_ERR_INVALID_ARG), ("scale", float("nan"), nb.NS_ERR_INVALID_ARG),
             ("q_stride_t", 63, nb.NS_ERR_INVALID_ARG), ("q_stride_h", 65 * 64 + 1, nb.NS_ERR_INVALID_ARG),
             ("out_stride_t", 8, nb.NS_ERR_INVALID_ARG),
             ("head_dim", 128, nb.NS_ERR_UNSUPPORTED), ("radius", 2, nb.NS_ERR_UNSUPPORTED),
             ("n_global", 300, nb.NS_ERR_UNSUPPORTED), ("n_global", 0, nb.NS_ERR_INVALID_ARG)]
    for field, value, code in cases:
        d = good_desc(nb)
        setattr(d, field, value)
        if field == "n_global":
            d.tokens = 64 + value
        assert attn_call(nb, d) == code, field
        assert nb.lib.ns_last_error()
        assert nb.lib.ns_attn_workspace_bytes(ctypes.byref(d)) == 0
    assert nb.lib.ns_attn_forward(None, FAKE, FAKE, FAKE, FAKE, None, None, None, 0, None) == nb.NS_ERR_INVALID_ARG


def test_pointer_and_workspace_validation(nb):
    d = good_desc(nb)
    assert attn_call(nb, d, q=None) == nb.NS_ERR_INVALID_ARG
    assert attn_call(nb, d, q=ctypes.c_void_p(0x10008)) == nb.NS_ERR_INVALID_ARG       # misaligned
    assert attn_call(nb, d, out=FAKE) == nb.NS_ERR_INVALID_ARG                         # aliasing
    assert attn_call(nb, d, ws=None) == nb.NS_ERR_WORKSPACE
    assert attn_call(nb, d, ws=ctypes.c_void_p(0x30010)) == nb.NS_ERR_WORKSPACE        # misaligned
    assert attn_call(nb, d, ws_bytes=16) == nb.NS_ERR_WORKSPACE
    assert b"needed" in nb.lib.ns_last_error()


def test_forward_scores_validation(nb):
    L, d = nb.lib, good_desc(nb)
    out, ws = ctypes.c_void_p(0x20000), ctypes.c_void_p(0x30000)
    def call(logits=FAKE, scores=FAKE, desc=d):
        return L.ns_attn_forward_scores(ctypes.byref(desc), FAKE, FAKE, FAKE, out, logits, None, scores, ws, 1 << 30, None)
    assert call(logits=None) == nb.NS_ERR_INVALID_ARG            # the scoring reads the logits back
    assert call(scores=None) == nb.NS_ERR_INVALID_ARG
    assert call(scores=ctypes.c_void_p(0x10002)) == nb.NS_ERR_INVALID_ARG
    bad = good_desc(nb)
    bad.heads = 0
    assert call(desc=bad) == nb.NS_ERR_INVALID_ARG


def test_topk_and_scores_validation(nb):
    L = nb.lib
    args = dict(x=None, C=0, dt=nb.NS_BF16, cin=None, kept=FAKE, y=None, cout=None)
    def call(B, N, k, scores=FAKE, **kw):
        a = dict(args); a.update(kw)
        return L.topk_filter(B, N, k, scores, a["x"], a["C"], a["dt"], a["cin"], a["kept"], a["y"],
                             a["cout"], None, 0, None)
    assert call(1, 100, 0) == nb.NS_ERR_INVALID_ARG
    assert call(1, 100, 101) == nb.NS_ERR_INVALID_ARG
    assert call(0, 100, 10) == nb.NS_ERR_INVALID_ARG
    assert call(1, 100, 10, scores=None) == nb.NS_ERR_INVALID_ARG
    assert call(1, 100, 10, x=FAKE, C=64) == nb.NS_ERR_INVALID_ARG                   # y missing
    assert call(1, 100, 10, x=FAKE, y=ctypes.c_void_p(0x20000), C=3) == nb.NS_ERR_UNSUPPORTED
    assert call(1, 100, 10, cin=FAKE) == nb.NS_ERR_INVALID_ARG                       # coords_out missing
    # rows above 32768 scores need a workspace (several workgroups per image)
    assert L.topk_filter_workspace_bytes(4, 16384, 100) == 0
    assert L.topk_filter_workspace_bytes(1, 32768, 100) == 0
    assert L.topk_filter_workspace_bytes(1, 70001, 100) == 4 * 69 * 1024 + 4 * 8 + 69 * 4
    assert L.topk_filter_workspace_bytes(2, 300000, 100) == 2 * (4 * 98 * 1024 + 4 * 8 + 98 * 4)   # 3 keys per thread
    assert call(1, 70001, 10) == nb.NS_ERR_WORKSPACE
    assert b"needed" in nb.lib.ns_last_error()
    assert L.cls_scores_from_logits(1, 2, 1, 1, FAKE, FAKE, FAKE, None) == nb.NS_ERR_INVALID_ARG
    assert L.cls_scores_from_logits(1, 2, 10, 1, None, FAKE, FAKE, None) == nb.NS_ERR_INVALID_ARG
    d = good_desc(nb)
    assert L.cls_scores(ctypes.byref(d), FAKE, FAKE, None, FAKE, 1 << 30, None) == nb.NS_ERR_INVALID_ARG
    assert L.cls_scores_workspace_bytes(ctypes.byref(d)) > 0


def test_embed_validation(nb):
    L = nb.lib
    assert L.vit_embed_workspace_bytes(1, 3, 128, 128, 14, 1024) == 16384 * 640 * 2 + 1024 * 640 * 2   # 588 -> 640 columns
    assert L.vit_embed_workspace_bytes(1, 3, 8, 8, 16, 100) == 0                                      # dim % 128
    def call(B=1, ch=3, gh=8, gw=8, ps=14, dim=512, px=FAKE, w=FAKE, ws=FAKE, ws_bytes=1 << 30):
        return L.vit_embed(B, ch, gh, gw, ps, dim, px, w, FAKE, FAKE, FAKE, FAKE, ws, ws_bytes, None)
    assert call(B=0) == nb.NS_ERR_INVALID_ARG
    assert call(dim=100) == nb.NS_ERR_UNSUPPORTED
    assert call(px=None) == nb.NS_ERR_INVALID_ARG
    assert call(w=ctypes.c_void_p(0x10008)) == nb.NS_ERR_INVALID_ARG          # misaligned
    assert call(ws=None) == nb.NS_ERR_WORKSPACE
    assert call(ws_bytes=1024) == nb.NS_ERR_WORKSPACE


def test_a_batch_no_launch_can_hold_is_refused_first(nb):
    """The merge of the global rows, the scoring and the lists have the image in a grid dimension of 16 bits: more
    images are refused before the attention kernel, which has not, is launched."""
    L = nb.lib
    d = good_desc(nb)
    ok = d.batch
    d.batch = 65536
    need = L.ns_attn_workspace_bytes(ctypes.byref(d))
    out = ctypes.c_void_p(0x90000)
    ptrs = [ctypes.c_void_p(p) for p in (0x10000, 0x20000, 0x30000)]
    assert L.ns_attn_forward(ctypes.byref(d), *ptrs, out, None, None, FAKE, need, None) == nb.NS_ERR_UNSUPPORTED
    assert b"batch" in nb.lib.ns_last_error()
    need = L.cls_scores_workspace_bytes(ctypes.byref(d))
    assert L.cls_scores(ctypes.byref(d), *ptrs[:2], FAKE, FAKE, need, None) == nb.NS_ERR_UNSUPPORTED
    bd = nb.ns_vit_block_desc()
    bd.attn = d
    bd.attn.heads, bd.attn.dtype = 8, nb.NS_BF16
    bd.dim, bd.mlp_dim, bd.ln_eps = 512, 1024, 1e-6
    w = nb.ns_vit_block_weights(*[0x10000] * 12)
    assert L.vit_block_forward(ctypes.byref(bd), ctypes.byref(w), FAKE, out, None, FAKE, 1 << 62, None) == nb.NS_ERR_UNSUPPORTED
    d.batch = ok


def test_kernel_choice_policy(nb, monkeypatch):
    """Which kernel is launched for which problem, both sides of every rule (host logic; without a device the CU count
    defaults to 256)."""
    monkeypatch.delenv("NSATTN_KERNEL", raising=False)

    def desc(B, H, g, block, dtype=None, coords=False, G=1, gw=None):
        d = nb.ns_attn_desc()
        d.batch, d.heads, d.head_dim = B, H, 64
        d.grid_h, d.grid_w = g, gw or g
        d.block, d.radius, d.n_global = block, 1, G
        d.dtype = nb.NS_BF16 if dtype is None else dtype
        d.tokens = G + d.grid_h * d.grid_w if not coords else G + (d.grid_h * d.grid_w) // 2
        d.scale = 0.125
        T = d.tokens
        d.q_stride_b, d.q_stride_h, d.q_stride_t = H * T * 64, T * 64, 64
        d.out_stride_b, d.out_stride_h, d.out_stride_t = H * T * 64, T * 64, 64
        d.coords = 0x40000 if coords else None
        return d

    name = lambda d: nb.lib.ns_attn_patch_kernel_name(ctypes.byref(d)).decode()
    sweep, block16, window, fp32 = "attn_sweep_kernel", "attn_block16_kernel", "attn_mfma_ragged_kernel", "attn_generic_kernel"
    # 8x8 blocks: rows of blocks ("strips") that fill 256 CUs twice over in whole rounds, or nearly, are the sweep's
    assert name(desc(2, 16, 128, 8)) == sweep                           # 512 strips of 16 columns
    assert name(desc(4, 16, 64, 8)) == sweep                            # 512 of 8
    assert name(desc(4, 16, 128, 8)) == sweep                           # 1024 of 16: two rounds
    assert name(desc(3, 24, 160, 8)) == sweep                           # 1440 of 20: 2.8
    assert name(desc(1, 16, 245, 8)) == sweep                           # 496 of 31, short edge blocks
    assert name(desc(1, 16, 128, 8)) == window                          # 256 of 16: one round, half full
    assert name(desc(1, 16, 120, 8)) == window                          # 240: not one per CU
    assert name(desc(3, 16, 88, 8)) == window                           # 528 of 11: a second round for 16
    assert name(desc(3, 24, 64, 8)) == window                           # 576 of 8
    assert name(desc(1, 4, 24, 8)) == window
    assert name(desc(1, 16, 16, 8)) == window
    assert name(desc(1, 2, 8, 8)) == window                             # a single block
    assert name(desc(2, 16, 128, 8, G=2)) == window                     # several global tokens
    assert name(desc(2, 16, 64, 8, G=5)) == window
    # 4x4 and 2x2 blocks, other sides
    assert name(desc(2, 16, 128, 4)) == window
    assert name(desc(1, 16, 245, 2)) == window
    assert name(desc(1, 16, 245, 3)) == window
    assert name(desc(1, 16, 245, 24)) == window                         # no multiple of 16
    # multiples of 16: so many workgroups of 256 queries of a block per CU are the block kernel's: one with 16x16 blocks, else
    # three, or two where the block divides the grid
    assert name(desc(1, 16, 256, 16)) == block16                        # 4096
    assert name(desc(1, 16, 140, 16, gw=144)) == block16                # 1296, short edge blocks
    assert name(desc(1, 16, 120, 16)) == block16                        # 1024, short edge blocks
    assert name(desc(1, 16, 64, 16)) == block16                         # 256
    assert name(desc(1, 16, 64, 16, G=5)) == block16
    assert name(desc(1, 15, 64, 16)) == window                          # 240
    assert name(desc(1, 16, 50, 16, gw=64)) == block16                  # 256: 12 whole blocks, 4 of 2 x 16
    assert name(desc(1, 2, 32, 16)) == window
    assert name(desc(1, 12, 128, 64)) == block16                        # 768
    assert name(desc(1, 8, 128, 64)) == block16                         # 512, no short block
    assert name(desc(1, 7, 128, 64)) == window                          # 448
    assert name(desc(1, 16, 96, 32)) == block16                         # 576, no short block
    assert name(desc(1, 16, 96, 64)) == window                          # 576: 16 + 8 + 8 + 4 an image
    assert name(desc(1, 16, 120, 64)) == block16                        # 912: 16 + 14 + 14 + 13
    assert name(desc(1, 16, 53, 32, gw=128)) == window                  # 448: four of 4 and of 3
    assert name(desc(1, 27, 53, 32, gw=128)) == window                  # 756
    assert name(desc(1, 28, 53, 32, gw=128)) == block16                 # 784
    assert name(desc(1, 16, 245, 16)) == block16
    assert name(desc(1, 16, 245, 32)) == block16
    assert name(desc(1, 16, 245, 64)) == block16
    assert name(desc(1, 16, 256, 16, G=8)) == block16
    assert name(desc(1, 16, 256, 16, G=9)) == window
    # pruned sequences
    assert name(desc(1, 2, 24, 8, coords=True)) == window
    assert name(desc(2, 16, 256, 16, coords=True)) == window
    # fp32; bf16 with a scale or strides that the matrix-instruction kernels do not take
    assert name(desc(1, 2, 24, 8, dtype=nb.NS_F32)) == fp32
    assert name(desc(2, 16, 128, 8, dtype=nb.NS_F32)) == fp32
    d = desc(2, 16, 128, 8)
    d.scale = -0.125
    assert name(d) == fp32
    d = desc(1, 16, 256, 16)
    d.q_stride_t = 16384                                                # 65537 tokens x 32 KB: beyond 31 bits
    assert name(d) == fp32
    monkeypatch.setenv("NSATTN_KERNEL", "lists")
    assert name(desc(2, 16, 128, 8)) == window
    monkeypatch.setenv("NSATTN_KERNEL", "sweep")
    assert name(desc(1, 1, 8, 2, G=8)) == sweep
    monkeypatch.setenv("NSATTN_KERNEL", "generic")
    assert name(desc(1, 16, 100, 8)) == "attn_generic_kernel"
    assert name(desc(2, 16, 128, 8)) == "attn_generic_kernel"
    monkeypatch.setenv("NSATTN_KERNEL", "block")
    assert name(desc(1, 2, 32, 16)) == "attn_block16_kernel"
    assert name(desc(2, 16, 128, 8)) != "attn_block16_kernel"           # a forced kernel that cannot serve falls back
    bad = desc(2, 16, 128, 8)
    bad.heads = 0
    assert name(bad) == ""


def _stack_desc(nb, keep_k, grid=128, block=8):
    d = nb.ns_vit_desc()
    a = d.block.attn
    a.batch, a.heads, a.head_dim = 1, 16, 64
    a.grid_h = a.grid_w = grid
    a.block, a.radius, a.n_global, a.dtype, a.tokens = block, 1, 1, nb.NS_BF16, 1 + grid * grid
    a.scale = 0.125
    d.block.dim, d.block.mlp_dim, d.block.ln_eps = 1024, 4096, 1e-6
    d.layers, d.prune_after, d.keep_k = 4, 2, keep_k
    return d


def test_stack_workspace_covers_the_pruned_blocks(nb):
    """A keep count within a few tokens of the grid size makes the blocks after the pruning stage need
    more workspace (token lists and counts) than the blocks on the full grid: the stack's workspace
    must cover both, for every proportion 0 <= p < 1 of the paper's pruning stage (keep_k = N is p = 0)."""
    N = 128 * 128
    for keep_k in (N, N - 1, N - 3, N - 100, (N * 60 + 99) // 100, 1):
        d = _stack_desc(nb, keep_k)
        total = nb.lib.vit_workspace_bytes(ctypes.byref(d))
        assert total > 0, nb.lib.ns_last_error()
        # the block on the pruned sequence, sized on its own
        pd = nb.ns_vit_block_desc()
        ctypes.memmove(ctypes.byref(pd), ctypes.byref(d.block), ctypes.sizeof(pd))
        pd.attn.tokens = 1 + keep_k
        pd.attn.coords = 0x1000          # never dereferenced on the host
        need_pruned = nb.lib.vit_block_workspace_bytes(ctypes.byref(pd))
        need_full = nb.lib.vit_block_workspace_bytes(ctypes.byref(d.block))
        assert need_pruned > 0 and need_full > 0
        no_prune = _stack_desc(nb, 0)
        base = nb.lib.vit_workspace_bytes(ctypes.byref(no_prune))
        # what the stack adds around a block does not depend on the block's workspace
        assert total - max(need_full, need_pruned) >= base - need_full - 4096
        assert total >= max(need_full, need_pruned)
    # the case that used to fall short: keep_k = N needs more than the full grid
    pd.attn.tokens = 1 + N
    assert nb.lib.vit_block_workspace_bytes(ctypes.byref(pd)) > nb.lib.vit_block_workspace_bytes(ctypes.byref(d.block))


def test_wrong_arguments_are_reported_without_a_device(nb):
    """What is wrong with the arguments comes before the current stream is asked for."""
    import torch
    q = torch.zeros(1, 1, 65, 64, dtype=torch.bfloat16)
    x = torch.zeros(1, 65, 64, dtype=torch.bfloat16)
    with pytest.raises(ValueError):
        nb.ns_attn_forward(q, q[:, :, :3], q, 8, 8, 8)
    with pytest.raises(ValueError):
        nb.ns_attn_forward_scores(q, q.float(), q, 8, 8, 8)
    with pytest.raises(TypeError):
        nb.ns_attn_forward(q, q, q, 8.0, 8, 8)
    with pytest.raises(ValueError):
        nb.cls_scores(q, q[:, :, 1:])
    with pytest.raises(ValueError):
        nb.topk_filter(torch.zeros(1, 3, dtype=torch.float64), 1)
    with pytest.raises(ValueError):
        nb.vit_embed(q, q, q, q, q, 14)
    with pytest.raises(KeyError):
        nb.vit_block_forward(x, {}, 8, 8, 8, 1)
    with pytest.raises(ValueError):
        nb.vit_forward(q, [{}], 8, 8, 8, 1)


def test_weights_that_a_mapping_makes_on_demand_stay_alive(nb):
    """The binding takes pointers out of a block's weights one after the other: each must still be alive when the
    call is made.  (head_dim 32 is refused, so nothing is launched.)"""
    import weakref
    import torch
    dim, mlp = 64, 128
    shapes = {"w_qkv": (3 * dim, dim), "w_proj": (dim, dim), "w_fc1": (mlp, dim), "w_fc2": (dim, mlp), "b_qkv": (3 * dim,),
              "b_fc1": (mlp,)}
    given = []

    class Lazy:
        def __getitem__(self, name):
            assert all(r() is not None for r in given), "a weight was released before %s was read" % name
            t = torch.zeros(shapes.get(name, (dim,)), dtype=torch.bfloat16 if name.startswith("w_") else torch.float32)
            given.append(weakref.ref(t))
            return t

    class Stream:
        cuda_stream = 0

    x = torch.zeros(1, 65, dim, dtype=torch.bfloat16)
    with pytest.raises(nb.NsError):
        nb.vit_block_forward(x, Lazy(), 8, 8, 4, 2, stream=Stream())
    assert len(given) == 13                 # the twelve, and w_fc1 once more for its shape
    assert all(r() is None for r in given)  # and the call keeps none of them
    given.clear()
    with pytest.raises(nb.NsError):
        nb.vit_forward(x, [Lazy(), Lazy()], 8, 8, 4, 2, stream=Stream())
    assert len(given) == 25 and all(r() is None for r in given)
