"""The window kernels (a query tile's keys shared out over 1, 2 or 4 waves; global rows in the same
launch) at the sizes where their bookkeeping can go wrong, each split forced in turn."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_12150_amd import synth
from _util import assert_attn_close, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nb():
    from paper_2601_12150_amd import binding
    return binding


# (grid_h, grid_w, block, global tokens, gain): one key step for four waves, one step each, a step more than the
# ring has slots, tiles of a single query, squares of several blocks (side 1, 2, 3, 4), a query tile whose
# first keys it may not see, global tokens in one and in two groups, peaked rows (25x18: beyond the fixed reference; the
# second walk by itself is tested in test_gpu_nonfinite.py)
SHAPES = [(1, 1, 8, 1, 1.0), (5, 6, 8, 1, 1.0), (11, 11, 8, 7, 1.0), (12, 24, 8, 1, 1.0), (9, 17, 8, 2, 1.0), (13, 15, 5, 3, 1.0),
          (10, 11, 1, 1, 1.0), (20, 19, 2, 1, 1.0), (14, 13, 3, 5, 1.0), (25, 18, 4, 1, 14.0), (7, 33, 7, 17, 1.0), (18, 20, 16, 33, 1.0),
          (33, 17, 12, 1, 14.0), (16, 40, 64, 1, 1.0)]


@pytest.mark.parametrize("split", ["1", "2", "4"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("gh,gw,block,G,gain", SHAPES)
def test_complete_grid(nb, monkeypatch, gh, gw, block, G, gain, dtype, split):
    monkeypatch.setenv("NSATTN_KERNEL", ("lists" if dtype == "bf16" else "generic") + split)
    q, k, v = synth.small_case(900 + gh * gw, 2, 3, 64, gh, gw, dtype, n_global=G)
    q = synth.round_to_bf16(q * gain) if dtype == "bf16" else q * np.float32(gain)
    print("grid %dx%d block %d G=%d %s split %s" % (gh, gw, block, G, dtype, split), flush=True)
    out, logits, lse, scores = nb.ns_attn_forward_scores(*(to_dev(a, dtype) for a in (q, k, v)), gh, gw, block, 0.125, n_global=G)
    torch.cuda.synchronize()
    assert np.isfinite(to_np(out)).all()
    assert_attn_close(to_np(out), oracle.ns_attn(q, k, v, gh, gw, block, 0.125, n_global=G), dtype, "window kernel")
    # by-products: fp32 sums of 64 exact products of size gain, a softmax of them (twice a logit's error)
    ref_logits = 0.125 * np.einsum("bhgd,bhtd->bhgt", q[:, :, :G].astype(np.float64), k.astype(np.float64))
    m = ref_logits.max(axis=-1, keepdims=True)
    ref_lse = (m + np.log(np.exp(ref_logits - m).sum(axis=-1, keepdims=True)))[..., 0]
    np.testing.assert_allclose(to_np(logits).reshape(ref_logits.shape), ref_logits, rtol=0, atol=2e-5 * gain)
    np.testing.assert_allclose(to_np(lse).reshape(ref_lse.shape), ref_lse, rtol=0, atol=2e-5 * gain)
    np.testing.assert_allclose(to_np(scores), oracle.cls_scores(q, k, 0.125, n_global=G), rtol=5e-5 * gain, atol=1e-10)


@pytest.mark.parametrize("split", ["1", "2", "4"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("g,block,keep,G", [(24, 8, 0.6, 1), (40, 8, 0.05, 5), (33, 16, 0.7, 1), (20, 3, 0.5, 2)])
def test_pruned_sequence(nb, monkeypatch, g, block, keep, G, dtype, split):
    """Lists with empty blocks (a workgroup's other tile then waits for a wave without work), blocks with one
    token, and survivors in no order."""
    monkeypatch.setenv("NSATTN_KERNEL", ("lists" if dtype == "bf16" else "generic") + split)
    rng = np.random.default_rng(g + block)
    alive = rng.random(g * g) < keep
    r, c = np.divmod(np.arange(g * g), g)
    alive[(r // block == 0) & (c // block == 0)] = False
    kept = rng.permutation(np.flatnonzero(alive))
    q, k, v = synth.small_case(70 + g, 2, 2, 64, 1, len(kept), dtype, n_global=G)
    coords = np.ascontiguousarray(np.broadcast_to(synth.raster_coords(g, g)[kept], (2, len(kept))))
    print("pruned %d of %d, block %d G=%d %s split %s" % (len(kept), g * g, block, G, dtype, split), flush=True)
    out = nb.ns_attn_forward(*(to_dev(a, dtype) for a in (q, k, v)), g, g, block, 0.125, coords=torch.from_numpy(coords).cuda(),
                             n_global=G)
    torch.cuda.synchronize()
    ref = oracle.ns_attn(q, k, v, g, g, block, 0.125, coords=coords, n_global=G)
    assert_attn_close(to_np(out), ref, dtype, "window kernel, pruned sequence")


@pytest.mark.parametrize("gh,gw,gain", [(16, 16, 1.0), (16, 32, 1.0), (17, 31, 1.0), (33, 31, 14.0), (64, 48, 1.0)])
def test_global_row_in_a_launch_of_its_own(nb, monkeypatch, gh, gw, gain):
    """The block kernel leaves the global row to another launch: fewer keys than a chunk (257), one over a chunk
    (513), one over two (1024 + 1), the last chunk partly filled; peaked rows."""
    monkeypatch.setenv("NSATTN_KERNEL", "block")
    q, k, v = synth.small_case(40 + gw, 2, 3, 64, gh, gw, "bf16")
    q = synth.round_to_bf16(q * gain)
    print("global row, grid %dx%d gain %g" % (gh, gw, gain), flush=True)
    out, logits, lse, scores = nb.ns_attn_forward_scores(*(to_dev(a, "bf16") for a in (q, k, v)), gh, gw, 16, 0.125)
    alone = nb.ns_attn_forward(*(to_dev(a, "bf16") for a in (q, k, v)), gh, gw, 16, 0.125)
    torch.cuda.synchronize()
    assert torch.equal(out, alone)
    assert_attn_close(to_np(out), oracle.ns_attn(q, k, v, gh, gw, 16, 0.125), "bf16", "global row")
    ref_logits = 0.125 * np.einsum("bhd,bhtd->bht", q[:, :, 0].astype(np.float64), k.astype(np.float64))
    m = ref_logits.max(axis=-1, keepdims=True)
    ref_lse = (m + np.log(np.exp(ref_logits - m).sum(axis=-1, keepdims=True)))[..., 0]
    np.testing.assert_allclose(to_np(logits).reshape(ref_logits.shape), ref_logits, rtol=0, atol=2e-5 * gain)
    np.testing.assert_allclose(to_np(lse).reshape(ref_lse.shape), ref_lse, rtol=0, atol=2e-5 * gain)
    np.testing.assert_allclose(to_np(scores), oracle.cls_scores(q, k, 0.125), rtol=5e-5 * gain, atol=1e-10)


@pytest.mark.parametrize("g,block,B,n", [(64, 8, 8, 2457), (64, 8, 9, 2457), (92, 8, 1, 8193), (92, 2, 1, 5001), (72, 1, 1, 4097), (72, 1, 1, 4096)])
def test_block_lists_of_few_and_of_many_blocks(nb, monkeypatch, g, block, B, n):
    """Up to two blocks per CU (512) and more than that take other numbers of waves per block; one to three rounds of 4096 coordinates,
    the last of one or of all; survivors in no order."""
    monkeypatch.setenv("NSATTN_KERNEL", "lists")
    rng = np.random.default_rng(n)
    kept = np.stack([rng.permutation(g * g)[:n] for _ in range(B)])
    q, k, v = synth.small_case(n, B, 1, 64, 1, n, "bf16")
    coords = np.ascontiguousarray(synth.raster_coords(g, g)[kept])
    out = nb.ns_attn_forward(*(to_dev(a, "bf16") for a in (q, k, v)), g, g, block, 0.125, coords=torch.from_numpy(coords).cuda())
    torch.cuda.synchronize()
    at = [0, B - 1] if B > 1 else [0]
    rows = np.unique(np.concatenate([[0, 1, n], 1 + rng.integers(0, n, 500)]))
    ref = oracle.ns_attn(q[at], k[at], v[at], g, g, block, 0.125, coords=np.ascontiguousarray(coords[at]), rows=rows)
    assert_attn_close(to_np(out)[at][:, :, rows], ref, "bf16", "%d blocks" % (-(-g // block)) ** 2)
