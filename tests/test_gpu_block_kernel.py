"""The block kernel's numbering of queries and keys (raster order within the block and within the rectangle that its 3x3
blocks cover, 64 keys a tile, 64 queries a wave) and the row sums that the matrix instructions form."""
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


# rectangles of 1 to 5 tiles (fewer than the ring has slots) and of many, last tiles of 1, 63 and 64 keys, rectangles
# narrower than, as wide as and wider than a tile's 64 keys; blocks whose last wave has one query and waves with none;
# one, two, three and four blocks a side in either direction
@pytest.mark.parametrize("gh,gw,block,G", [
    (1, 1, 16, 1), (1, 65, 16, 1), (65, 1, 16, 2), (7, 9, 16, 1), (8, 8, 16, 1), (13, 5, 16, 8), (16, 16, 16, 1), (17, 15, 16, 1),
    (31, 33, 16, 3), (32, 96, 32, 1), (63, 65, 32, 1), (64, 21, 48, 1), (97, 33, 32, 2), (50, 145, 48, 1), (128, 20, 64, 1),
    (70, 200, 64, 5)])
def test_numbering(nb, monkeypatch, gh, gw, block, G):
    monkeypatch.setenv("NSATTN_KERNEL", "block")
    q, k, v = synth.small_case(gh * 300 + gw, 2, 2, 64, gh, gw, "bf16", n_global=G)
    dq, dk, dv = (to_dev(a, "bf16") for a in (q, k, v))
    assert nb.ns_attn_patch_kernel_name(dq, gh, gw, block, n_global=G) == "attn_block16_kernel"
    print("block kernel: %dx%d block %d G=%d" % (gh, gw, block, G), flush=True)
    out = nb.ns_attn_forward(dq, dk, dv, gh, gw, block, 0.125, n_global=G)
    torch.cuda.synchronize()
    assert_attn_close(to_np(out), oracle.ns_attn(q, k, v, gh, gw, block, 0.125, n_global=G), "bf16", "numbering")


# (the sweep forms its sums like the others on grids that 8 divides, with and without masked keys, and lane by lane on others)
@pytest.mark.parametrize("force,g,block", [("lists1", 24, 8), ("lists2", 24, 8), ("lists4", 33, 16), ("block", 33, 16), ("block", 48, 16),
                                           ("sweep", 24, 8), ("sweep", 27, 8), ("sweep", 24, 4), ("sweep", 27, 2)])
def test_a_row_that_is_not_finite_stays_alone(nb, monkeypatch, force, g, block):
    """The matrix instruction that sums a fragment's weights takes two queries' lanes and multiplies one by 0: a row whose
    weights are NaN (its query is) or infinite must not reach the other's sum."""
    monkeypatch.setenv("NSATTN_KERNEL", force)
    q, k, v = synth.small_case(g, 1, 2, 64, g, g, "bf16")
    bad = [1 + 5, 1 + 3 * g + 17, 1 + g * g - 1]
    q2 = q.copy()
    q2[:, :, bad] = np.nan
    q2[:, :, 1 + 9 * g:1 + 10 * g:3] *= 1e4           # weights beyond fp32's range with the first reference
    print("rows that are not finite: %s %d block %d" % (force, g, block), flush=True)
    out = to_np(nb.ns_attn_forward(*(to_dev(a, "bf16") for a in (q2, k, v)), g, g, block, 0.125))
    torch.cuda.synchronize()
    q2[:, :, bad] = 0.0
    ref = oracle.ns_attn(synth.round_to_bf16(q2), k, v, g, g, block, 0.125)
    assert np.isnan(out[:, :, bad]).all()
    rest = np.setdiff1d(np.arange(1 + g * g), bad)
    assert_attn_close(out[:, :, rest], ref[:, :, rest], "bf16", "other rows")
