"""Places where fp32 weights show through the rounding of the result."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_12150_amd import synth
from _util import to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nb():
    from paper_2601_12150_amd import binding
    return binding


@pytest.mark.parametrize("split", ["1", "2", "4"])
@pytest.mark.parametrize("G", [1, 5, 8])
@pytest.mark.parametrize("pruned,g,block,strong", [(False, 24, 8, False), (False, 21, 3, False), (True, 24, 8, False),
                                                   (False, 24, 8, True), (True, 24, 8, True)])
def test_a_global_tokens_weight_is_not_rounded(nb, monkeypatch, pruned, g, block, strong, G, split):
    """Global token c has the value 1 in channel c and patches have none: a patch row's channel c is one weight, and
    the one bf16 rounding is that of the result: at most 2^-8 of it.  (A weight rounded to bf16 as well: up to 2^-7.)
    strong: some queries of every tile have logits beyond the first step's reference, so the tile is walked again."""
    monkeypatch.setenv("NSATTN_KERNEL", "lists" + split)
    N = g * g
    q, k, v = synth.small_case(300 + g + G, 1, 2, 64, g, g, "bf16", n_global=G)
    v[:] = 0
    rows = np.arange(N) % 29 != 3
    if strong:
        q[:, :, G:][:, :, ~rows] *= 64.0
    for c in range(G):
        v[:, :, c, c] = 1.0
    coords = np.ascontiguousarray(synth.raster_coords(g, g)[None]) if pruned else None
    print("global weight: %d block %d G=%d split %s pruned %s strong %s" % (g, block, G, split, pruned, strong), flush=True)
    out = nb.ns_attn_forward(*(to_dev(a, "bf16") for a in (q, k, v)), g, g, block, 0.125, n_global=G,
                             coords=None if coords is None else torch.from_numpy(coords).cuda())
    torch.cuda.synchronize()
    ref = oracle.ns_attn(q, k, v, g, g, block, 0.125, n_global=G, coords=coords)[:, :, G:][:, :, rows, :G]
    err = np.abs(to_np(out)[:, :, G:][:, :, rows, :G] - ref) / ref
    # 2^-8 for the result, 64 products and N weights summed in fp32
    assert err.max() <= 2.0 ** -8 + 1e-5, "largest relative error %.3g" % err.max()
