"""Values that are not finite, and sums that leave fp32's range, in the window kernels and the global rows: a row is
what the patches it attends to make it, whatever stands in the others."""
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


def force(monkeypatch, dtype, split):
    monkeypatch.setenv("NSATTN_KERNEL", ("lists" if dtype == "bf16" else "generic") + split)


def assert_same_values(got, ref, dtype, what):
    """Infinities and NaN at the same places, the rest within the parity bar."""
    for name, test in (("NaN", np.isnan), ("+inf", np.isposinf), ("-inf", np.isneginf)):
        wrong = np.argwhere(test(got) != test(ref))
        assert len(wrong) == 0, "%s: %d values differ in being %s, the first at %s" % (what, len(wrong), name, wrong[0])
    fin = np.isfinite(ref)
    assert_attn_close(np.where(fin, got, 0.0), np.where(fin, ref, 0.0), dtype, what)


def poison(v, G, N, n=3):
    """inf and NaN in a few channels of a few patches; the last patch is the one that stands in for keys past a
    tile's end."""
    p = [N // 3, N // 2 + 1, N // 2 + 2][:n]
    v[0, 1, G + p[0], 5] = np.inf
    v[0, 1, G + p[1 % n], 40] = np.nan
    v[0, 0, G + p[1 % n], 7] = np.inf
    v[0, 0, G + p[2 % n], 7] = -np.inf
    v[0, 0, G + N - 1, 63] = -np.inf
    v[0, 1, G + N - 1, 0] = np.inf


@pytest.mark.parametrize("split", ["1", "2", "4"])
@pytest.mark.parametrize("dtype", ["bf16", "f32", "bf16 in fp32"])
@pytest.mark.parametrize("gh,gw,block,G", [(20, 19, 1, 1), (19, 22, 2, 1), (21, 26, 3, 2), (25, 18, 4, 1), (17, 13, 5, 1), (20, 27, 8, 1),
                                           (37, 21, 16, 1)])
def test_values_that_are_not_finite(nb, monkeypatch, gh, gw, block, G, dtype, split):
    """Block sides 1 to 4 put several blocks into a tile, whose queries then see different keys of it."""
    force(monkeypatch, dtype, split)
    dt = dtype[:4] if dtype.startswith("bf16") else dtype
    q, k, v = synth.small_case(31 + gh * gw, 1, 2, 64, gh, gw, dt, n_global=G)
    poison(v, G, gh * gw)
    print("not finite: grid %dx%d block %d G=%d %s split %s" % (gh, gw, block, G, dtype, split), flush=True)
    out = nb.ns_attn_forward(*(to_dev(a, dt) for a in (q, k, v)), gh, gw, block, 0.125, n_global=G)
    torch.cuda.synchronize()
    ref = oracle.ns_attn(q, k, v, gh, gw, block, 0.125, n_global=G)
    assert not np.isfinite(ref).all() and np.isfinite(ref[:, :, G:]).mean() > 0.9
    assert_same_values(to_np(out), ref, dt, "not finite")


@pytest.mark.parametrize("split", ["1", "2", "4"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("g,block,G", [(24, 8, 1), (20, 3, 2)])
def test_values_that_are_not_finite_in_a_pruned_sequence(nb, monkeypatch, g, block, G, dtype, split):
    force(monkeypatch, dtype, split)
    rng = np.random.default_rng(g)
    kept = rng.permutation(np.flatnonzero(rng.random(g * g) < 0.6))
    q, k, v = synth.small_case(50 + g, 1, 2, 64, 1, len(kept), dtype, n_global=G)
    poison(v, G, len(kept))
    coords = np.ascontiguousarray(synth.raster_coords(g, g)[kept][None])
    print("not finite, pruned: %d of %d, block %d G=%d %s split %s" % (len(kept), g * g, block, G, dtype, split), flush=True)
    out = nb.ns_attn_forward(*(to_dev(a, dtype) for a in (q, k, v)), g, g, block, 0.125, coords=torch.from_numpy(coords).cuda(), n_global=G)
    torch.cuda.synchronize()
    ref = oracle.ns_attn(q, k, v, g, g, block, 0.125, coords=coords, n_global=G)
    assert_same_values(to_np(out), ref, dtype, "not finite, pruned")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_a_global_token_that_is_not_finite(nb, monkeypatch, dtype):
    """Everybody sees it: its channel is lost in every row, and no other."""
    force(monkeypatch, dtype, "")
    G, gh, gw = 2, 18, 21
    q, k, v = synth.small_case(8, 1, 2, 64, gh, gw, dtype, n_global=G)
    v[0, 0, 1, 9] = np.inf
    v[0, 1, 0, 33] = np.nan
    for block in (4, 8):
        out = nb.ns_attn_forward(*(to_dev(a, dtype) for a in (q, k, v)), gh, gw, block, 0.125, n_global=G)
        torch.cuda.synchronize()
        assert_same_values(to_np(out), oracle.ns_attn(q, k, v, gh, gw, block, 0.125, n_global=G), dtype, "global token, block %d" % block)


def high_case(N, first_high, half, dtype, logit=60.5, big=1e14):
    """Patches from number first_high on have logits `logit` above the ones before, values of big up to patch `half`
    and of -big/2 behind it: their weights against the first ones' maximum, times these, are beyond fp32."""
    rnd = synth.round_to_bf16 if dtype == "bf16" else (lambda a: a.astype(np.float32))
    q = np.zeros((1, 2, 1 + N, 64), np.float32)
    k, v = np.zeros_like(q), np.zeros_like(q)
    q[..., 0] = 22.0
    k[:, :, 1 + first_high:, 0] = logit / (0.125 * 22.0)
    v[:, :, 1 + first_high:] = big
    v[:, :, 1 + half:] = -0.5 * big
    return rnd(q), rnd(k), rnd(v)


@pytest.mark.parametrize("split", ["1", "2", "4"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("pruned", [False, True])
@pytest.mark.parametrize("logit,big", [(60.5, 1e14), (5.0, 2e35)])
def test_sums_beyond_the_range(nb, monkeypatch, logit, big, dtype, split, pruned):
    """Finite results whose sums leave fp32's range against the first step's maximum.  60.5 nats above it: some tiles hold
    keys of both signs, and +inf - inf is NaN.  5 nats: weights of 148 are too large for the values though not
    for the sum of weights.  (Weights of at most 1 sum up to 384 x 2e35.)"""
    force(monkeypatch, dtype, split)
    g, block = 24, 8
    q, k, v = high_case(g * g, 8 * g, 16 * g, dtype, logit, big)
    coords = np.ascontiguousarray(synth.raster_coords(g, g)[None]) if pruned else None
    print("sums beyond the range: %g nats, values of %g, %s split %s pruned %s" % (logit, big, dtype, split, pruned), flush=True)
    out = nb.ns_attn_forward(*(to_dev(a, dtype) for a in (q, k, v)), g, g, block, 0.125,
                             coords=None if coords is None else torch.from_numpy(coords).cuda())
    torch.cuda.synchronize()
    got, ref = to_np(out), oracle.ns_attn(q, k, v, g, g, block, 0.125, coords=coords)
    assert np.isfinite(got).all()
    assert_attn_close(got / big, ref / big, dtype, "sums beyond the range")


@pytest.mark.parametrize("kernel,gh,gw,block", [("sweep", 24, 24, 8), ("sweep", 20, 27, 8), ("block", 48, 48, 16), ("block", 40, 41, 16)])
def test_sums_that_cancel_in_the_tiled_kernels(nb, monkeypatch, kernel, gh, gw, block):
    """As above, 60.5 nats, in the kernels whose waves walk a tile's keys block after block."""
    monkeypatch.setenv("NSATTN_KERNEL", kernel)
    q, k, v = high_case(gh * gw, block * gw, 2 * block * gw, "bf16")
    out = nb.ns_attn_forward(*(to_dev(a, "bf16") for a in (q, k, v)), gh, gw, block, 0.125)
    torch.cuda.synchronize()
    got, ref = to_np(out), oracle.ns_attn(q, k, v, gh, gw, block, 0.125)
    assert np.isfinite(got).all()
    assert_attn_close(got / 1e14, ref / 1e14, "bf16", "cancelling sums, %s" % kernel)


@pytest.mark.parametrize("split", ["1", "2", "4"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("pruned,g,block", [(True, 24, 8), (True, 33, 16), (False, 24, 8), (False, 33, 16)])
def test_weights_beyond_the_first_steps_reference(nb, monkeypatch, dtype, split, pruned, g, block):
    """The second walk, with the token ring and without: every query's largest logit lies more than 2^100 above
    those of a wave's first step (32 keys; the walk starts over where a sum exceeds 1e30)."""
    force(monkeypatch, dtype, split)
    rng = np.random.default_rng(g)
    N = g * g
    q, k, v = synth.small_case(60 + g, 1, 2, 64, g, g, dtype)
    q = q * np.float32(12.0)
    # keys in raster order: small ones in the first eight rows of the grid, then large ones
    k[:, :, 1:1 + 8 * g] *= np.float32(0.05)
    if dtype == "bf16":
        q, k = synth.round_to_bf16(q), synth.round_to_bf16(k)
    coords = np.ascontiguousarray(synth.raster_coords(g, g)[None]) if pruned else None
    # the tile of the grid's middle block: it sees the rows of three blocks
    mid = (g // 2 // block) * block
    lo = max(mid - block, 0)
    qm = q[:, :, 1 + mid * g + mid].astype(np.float64)
    logits = np.einsum("bhd,bhtd->bht", qm, k.astype(np.float64)) / np.log(2.0)
    small = np.r_[0, 1 + lo * g:1 + 8 * g]
    assert lo < 8 and (logits.max(-1) - logits[..., small].max(-1)).min() > 110
    print("second walk: %d block %d %s split %s pruned %s" % (g, block, dtype, split, pruned), flush=True)
    out = nb.ns_attn_forward(*(to_dev(a, dtype) for a in (q, k, v)), g, g, block, 1.0,
                             coords=None if coords is None else torch.from_numpy(coords).cuda())
    torch.cuda.synchronize()
    ref = oracle.ns_attn(q, k, v, g, g, block, 1.0, coords=coords)
    got = to_np(out)
    assert np.isfinite(got).all()
    if dtype == "f32":
        # a logit of size L carries L * 2^-24 per product and so does its weight: 64 products of up to 150
        assert np.abs(got - ref).max() <= 1e-3
    else:
        assert_attn_close(got, ref, dtype, "second walk")


@pytest.mark.parametrize("split", ["1", "2", "4"])
@pytest.mark.parametrize("gh,gw,block,G", [(21, 26, 3, 2), (20, 27, 8, 1)])
def test_keys_that_are_not_finite_in_fp32(nb, monkeypatch, gh, gw, block, G, split):
    """A key with -inf where every query is positive counts for nothing; one with +inf makes the rows NaN whose query is positive
    there.  (The fp32 products work on parts of a value, and those of an infinite one are NaN.)"""
    force(monkeypatch, "f32", split)
    N = gh * gw
    q, k, v = synth.small_case(7 + N, 1, 2, 64, gh, gw, "f32", n_global=G)
    q[:, :, :, 7] = np.abs(q[:, :, :, 7]) + np.float32(0.1)
    k[0, 1, G + N // 2, 7] = -np.inf
    k[0, 1, G + N - 1, 7] = -np.inf
    k[0, 0, G + N // 3, 9] = np.inf
    print("keys not finite: grid %dx%d block %d G=%d split %s" % (gh, gw, block, G, split), flush=True)
    out = nb.ns_attn_forward(*(to_dev(a, "f32") for a in (q, k, v)), gh, gw, block, 0.125, n_global=G)
    torch.cuda.synchronize()
    ref = oracle.ns_attn(q, k, v, gh, gw, block, 0.125, n_global=G)
    assert np.isfinite(ref[0, 1]).all() and not np.isfinite(ref[0, 0]).all() and np.isfinite(ref[0, 0]).any()
    assert_same_values(to_np(out), ref, "f32", "keys not finite")


@pytest.mark.parametrize("pruned", [False, True])
@pytest.mark.parametrize("G", [1, 3, 40])
@pytest.mark.parametrize("dtype,what", [("f32", "-inf"), ("f32", "large"), ("f32", "query"), ("bf16 in fp32", "-inf"), ("bf16 in fp32", "query")])
def test_by_products_of_keys_that_are_not_finite_in_fp32(nb, monkeypatch, dtype, what, G, pruned):
    """Logits, log-sum-exps and scores beside the rows, by every route.  A key whose logit is -inf has the weight 0 and is nobody else's
    business.  large: finite values that bf16 rounds to infinity.  query: an infinite value in a global token's row, whose
    logits are infinities of either sign (its log-sum-exp and the scores of its image are NaN).  bf16 rows are computed in
    fp32 where the scale is negative.  A run of 40 such keys is a wave's whole first step."""
    monkeypatch.delenv("NSATTN_KERNEL", raising=False)
    dt, scale = (dtype, 0.125) if dtype == "f32" else ("bf16", -0.125)
    gh, gw, block, H = 26, 27, 8, 2
    rng = np.random.default_rng(G)
    kept = np.flatnonzero(rng.random(gh * gw) < 0.8) if pruned else np.arange(gh * gw)
    N = len(kept)
    q, k, v = synth.small_case(900 + G, 2, H, 64, 1, N, dt, n_global=G)
    q[:, :, :, 7] = np.maximum(np.abs(q[:, :, :, 7]), np.float32(0.125))
    if what == "query":
        q[0, 1, G - 1, 9] = np.inf
    else:
        bad = np.float32({"-inf": -np.inf, "large": -3.4e38}[what] * np.sign(scale))
        k[0, 1, G + N // 2, 7] = bad                    # one head's
        k[0, :, G + N // 3, 7] = bad                    # all heads'
        k[1, 0, G + 96:G + 136, 7] = bad
        k[1, 1, G + N - 1, 7] = bad                     # the last token stands in for keys past the end
    coords = np.ascontiguousarray(np.broadcast_to(synth.raster_coords(gh, gw)[kept], (2, N))) if pruned else None
    print("by-products: %s %s G=%d pruned %s" % (dtype, what, G, pruned), flush=True)
    dq, dk, dv = (to_dev(a, dt) for a in (q, k, v))
    dc = None if coords is None else torch.from_numpy(coords).cuda()
    out, logits, lse = nb.ns_attn_forward(dq, dk, dv, gh, gw, block, scale, coords=dc, want_cls=True, n_global=G)
    out2, logits2, lse2, scores = nb.ns_attn_forward_scores(dq, dk, dv, gh, gw, block, scale, coords=dc, n_global=G)
    alone, later = nb.cls_scores(dq, dk, scale, n_global=G), nb.cls_scores_from_logits(logits, lse, n_global=G)
    torch.cuda.synchronize()
    with np.errstate(invalid="ignore"):
        s = scale * np.einsum("bhgd,bhtd->bhgt", q[:, :, :G].astype(np.float64), k.astype(np.float64))
        m = s.max(axis=-1, keepdims=True)
        ref_lse = (m + np.log(np.exp(s - m).sum(axis=-1, keepdims=True)))[..., 0]
        ref, ref_scores = oracle.ns_attn(q, k, v, gh, gw, block, scale, coords=coords, n_global=G), oracle.cls_scores(q, k, scale, n_global=G)
    assert not np.isnan(s).any() and np.isfinite(ref_lse).all() == np.isfinite(ref_scores).all() == (what != "query")
    assert not np.isfinite(s).all() or np.abs(s).max() > 1e36
    assert_same_values(to_np(out), ref, dt, "rows")
    # (the bounds that these values have where all keys are finite; 2^-20 of a logit where it is large)
    np.testing.assert_allclose(to_np(logits).reshape(s.shape), s, rtol=2.0 ** -20, atol=2e-5)
    np.testing.assert_allclose(to_np(lse).reshape(ref_lse.shape), ref_lse, rtol=0, atol=2e-5)
    for name, got in (("with the attention", scores), ("by itself", alone), ("from the logits", later)):
        np.testing.assert_allclose(to_np(got), ref_scores, rtol=5e-5, atol=1e-10, err_msg=name)
    same = lambda a, b: torch.equal(torch.nan_to_num(a), torch.nan_to_num(b)) and torch.equal(a.isnan(), b.isnan())
    assert same(out, out2) and same(logits, logits2) and same(lse, lse2)
