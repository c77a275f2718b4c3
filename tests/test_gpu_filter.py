"""GPU parity: cls_scores, cls_scores_from_logits and topk_filter against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_12150_amd import synth
from _util import assert_kept_sets_match, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nb():
    from paper_2601_12150_amd import binding
    return binding


@pytest.mark.parametrize("dtype,g,B,H", [("bf16", 24, 2, 16), ("f32", 28, 1, 16), ("bf16", 45, 3, 5),
                                         ("f32", 7, 2, 3), ("bf16", 1, 1, 1)])
def test_cls_scores_standalone_and_fused(nb, dtype, g, B, H):
    q, k, v = synth.small_case(61, B, H, 64, g, g, dtype)
    ref = oracle.cls_scores(q, k, 0.125)
    dq, dk, dv = (to_dev(a, dtype) for a in (q, k, v))
    got = nb.cls_scores(dq, dk, 0.125)
    # scores are O(1/T); fp32 arithmetic on exact inputs: relative error ~1e-6
    np.testing.assert_allclose(to_np(got), ref, rtol=2e-5, atol=1e-9)
    # the same numbers from the attention call's by-products
    _, logits, lse = nb.ns_attn_forward(dq, dk, dv, g, g, 4, 0.125, want_cls=True)
    fused = nb.cls_scores_from_logits(logits, lse)
    torch.cuda.synchronize()
    np.testing.assert_allclose(to_np(fused), ref, rtol=2e-5, atol=1e-9)


@pytest.mark.parametrize("dtype,g,block,B,H,G,force", [
    ("bf16", 24, 8, 2, 16, 1, "sweep"), ("bf16", 48, 16, 1, 4, 1, "block"), ("bf16", 30, 5, 2, 3, 1, None),
    ("f32", 28, 7, 1, 16, 1, None), ("bf16", 37, 8, 1, 2, 1, "sweep"), ("bf16", 20, 4, 2, 3, 3, None),
    ("bf16", 1, 8, 1, 1, 1, None)])
def test_attention_and_scores_in_one_call(nb, monkeypatch, dtype, g, block, B, H, G, force):
    """ns_attn_forward_scores: the attention outputs and by-products are bit-equal to
    ns_attn_forward's, and the scores (merged and computed in one launch) match the oracle."""
    if force:
        monkeypatch.setenv("NSATTN_KERNEL", force)
    if G == 1:
        q, k, v = synth.small_case(62, B, H, 64, g, g, dtype)
    else:
        rng = np.random.default_rng(62)
        shape = (B, H, G + g * g, 64)
        q, k, v = (synth.round_to_bf16(rng.standard_normal(shape).astype(np.float32)) for _ in range(3))
    ref = oracle.cls_scores(q, k, 0.125, n_global=G) if G > 1 else oracle.cls_scores(q, k, 0.125)
    dq, dk, dv = (to_dev(a, dtype) for a in (q, k, v))
    out, logits, lse, scores = nb.ns_attn_forward_scores(dq, dk, dv, g, g, block, 0.125, n_global=G)
    out2, logits2, lse2 = nb.ns_attn_forward(dq, dk, dv, g, g, block, 0.125, want_cls=True, n_global=G)
    torch.cuda.synchronize()
    assert torch.equal(out, out2) and torch.equal(logits, logits2) and torch.equal(lse, lse2)
    np.testing.assert_allclose(to_np(scores), ref, rtol=2e-5, atol=1e-9)


def topk_case(nb, scores, k):
    ref = oracle.topk(scores, k)
    kept, _, _ = nb.topk_filter(torch.from_numpy(scores).cuda(), k)
    torch.cuda.synchronize()
    assert np.array_equal(kept.cpu().numpy(), ref)


@pytest.mark.parametrize("N,k", [(1, 1), (7, 3), (64, 64), (1000, 377), (1024, 1), (4096, 2458),
                                 (16384, 9831), (65536, 26215), (70001, 35000)])
def test_topk_random_scores_bit_exact(nb, N, k):
    rng = np.random.default_rng(N + k)
    topk_case(nb, rng.random((3, N)).astype(np.float32), k)


def test_topk_ties_signs_and_clusters(nb):
    rng = np.random.default_rng(9)
    # heavy exact ties: the lower index must win
    topk_case(nb, rng.integers(0, 5, size=(2, 5000)).astype(np.float32), 1234)
    # all equal
    topk_case(nb, np.full((2, 3000), 0.25, np.float32), 1000)
    # negative, zero, minus zero, denormals, infinities
    s = rng.standard_normal((2, 4000)).astype(np.float32)
    s[:, ::7] = 0.0
    s[:, 3::7] = -0.0
    s[:, 5::11] = 1e-40
    s[0, 17] = np.inf
    s[1, 23] = -np.inf
    for k in (1, 500, 2000, 3999, 4000):
        topk_case(nb, s, k)
    # clustered like the background tokens: most keys share their leading digits
    c = (1e-4 * (1.0 + 1e-3 * rng.standard_normal((2, 16384)))).astype(np.float32)
    c[:, :6000] = rng.random((2, 6000)).astype(np.float32) * 2e-4
    topk_case(nb, c, 9831)


@pytest.mark.parametrize("N", [16385, 17408, 32768, 32769, 60025, 65536, 65537, 131072, 131073, 300000])
def test_topk_long_rows(nb, N):
    """Rows of up to 32768 scores are selected in one launch, each workgroup of an image from all of its keys, up to 32 per
    thread, longer ones by several workgroups that exchange digit histograms between
    launches: random, tied, clustered and signed scores, k from 1 to N, the coordinates compacted
    along."""
    rng = np.random.default_rng(N)
    topk_case(nb, rng.random((2, N)).astype(np.float32), (N * 6) // 10)
    topk_case(nb, rng.integers(0, 4, size=(2, N)).astype(np.float32), N // 3)          # heavy ties across chunks
    topk_case(nb, np.full((1, N), 0.5, np.float32), N // 2)                              # all equal
    c = (1e-5 * (1.0 + 1e-3 * rng.standard_normal((2, N)))).astype(np.float32)          # clustered
    c[:, : N // 3] = rng.random((2, N // 3)).astype(np.float32) * 2e-5
    topk_case(nb, c, (N * 6) // 10)
    s = rng.standard_normal((2, N)).astype(np.float32)
    s[:, ::7] = 0.0
    s[:, 3::7] = -0.0
    s[0, 17] = np.inf
    s[1, N - 1] = -np.inf
    for k in (1, 2, N // 2, N - 1, N):
        topk_case(nb, s, k)
    coords = rng.integers(0, 2 ** 31 - 1, size=(2, N), dtype=np.int32)
    kept, _, cout = nb.topk_filter(torch.from_numpy(c).cuda(), N // 5, coords=torch.from_numpy(coords).cuda())
    torch.cuda.synchronize()
    ref = oracle.topk(c, N // 5)
    assert np.array_equal(kept.cpu().numpy(), ref)
    assert np.array_equal(cout.cpu().numpy(), np.take_along_axis(coords, ref.astype(np.int64), axis=1))


@pytest.mark.parametrize("N", [70, 4096, 5000, 8192, 16384, 20001, 32768])
def test_topk_ties_and_wide_ranges(nb, N):
    """What the short-row selection decides on the way: the k-th score more than 16 octaves below the largest one, or right at
    that border; more equal scores than it ranks against each other, the k-th among them, above them and below them."""
    rng = np.random.default_rng(N + 1)
    u = (1.0 + rng.random((2, N))).astype(np.float32)
    wide = u * np.float32(2.0) ** rng.integers(-40, 0, size=(2, N)).astype(np.float32)
    tiny = u * np.float32(1e-30)                                # most scores far below a few large ones
    tiny[:, ::16] = u[:, ::16]
    border = u * np.float32(2.0) ** rng.integers(-17, -14, size=(2, N)).astype(np.float32)
    border[:, N // 3] = 1.9999999
    denormal = (u * np.float32(1e-39)).astype(np.float32)       # (all of one row, half of the other)
    denormal[1, ::2] = 0.25
    half = u.copy()
    half[:, rng.permutation(N)[: N // 2]] = 1.5                 # half of them equal
    two = np.float32(2.0) ** rng.integers(0, 2, size=(2, N)).astype(np.float32)
    zero = u * (rng.random((2, N)) < 0.4).astype(np.float32)    # 60 % are zero
    levels = (rng.integers(0, 40, size=(2, N)) / 40.0 + 1.0).astype(np.float32)
    signed = rng.standard_normal((2, N)).astype(np.float32)
    signed[:, rng.permutation(N)[: N // 2]] = -0.25
    for s in (wide, tiny, border, denormal, half, two, zero, levels, signed, np.zeros((2, N), np.float32)):
        for k in {1, N // 16, N // 4, N // 2, (6 * N) // 10, (9 * N) // 10, N - 1, N}:
            topk_case(nb, s, k)


def test_gather_and_coords_compaction_bit_exact(nb):
    rng = np.random.default_rng(4)
    B, N, C, k = 2, 500, 1024, 301
    scores = rng.random((B, N)).astype(np.float32)
    xbits = rng.integers(0, 2 ** 16, size=(B, 1 + N, C), dtype=np.uint16)     # arbitrary bf16 bit patterns
    x = torch.from_numpy(xbits.view(np.int16)).cuda().view(torch.bfloat16)
    coords = rng.integers(0, 2 ** 31 - 1, size=(B, N), dtype=np.int32)
    kept, y, cout = nb.topk_filter(torch.from_numpy(scores).cuda(), k, x=x, coords=torch.from_numpy(coords).cuda())
    torch.cuda.synchronize()
    ref_kept = oracle.topk(scores, k)
    assert np.array_equal(kept.cpu().numpy(), ref_kept)
    ybits = y.view(torch.int16).cpu().numpy().view(np.uint16)
    assert np.array_equal(ybits, oracle.gather(xbits, ref_kept))
    assert np.array_equal(cout.cpu().numpy(), np.take_along_axis(coords, ref_kept.astype(np.int64), axis=1))
    # fp32 rows
    xf = rng.standard_normal((B, 1 + N, 68)).astype(np.float32)
    _, yf, _ = nb.topk_filter(torch.from_numpy(scores).cuda(), k, x=torch.from_numpy(xf).cuda())
    torch.cuda.synchronize()
    assert np.array_equal(yf.cpu().numpy(), oracle.gather(xf, ref_kept))


@pytest.mark.parametrize("B,N,keep,G,C,dtype,clustered", [
    (1, 16384, 9831, 1, 64, "bf16", False),     # 16 workgroups
    (2, 4096, 2458, 5, 1024, "bf16", True),     # four keys per thread, all kept rows in one half of the row
    (3, 4097, 1230, 1, 520, "bf16", True),      # eight keys per thread, unaligned score rows
    (1, 32768, 32768, 3, 8, "bf16", False),     # everything is kept, 32 keys per thread
    (128, 300, 150, 2, 8, "bf16", False),       # two workgroups per image
    (129, 300, 150, 2, 8, "bf16", True),        # one
    (2, 50, 7, 9, 24, "f32", False),            # fewer outputs than one workgroup's least
    (1, 1, 1, 1, 4, "f32", False)])
def test_selection_by_several_workgroups(nb, B, N, keep, G, C, dtype, clustered):
    """Edges of the ranges of outputs that an image's workgroups place; exact."""
    rng = np.random.default_rng(B * 1000 + N)
    scores = rng.random((B, N)).astype(np.float32)
    if clustered:
        scores[:, : N // 2] = 0.125 + 1e-6 * scores[:, : N // 2]      # near ties
        scores[:, N // 2::5] = 0.75                                   # exact ones
    bits = np.uint16 if dtype == "bf16" else np.uint32
    x = rng.integers(0, np.iinfo(bits).max, size=(B, G + N, C), dtype=bits, endpoint=True)
    signed = x.view(np.int16 if dtype == "bf16" else np.int32)
    dx = torch.from_numpy(signed).cuda().view(torch.bfloat16 if dtype == "bf16" else torch.float32)
    coords = rng.integers(0, 2 ** 31 - 1, size=(B, N), dtype=np.int32)
    y = torch.empty((B, G + keep, C), dtype=dx.dtype, device="cuda")
    kept, y, cout = nb.topk_filter(torch.from_numpy(scores).cuda(), keep, x=dx, y=y, coords=torch.from_numpy(coords).cuda(),
                                   n_global=G)
    torch.cuda.synchronize()
    ref = oracle.topk(scores, keep)
    assert np.array_equal(kept.cpu().numpy(), ref)
    assert np.array_equal(cout.cpu().numpy(), np.take_along_axis(coords, ref.astype(np.int64), axis=1))
    want = np.concatenate([x[:, :G], np.take_along_axis(x[:, G:], ref.astype(np.int64)[:, :, None], axis=1)], axis=1)
    assert np.array_equal(y.view(torch.int16 if dtype == "bf16" else torch.int32).cpu().numpy().view(bits), want)


def test_scores_to_kept_set_end_to_end(nb):
    g = 40
    q, k, v = synth.small_case(77, 2, 16, 64, g, g, "bf16")
    ref_scores = oracle.cls_scores(q, k, 0.125)
    kk = (g * g * 60 + 99) // 100
    ref_kept = oracle.topk(ref_scores.astype(np.float32), kk)
    got_scores = nb.cls_scores(to_dev(q, "bf16"), to_dev(k, "bf16"), 0.125)
    kept, _, _ = nb.topk_filter(got_scores, kk)
    torch.cuda.synchronize()
    assert_kept_sets_match(kept.cpu().numpy(), ref_kept, ref_scores, kk)


def test_running_out_of_memory_is_reported_as_such(nb):
    """An output that no device holds: the allocator's own exception, as from any torch call."""
    with pytest.raises(torch.cuda.OutOfMemoryError):
        nb.topk_filter(torch.zeros(1, 64, device="cuda"), 2 ** 42)


def test_indices_written_over_the_scores(nb):
    """The one row's scores are all read before the first index is written, where they share memory."""
    rng = np.random.default_rng(12)
    scores = rng.random((1, 16384)).astype(np.float32)
    buf = torch.from_numpy(scores).cuda()
    kept, _, _ = nb.topk_filter(buf, 9831, kept_idx=buf.view(torch.int32)[:, :9831])
    torch.cuda.synchronize()
    assert np.array_equal(kept.cpu().numpy(), oracle.topk(scores, 9831))


@pytest.mark.parametrize("H,G,N", [(1, 1, 50001), (3, 1, 49920), (4, 1, 50000), (5, 3, 45000), (16, 1, 44801), (1, 7, 131073)])
def test_scores_do_not_depend_on_the_launch(nb, H, G, N):
    """Three images are more workgroups than the chip holds at once, one image (but the last) is not: other numbers of threads to a
    patch, the same sums.  Exponentials and sums of at most 21 positive terms in fp32: 2^-20 of the result."""
    gen = torch.Generator(device="cuda").manual_seed(N)
    logits = torch.randn((3, H, G, G + N), generator=gen, device="cuda") * 2.0
    lse = torch.logsumexp(logits.double(), dim=-1).float()
    got = nb.cls_scores_from_logits(logits, lse, n_global=G)
    alone = torch.cat([nb.cls_scores_from_logits(logits[b:b + 1], lse[b:b + 1], n_global=G) for b in range(3)])
    ref = (logits.double() - lse.double()[..., None]).exp()[..., G:].mean(dim=(1, 2))
    torch.cuda.synchronize()
    assert torch.equal(got, alone)
    np.testing.assert_allclose(got.double().cpu().numpy(), ref.cpu().numpy(), rtol=2.0 ** -19, atol=0)


@pytest.mark.parametrize("H,G,B", [(2, 1, 60), (3, 2, 57)])
def test_scores_with_the_attention_do_not_depend_on_the_launch(nb, monkeypatch, H, G, B):
    """As above where the records are merged in the same launch."""
    monkeypatch.setenv("NSATTN_KERNEL", "lists1")
    g = 40
    gen = torch.Generator(device="cuda").manual_seed(H)
    q, k, v = (torch.randn((B, H, G + g * g, 64), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    out, logits, lse, scores = nb.ns_attn_forward_scores(q, k, v, g, g, 8, n_global=G)
    torch.cuda.synchronize()
    ref = torch.softmax(logits.double().reshape(B, H, G, -1), dim=-1)[..., G:].mean(dim=(1, 2))
    np.testing.assert_allclose(scores.double().cpu().numpy(), ref.cpu().numpy(), rtol=2.0 ** -17, atol=0)
    for b in (0, B - 1):
        few = nb.ns_attn_forward_scores(*(t[b:b + 2] if b == 0 else t[b - 1:b + 1] for t in (q, k, v)), g, g, 8, n_global=G)
        torch.cuda.synchronize()
        at = 0 if b == 0 else 1
        assert torch.equal(few[3][at], scores[b]) and torch.equal(few[0][at], out[b]) and torch.equal(few[2][at], lse[b])
