"""Host-side bounds models of the two attention kernels that share key tiles through LDS, on grids their blocks do not
divide as on others.  They mirror the kernels' address arithmetic - direct global -> LDS transfers add an UNSIGNED 32-bit lane
offset to a scalar base, divisions are fp32 products - and check that every address stays inside the (batch, head) slice.
A lane offset that underflows wraps to +4 GiB: that is the fault this test guards against."""
import numpy as np
import pytest

M32 = 1 << 32
def u32(x): return x % M32

LANE = np.arange(64)
L32, HH, ROW8 = LANE & 31, LANE >> 5, LANE >> 3
KCH = [16 * ((LANE & 7) ^ (4 * j + (LANE >> 4))) for j in range(2)]     # source chunk of a lane's 16 bytes of K, by request's parity
VCH = 16 * ((LANE & 7) ^ (((LANE >> 4) & 1) << 2))                      # ... of V


def div_small(a, d):
    """The kernel's quotient: fp32, one product."""
    return ((np.asarray(a).astype(np.float32) + np.float32(0.5)) * (np.float32(1) / np.float32(d))).astype(np.int64)


def check_block16(gh, gw, block, G=1, rowB=128):
    """Every access of attn_block16_kernel to Q, K, V and the output of one head, its redo included, as (token, byte of
    the row); rowB: bytes from row to row.  Returns how many leave the token rows' 128 bytes or miss the row that the numbering asks for."""
    T = G + gh * gw
    nbh, nbw, parts = -(-gh // block), -(-gw // block), -(-block * block // 256)
    bad = 0

    def access(at, size, want=None):
        nonlocal bad
        if len(at) == 0:
            return
        assert at.min() >= 0 and at.max() < M32          # (no 32-bit offset wraps)
        tok, byte = at // rowB, at % rowB
        bad += int(np.sum((tok >= T) | (byte + size > 128)))
        if want is not None:
            bad += int(np.sum(tok != want))

    access(np.minimum(ROW8, G - 1) * rowB + 16 * (LANE & 7), 16)             # the global tokens' rows
    for R in range(nbh):
        for C in range(nbw):
            r0, c0 = R * block, C * block
            bw = min(block, gw - c0)
            qn = min(block, gh - r0) * bw
            kr0, kc0 = max(r0 - block, 0), max(c0 - block, 0)
            kw = min(c0 + 2 * block, gw) - kc0
            nk = (min(r0 + 2 * block, gh) - kr0) * kw
            steps = (nk + 63) // 64

            def key(j):
                j = np.minimum(j, nk - 1)
                r = div_small(j, kw)
                return G + (kr0 + r) * gw + kc0 + j - r * kw

            exact = np.arange(64 * steps)
            exact = np.minimum(exact, nk - 1)
            exact = G + (kr0 + exact // kw) * gw + kc0 + exact % kw
            for wave in range(4):                        # transfers: a wave moves its share, whether it has queries or not
                row = [16 * wave + 8 * j + ROW8 for j in range(2)]
                r = [div_small(i, kw) for i in row]
                col = [i - q * kw for i, q in zip(row, r)]
                at = [u32((G + (kr0 + q) * gw + kc0 + c) * rowB) for q, c in zip(r, col)]
                for t in range(steps):
                    for j in range(2):
                        if t == steps - 1 and nk & 63:
                            at[j] = key(64 * t + row[j]) * rowB
                        access(at[j] + KCH[j], 16, exact[64 * t + row[j]])
                        access(at[j] + VCH, 16, exact[64 * t + row[j]])
                        col[j] = col[j] + 64 % kw
                        at[j] = u32(at[j] + ((64 // kw) * gw + 64 % kw) * rowB)
                        at[j] = u32(np.where(col[j] >= kw, at[j] + (gw - kw) * rowB, at[j]))
                        col[j] = np.where(col[j] >= kw, col[j] - kw, col[j])
            for t in range(steps):                       # the redo
                for mt in range(2):
                    for s in range(4):
                        access(key(64 * t + 32 * mt + L32) * rowB + 64 * HH + 16 * s, 16, exact[64 * t + 32 * mt + L32])
                for it in range(8):
                    access(key(64 * t + 8 * it + ROW8) * rowB + VCH, 16, exact[64 * t + 8 * it + ROW8])
            for part in range(parts):
                for wave in range(4):
                    q0 = part * 256 + wave * 64
                    qcnt = min(qn - q0, 64)
                    if part * 256 >= qn or qcnt <= 0:
                        continue
                    for nt in range(2):
                        i = 32 * nt + L32
                        s = q0 + np.minimum(i, qcnt - 1)
                        q = div_small(s, bw)
                        tok = G + (r0 + q) * gw + c0 + s - q * bw
                        want = G + (r0 + s // bw) * gw + c0 + s % bw
                        for f in range(4):
                            access(tok * rowB + 64 * HH + 16 * f, 16, want)
                        for dt in range(2):
                            for ig in range(2):          # stores: the output's rows are addressed with 64 bits
                                access((tok * rowB + 16 * HH + 64 * dt + 32 * ig)[i < qcnt], 16, want[i < qcnt])
    return bad

def check_sweep(gh, gw):
    rowB = 128; gridrowB = gw * rowB; T = 1 + gh * gw; size = T * rowB
    nbh, nbw = (gh + 7) // 8, (gw + 7) // 8
    hv_last, wv_last = gh - 8 * (nbh - 1), gw - 8 * (nbw - 1)
    bad = 0
    block_token = lambda Rb, Cb: 1 + Rb * 8 * gw + Cb * 8
    tile_off = lambda i, hv, wv: u32((min(i >> 3, hv - 1) * gw + min(i & 7, wv - 1)) * rowB)
    for R in range(nbh):
        hvq = hv_last if R == nbh - 1 else 8
        r0, r1 = max(R - 1, 0), min(R + 1, nbh - 1)
        for wave in range(4):
            for lane in range(64):
                l32, hh, drow = lane & 31, lane >> 5, lane >> 3
                for qc in range(nbw):
                    wvq = wv_last if qc == nbw - 1 else 8
                    for nt in range(2):
                        i = l32 + 32 * nt
                        a = block_token(R, qc) * rowB + u32(tile_off(i, hvq, wvq) + 64 * hh)
                        if not (rowB <= a and a + 64 <= size): bad += 1
                        a = (block_token(R, qc) + min(i >> 3, hvq - 1) * gw + min(i & 7, wvq - 1)) * rowB
                        if not (rowB <= a and a + 128 <= size): bad += 1
                    # logits store (lane = key)
                    wvc = wv_last if qc == nbw - 1 else 8
                    kr, kc = min(lane >> 3, hvq - 1), min(lane & 7, wvc - 1)
                    tok = block_token(R, qc) + kr * gw + kc
                    if not (1 <= tok < T): bad += 1
                for ic in range(nbw):
                    for ir in range(r1 - r0 + 1):
                        hvk = hv_last if r0 + ir == nbh - 1 else 8
                        base = block_token(r0 + ir, ic) * rowB
                        row, chunk = u32(min(drow, (wv_last if ic == nbw - 1 else 8) - 1) * rowB), 16 * ((lane & 7) ^ (lane >> 4))
                        for j, off in enumerate((chunk, chunk ^ 64)):
                            assert off == KCH[j][lane]
                            a = base + min(2 * wave + j, hvk - 1) * gridrowB + u32(row + off)
                            if not (rowB <= a and a + 16 <= size): bad += 1
                            if bad > 5: return bad
    return bad



# (several global tokens; rows of a fused q/k/v tensor with 16 heads; last tiles of 1 to 63 keys; blocks whose last workgroup
# has waves without queries; blocks larger than the grid)
@pytest.mark.parametrize("gh,gw,block,G,rowB", [
    (20, 27, 16, 1, 128), (37, 21, 16, 5, 128), (16, 50, 16, 1, 6144), (33, 16, 48, 8, 128), (1, 1, 16, 1, 128), (5, 70, 16, 2, 6144),
    (19, 30, 32, 1, 128), (3, 3, 256, 1, 128), (37, 21, 32, 1, 6144), (50, 70, 32, 3, 128), (70, 53, 64, 1, 128), (13, 5, 64, 1, 128),
    (65, 65, 64, 1, 128), (130, 20, 64, 5, 128), (16, 16, 16, 1, 128), (31, 33, 16, 1, 128)])
def test_block16_kernel_addresses_stay_in_bounds(gh, gw, block, G, rowB):
    assert check_block16(gh, gw, block, G, rowB) == 0


def test_division_of_the_largest_key_numbers():
    """Blocks are at most 256 a side: key numbers stay below 768 * 768, row lengths below 768."""
    for d in range(1, 769):
        a = np.unique(np.clip(np.concatenate([np.arange(0, 768 * d, d) + e for e in (-1, 0, 1)]), 0, 768 * 768 - 1))
        assert np.array_equal(div_small(a, d), a // d), d


@pytest.mark.parametrize("gh,gw", [(20, 27), (9, 9), (8, 100), (17, 8), (1, 1), (5, 5), (12, 30), (23, 33)])
def test_sweep_kernel_addresses_stay_in_bounds(gh, gw):
    assert check_sweep(gh, gw) == 0


def test_addresses_stay_in_bounds_on_random_grids():
    """A seeded sample of grid shapes (sides 1..75) through both address models."""
    import random
    rng = random.Random(2024)
    for _ in range(24):
        gh, gw = rng.randint(1, 75), rng.randint(1, 75)
        assert check_sweep(gh, gw) == 0, (gh, gw)
        assert check_block16(gh, gw, rng.choice([16, 32, 64]), rng.choice([1, 4]), rng.choice([128, 384])) == 0, (gh, gw)


# ---- the block kernel as it numbers queries and keys: in raster order within the block and within the rectangle of its keys


def block_of(blk, rim, nbh, nbw):
    if not rim:
        R = blk // (nbw - 2)
        return R + 1, 1 + blk - R * (nbw - 2)
    ends, b2 = min(nbw, 2), blk - nbw
    b3 = b2 - max(nbh - 2, 0) * ends
    if b2 < 0:
        return 0, blk
    return (1 + b2 // ends, nbw - 1 if b2 % ends else 0) if b3 < 0 else (nbh - 1, b3)


@pytest.mark.parametrize("gh,gw,block", [(16, 16, 16), (17, 33, 16), (245, 245, 64), (100, 53, 32), (48, 20, 64), (33, 64, 16), (80, 3, 16)])
def test_block_kernel_numbering(gh, gw, block):
    """Every token is the query of one slot and every key of a block's rectangle is brought in once, at the place where
    the next 64 keys follow by steps of whole rows and columns, as the kernel's lanes advance."""
    nbh, nbw, parts = -(-gh // block), -(-gw // block), -(-block * block // 256)
    inner = max(nbh - 2, 0) * max(nbw - 2, 0)
    blocks = [block_of(i, False, nbh, nbw) for i in range(inner)] + [block_of(i, True, nbh, nbw) for i in range(nbh * nbw - inner)]
    assert sorted(blocks) == [(R, C) for R in range(nbh) for C in range(nbw)]
    queries = []
    for R, C in blocks:
        r0, c0 = R * block, C * block
        bw = min(block, gw - c0)
        qn = min(block, gh - r0) * bw
        assert qn <= 256 * parts
        queries += [(r0 + s // bw) * gw + c0 + s % bw for s in range(qn)]
        kr0, kc0 = max(r0 - block, 0), max(c0 - block, 0)
        kw = min(c0 + 2 * block, gw) - kc0
        nk = (min(r0 + 2 * block, gh) - kr0) * kw
        right, step, wrap = 64 % kw, (64 // kw) * gw + 64 % kw, gw - kw
        for i in range(64):                        # the key rows that place i of a tile takes, tile by tile
            col, at = i % kw, (kr0 + i // kw) * gw + kc0 + i % kw
            for j in range(i, nk, 64):
                assert at == (kr0 + j // kw) * gw + kc0 + j % kw < gh * gw
                col, at = col + right, at + step
                if col >= kw:
                    col, at = col - kw, at + wrap
    assert sorted(queries) == list(range(gh * gw))
