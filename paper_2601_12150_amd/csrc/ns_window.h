// Query tiles and key lists of the kernels that split one query tile's keys over the waves of a
// workgroup (ns_attn_ragged.hip, ns_attn_generic.hip).
//
// A workgroup owns one tile of up to QT queries.  Complete grid: the grid is cut into squares of
// `side` patches - a block, or for blocks of side <= 4 the largest square of whole blocks that
// fits 8x8 - and a tile is a run of QT tokens of a square in raster order; its keys are the global
// tokens followed by the patches of the rectangle that the 3x3 blocks around the square's blocks
// cover, in raster order, so short edge blocks leave no holes.  Pruned sequence: a tile is a run
// of a block's token list, its keys the global tokens and the lists of the up to nine neighbouring
// blocks one after the other.  Either way keys are numbered 0 .. nkeys-1 without gaps and every
// lane turns the number of its key into a token.
#pragma once
#include "ns_common.h"
#include <algorithm>
#include <cmath>
#include <type_traits>

namespace ns {

struct WindowGeom {
  int grid_h, grid_w, block, n_global, tokens, heads;
  int side;                // squares' side: a multiple of block
  int nbh, nbw;            // squares per grid side
  int tpb;                 // tiles per square (pruned: per block list capacity)
  int cap;                 // slots per block in `lists`
  int tiles_per_image;     // nbh * nbw * tpb
  int tiles;               // batch * heads * tiles_per_image
  int per_xcd;             // workgroups per XCD
  int row_wgs;             // workgroups that own chunks of the global rows
  int rows_at, tiles_at;   // first workgroup of these and of the tiles' (a multiple of 8)
  int global_groups;       // groups of global rows per head
  int nchunks;             // key chunks per head-image
  const int32_t *lists, *counts;
};

// Tile of a workgroup: everything is wave-uniform except what the token functions return.
template <bool LISTS, int QT>
struct WindowTile {
  int b, h, R, C;
  int q0, qcnt;            // first slot of the tile in its square / list, queries in it
  int nkeys;
  int bw, kr0, kc0, kw;    // complete grid: columns of the square; key rectangle
  float inv_bw, inv_kw;
  int pre[10];             // pruned: first key number of each neighbour block (pre[9]: end)
  const int32_t *lst;      // pruned: this image's lists

  // false: no such tile
  __device__ __forceinline__ bool init(const WindowGeom &g, int id, int lane) {
    const int img = id / g.tiles_per_image, t = id - img * g.tiles_per_image;
    b = img / g.heads;
    h = img - b * g.heads;
    const int sq = t / g.tpb;
    q0 = (t - sq * g.tpb) * QT;
    R = sq / g.nbw;
    C = sq - R * g.nbw;
    if (LISTS) {
      const int nblocks = g.nbh * g.nbw;
      const int32_t *cnts = g.counts + (size_t)b * nblocks;
      lst = g.lists + (size_t)b * nblocks * g.cap;
      int fill = 0;
      if (lane < 9) {
        const int R2 = R + lane / 3 - 1, C2 = C + lane % 3 - 1;
        if (R2 >= 0 && R2 < g.nbh && C2 >= 0 && C2 < g.nbw) fill = cnts[R2 * g.nbw + C2];
      }
      int n = g.n_global;
#pragma unroll
      for (int i = 0; i < 9; i++) {
        pre[i] = n;
        n += __builtin_amdgcn_readlane(fill, i);
      }
      pre[9] = nkeys = n;
      qcnt = min(pre[5] - pre[4] - q0, QT);
    } else {
      const int bh = min(g.side, g.grid_h - R * g.side);
      bw = min(g.side, g.grid_w - C * g.side);
      qcnt = min(bh * bw - q0, QT);
      kr0 = max(R * g.side - g.block, 0);
      kc0 = max(C * g.side - g.block, 0);
      kw = min((C + 1) * g.side + g.block, g.grid_w) - kc0;
      nkeys = g.n_global + (min((R + 1) * g.side + g.block, g.grid_h) - kr0) * kw;
      inv_bw = 1.f / (float)bw;
      inv_kw = 1.f / (float)kw;
    }
    return qcnt > 0;
  }
  // token of query slot i (slots past the end repeat the last one)
  __device__ __forceinline__ int query(const WindowGeom &g, int i) const {
    const int s = q0 + min(i, qcnt - 1);
    if (LISTS) return lst[(size_t)(R * g.nbw + C) * g.cap + s];
    const int r = div_small(s, inv_bw);
    return g.n_global + (R * g.side + r) * g.grid_w + C * g.side + s - r * bw;
  }
  // Complete grid: token of key j (numbers past the end repeat the last one).
  __device__ __forceinline__ int key(const WindowGeom &g, int j) const {
    j = min(j, nkeys - 1);
    const int jj = max(j - g.n_global, 0), r = div_small(jj, inv_kw);
    const int tok = g.n_global + (kr0 + r) * g.grid_w + kc0 + jj - r * kw;
    return j < g.n_global ? j : tok;
  }
  // Pruned: where the token of key j stands (a global token has no entry: its number is its token,
  // and the address given for it is some valid entry).
  __device__ __forceinline__ const int32_t *key_entry(const WindowGeom &g, int j) const {
    j = min(j, nkeys - 1);
    int i = 4, start = pre[4];
    if (j >= g.n_global) {
      i = 0; start = pre[0];
#pragma unroll
      for (int n = 1; n < 9; n++) {
        i = j >= pre[n] ? n : i;
        start = j >= pre[n] ? pre[n] : start;
      }
    }
    const int dr = (i * 11) >> 5;          // i / 3 for i < 9
    const int blk = (R + dr - 1) * g.nbw + C + i - 3 * dr - 1;
    return lst + (size_t)blk * g.cap + max(j - start, 0);
  }
  // Squares of several blocks: a key may be seen by a query if every bit of the key's code is set
  // in the query's.  Bits 0.. are block rows, bits 16.. block columns, both counted from one block
  // before the square; a global token has no bits, a key past the end one that no query has.
  __device__ __forceinline__ uint32_t key_code(const WindowGeom &g, int j, float inv_block) const {
    const int jj = max(j - g.n_global, 0), r = div_small(jj, inv_kw), c = jj - r * kw;
    // (counted from row R*side - block and column C*side - block, at or before the rectangle's first)
    const int rb = div_small(kr0 + r - (R * g.side - g.block), inv_block);
    const int cb = div_small(kc0 + c - (C * g.side - g.block), inv_block);
    const uint32_t code = (1u << rb) | (0x10000u << cb);
    return j >= nkeys ? 0x8000u : (j < g.n_global ? 0u : code);
  }
  __device__ __forceinline__ uint32_t query_code(const WindowGeom &g, int i, float inv_block) const {
    const int s = q0 + min(i, qcnt - 1), r = div_small(s, inv_bw), c = s - r * bw;
    return (7u << div_small(r, inv_block)) | (0x70000u << div_small(c, inv_block));
  }
};

// Position of workgroup `bid`: workgroups are dealt round-robin to the 8 XCDs, and each XCD gets a contiguous range of
// tiles, so that the K and V rows which neighbouring tiles share are fetched into one L2.
__device__ __forceinline__ int window_tile_id(const WindowGeom &g, int bid) {
  return (bid & 7) * g.per_xcd + (bid >> 3);
}

// ------------------------------------------------------------------------------------------
// A step: 32 keys against 32*NT queries by one wave.  S^T = K Q^T and O^T += V^T P^T, so that a
// query's statistics live in one lane pair (l32, l32 + 32) and the logits' accumulator layout -
// register e of lane (query l32, half hh) is key 8*(e/4) + 4*hh + e%4 - is the operand layout of
// the second product: the weights never leave the registers.  K and V rows come global -> LDS by
// direct 16-byte transfers, whole rows per request, into rings of kDepth slots each that belong
// to the wave alone (no barriers); the transfer into a slot is requested as soon as the wave has
// read it.
// ------------------------------------------------------------------------------------------

// What the passes of walk_not_finite() make of a value (the bits of a float): 0, 1: 1 where it is +inf or -inf or,
// in both, NaN, else 0; 2: 0 in place of a value that is not finite.
__device__ __forceinline__ uint32_t screened(uint32_t x, int pass) {
  const bool bad = (x & 0x7f800000u) == 0x7f800000u, nan = bad && (x & 0x7fffffu) != 0;
  if (pass == 2) return bad ? 0u : x;
  return nan || (bad && (int)(x >> 31) == pass) ? 0x3f800000u : 0u;
}

// bf16: v_mfma_f32_32x32x16_bf16, weights rounded to bf16 for the second product.
struct StepBf16 {
  typedef uint16_t elem;
  static constexpr bool kParts = false;
  static constexpr int kDepth = 2, kReq = 4, kHalf = 4096;     // slots, requests per 32 rows, bytes of 32 rows
  struct Q { bf16x8 f[4]; };
  typedef s16x4 __attribute__((address_space(3))) *tr_ptr;
  typedef bf16x8 __attribute__((address_space(3))) *frag_ptr;
  uint32_t kch[2], vch;       // source chunk of this lane's 16 bytes
  uint32_t krd[4], vrd[2][2];
  int rrow;                   // row of request 0 this lane moves; request it: + 8 it
  // The first step's first keys are global tokens, which every row sees and which can be most of a row: their weights
  // enter with the bits they have in fp32, what bf16 rounding leaves in two further terms.
  int exact;                  // so many keys (8 at most) do
  // Selects, as the left operand of v_mfma_f32_16x16x32_bf16, the lanes whose bit 4 is the row's bit 0.  The weights of
  // a fragment (lane: query l32, eight keys) as right operand then give query lane % 16's sum in the even registers of the
  // result and query 16 + lane % 16's in the odd ones: both halves' keys, no vector instruction.
  uint32_t sel;               // (two equal values; the operand is four of these)

  __device__ __forceinline__ void init(int lane) {
    const int l32 = lane & 31, hh = lane >> 5;
    exact = 0;
    sel = ((lane ^ (lane >> 4)) & 1) ? 0u : 0x3f803f80u;
    rrow = lane >> 3;
    // LDS chunk c of row r holds chunk c ^ ((r>>1)&7) of K and c ^ 4*((r>>1)&1) of V: conflict-free reads
    kch[0] = 16u * ((lane & 7) ^ (lane >> 4));
    kch[1] = 16u * ((lane & 7) ^ (4 + (lane >> 4)));
    vch = 16u * ((lane & 7) ^ (((lane >> 4) & 1) << 2));
#pragma unroll
    for (int s = 0; s < 4; s++) krd[s] = l32 * 128 + 16 * ((4 * hh + s) ^ ((l32 >> 1) & 7));
    const int g = lane >> 4, s = lane & 15;
    const int dbyte = (16 * (g & 1) + 4 * (s & 3)) * 2;
#pragma unroll
    for (int half = 0; half < 2; half++) {
      const int key = 8 * half + 4 * hh + (s >> 2);
      const int off = key * 128 + (dbyte ^ (((key >> 1) & 1) << 6));
      vrd[0][half] = off;
      vrd[1][half] = off ^ 64;
    }
  }
  // (rows are addressed with 32-bit byte offsets from the head's first row: checked by the launcher)
  template <class F>                  // Q or K: a row's fragments, straight from memory
  __device__ __forceinline__ void load_q(F &q, const char *base, int64_t rowB, int tok, int lane, float) const {
    const char *row = base + (uint32_t)tok * (uint32_t)rowB + 64 * (lane >> 5);
#pragma unroll
    for (int s = 0; s < 4; s++) q.f[s] = *reinterpret_cast<const bf16x8 *>(row + 16 * s);
  }
  // a row's byte offset, passed from lane to lane instead of its token: one multiplication per key
  static __device__ __forceinline__ uint32_t place(int tok, int64_t rowB) { return (uint32_t)tok * (uint32_t)rowB; }
  __device__ __forceinline__ void issue_k(const char *base, int64_t, const uint32_t (&at)[kReq], unsigned char *, uint32_t lds, int) const {
#pragma unroll
    for (int it = 0; it < kReq; it++) dma16(base, at[it] + kch[it & 1], lds + it * 1024);
  }
  __device__ __forceinline__ void issue_v(const char *base, int64_t, const uint32_t (&at)[kReq], unsigned char *, uint32_t lds, int) const {
#pragma unroll
    for (int it = 0; it < kReq; it++) dma16(base, at[it] + vch, lds + it * 1024);
  }
  struct K { bf16x8 f[4]; };
  __device__ __forceinline__ void load_k(K &k, const unsigned char *slot) const {
#pragma unroll
    for (int t = 0; t < 4; t++) k.f[t] = *(frag_ptr)(slot + krd[t]);
  }
  __device__ __forceinline__ f32x16 product(const K &k, const Q &q) const {
    f32x16 s = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 4; t++) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k.f[t], q.f[t], s, 0, 0, 0);
    return s;
  }
  struct V { bf16x8 f[2][2]; };      // [keys 16 sp ..][channels 32 dt ..]
  __device__ __forceinline__ void load_v(V &v, const unsigned char *slot, int sp) const {
#pragma unroll
    for (int dt = 0; dt < 2; dt++) {
      const s16x4 lo4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(slot + vrd[dt][0] + sp * 2048));
      const s16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(slot + vrd[dt][1] + sp * 2048));
      const bf16x4 a = __builtin_bit_cast(bf16x4, lo4), b2 = __builtin_bit_cast(bf16x4, hi4);
      v.f[sp][dt] = bf16x8{a[0], a[1], a[2], a[3], b2[0], b2[1], b2[2], b2[3]};
    }
  }
  template <int NT>
  __device__ __forceinline__ void logits(const Q (&q)[NT], const unsigned char *slot, f32x16 (&s)[NT]) const {
    K k;
    load_k(k, slot);
#pragma unroll
    for (int nt = 0; nt < NT; nt++) s[nt] = product(k, q[nt]);
  }
  // Half a pipelined step: the weights of 32 queries from their logits `cur`, interleaved with eight matrix
  // instructions: the last half's open output product (`open`: the second half of its keys' weights, o_open),
  // the logits `nxt` of the other queries, the first half of this output product.  One matrix instruction
  // (32 cycles) to the seven vector instructions of two weights (36 cycles); a weight's three links are a
  // group apart, so that no result is waited for.  The fences keep this order: left to itself the
  // scheduler groups the exponentials and then the matrix instructions.  (Sums by matrix instruction and the weights kept
  // in this order: 100 x 100 patches, 8 x 8 blocks, five global tokens, 104.3 -> 101.3 us a call.)
  // LOADV: load the second half of V once the open product has taken the old one.  NEXT: there are other logits to form.
  // OPEN: there is an open product.
  template <bool LOADV, bool NEXT = true, bool OPEN = true, class L>
  __device__ __forceinline__ void half_step(f32x16 &cur, float c, float nm, L &l, f32x16 (&o)[2], L &l_open,
                                            f32x16 (&o_open)[2], bf16x8 &open, V &v, const unsigned char *vslot, const K &k,
                                            const Q &q, f32x16 &nxt) const {
    // The sums are those of the rounded weights that the product takes, which adds them itself (add_weights): what
    // rounding does to a key that outweighs the others cancels.  Relative error of rows with logits of +-8, against sums
    // of the weights before rounding: 0.0021 -> 0.0017 (rounding the true result alone: 0.0016); of +-1: 0.00220 -> 0.00218.
    bf16x8 first, second;
    if (NEXT) nxt = f32x16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 4; e++) cur[e] = __builtin_fmaf(cur[e], c, nm);
    cur[0] = __builtin_amdgcn_exp2f(cur[0]);
    cur[1] = __builtin_amdgcn_exp2f(cur[1]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 8; j++) {
      if (j < 7) {
        cur[2 * j + 2] = __builtin_amdgcn_exp2f(cur[2 * j + 2]);
        cur[2 * j + 3] = __builtin_amdgcn_exp2f(cur[2 * j + 3]);
      }
      if (j < 6) {
        cur[2 * j + 4] = __builtin_fmaf(cur[2 * j + 4], c, nm);
        cur[2 * j + 5] = __builtin_fmaf(cur[2 * j + 5], c, nm);
      }
      uint32_t packed = pack_bf16(cur[2 * j], cur[2 * j + 1]);
      // (used here: the compiler would otherwise sink the second half of the weights behind a branch that follows, out of
      // the matrix instructions' shadow)
      asm volatile("" : "+v"(packed));
      const bf16x2 pk = __builtin_bit_cast(bf16x2, packed);
      add_pair(l, pk, j);
      if (j < 4) { first[2 * j] = pk[0]; first[2 * j + 1] = pk[1]; }
      else { second[2 * j - 8] = pk[0]; second[2 * j - 7] = pk[1]; }
      if (j < 2) { if (OPEN) o_open[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v.f[1][j], open, o_open[j], 0, 0, 0); }
      else if (j < 6) { if (NEXT) nxt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k.f[j - 2], q.f[j - 2], nxt, 0, 0, 0); }
      else o[j - 6] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v.f[0][j - 6], first, o[j - 6], 0, 0, 0);
      if (OPEN && j == 1) add_weights(l_open, open);
      if (j == 7) add_weights(l, first);
      __builtin_amdgcn_sched_barrier(0);
      if (LOADV && j == 1) load_v(v, vslot, 1);
    }
    open = second;
  }
  // A row's sum += a fragment's weights; what the sum is for this lane's query (of both half-waves' keys).  Sums: four
  // registers that the product adds to, LeanSums: the two of them that count, for a kernel that is short of registers.
  // LaneSums: each lane its own, for a kernel that computes a query in several lanes and needs the same bits in all.
  typedef f32x4 Sums;
  typedef f32x2 LeanSums;
  struct LaneSums { float l[2]; };
  __device__ __forceinline__ void add_weights(Sums &l, const bf16x8 &w) const {
    l = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, u32x4{sel, sel, sel, sel}), w, l, 0, 0, 0);
  }
  __device__ __forceinline__ void add_weights(LeanSums &l, const bf16x8 &w) const {
    uint32_t x = sel;
    asm volatile("" : "+v"(x));               // (put together here: not four registers that live through the loop)
    const f32x4 s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, u32x4{x, x, x, x}), w, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    l[0] += s[0];
    l[1] += s[1];
  }
  __device__ __forceinline__ void add_weights(LaneSums &, const bf16x8 &) const {}
  __device__ __forceinline__ void add_pair(LaneSums &l, const bf16x2 &w, int j) const {
    l.l[j & 1] = __builtin_amdgcn_fdot2_f32_bf16(w, bf16x2{(__bf16)1.f, (__bf16)1.f}, l.l[j & 1], false);
  }
  template <class L> __device__ __forceinline__ void add_pair(L &, const bf16x2 &, int) const {}
  // what half-wave hh adds to its query's sum
  static __device__ __forceinline__ float row_sum(const LaneSums &l, int) { return l.l[0] + l.l[1]; }
  template <class L>
  static __device__ __forceinline__ float row_sum(const L &l, int lane) { return lane >= 32 ? 0.f : (lane & 16 ? l[1] : l[0]); }
  // O^T += V^T w.  LO: columns 16..31 are the first 16 once more and take what bf16 rounding leaves of a weight,
  // w - bf16(w); what that leaves in turn comes in a second product, so that all 24 bits of a weight enter.
  template <int NT, bool LO>
  __device__ __forceinline__ void weigh(const f32x16 (&w)[NT], const unsigned char *slot, f32x16 (&o)[NT][2], int lane) const {
    bf16x8 pf[NT][2], pr[NT][2];
#pragma unroll
    for (int nt = 0; nt < NT; nt++)
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        uint32_t u = pack_bf16(w[nt][i], w[nt][i + 1]);
        if (LO) {
          const float r0 = w[nt][i] - bf16_lo(u), r1 = w[nt][i + 1] - bf16_hi(u);
          const uint32_t lo = pack_bf16(r0, r1), last = (lane & 16) ? 0u : pack_bf16(r0 - bf16_lo(lo), r1 - bf16_hi(lo));
          u = (lane & 16) ? lo : u;
          const bf16x2 pl = __builtin_bit_cast(bf16x2, last);
          pr[nt][i >> 3][i & 7] = pl[0];
          pr[nt][i >> 3][(i & 7) + 1] = pl[1];
        }
        const bf16x2 pk = __builtin_bit_cast(bf16x2, u);
        pf[nt][i >> 3][i & 7] = pk[0];
        pf[nt][i >> 3][(i & 7) + 1] = pk[1];
      }
#pragma unroll
    for (int sp = 0; sp < 2; sp++) {
      V v;
      load_v(v, slot, sp);
#pragma unroll
      for (int term = 0; term < (LO ? 2 : 1); term++)
#pragma unroll
        for (int dt = 0; dt < 2; dt++)
#pragma unroll
          for (int nt = 0; nt < NT; nt++)
            o[nt][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v.f[sp][dt], term ? pr[nt][sp] : pf[nt][sp], o[nt][dt], 0, 0, 0);
    }
  }
  // O^T += V^T (w - bf16(w)) for the first `exact` keys of a step, 16 bits of it in two terms: the keys 0..7 stand
  // in a fragment's first four elements, V's once more in the other four.  Returns the sum of what is left (of this
  // half-wave's keys).
  __device__ __forceinline__ float add_rest(const f32x16 &w, const unsigned char *slot, f32x16 (&o)[2], int lane) const {
    bf16x8 r;
    float sum = 0.f;
#pragma unroll
    for (int e = 0; e < 4; e += 2) {
      const int key = 4 * (lane >> 5) + e;
      float a = w[e], b = w[e + 1];
      uint32_t u = pack_bf16(a, b);
#pragma unroll
      for (int t = 0; t < 2; t++) {
        a = key < exact ? a - bf16_lo(u) : 0.f;
        b = key + 1 < exact ? b - bf16_hi(u) : 0.f;
        if (t == 0) sum += a + b;
        u = pack_bf16(a, b);
        const bf16x2 pk = __builtin_bit_cast(bf16x2, u);
        r[4 * t + e] = pk[0];
        r[4 * t + e + 1] = pk[1];
      }
    }
#pragma unroll
    for (int dt = 0; dt < 2; dt++) {
      const bf16x4 v = __builtin_bit_cast(bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(slot + vrd[dt][0])));
      const bf16x8 vv = {v[0], v[1], v[2], v[3], v[0], v[1], v[2], v[3]};
      o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vv, r, o[dt], 0, 0, 0);
    }
    return sum;
  }
  static __device__ __forceinline__ uint32_t screen(uint32_t two, int pass) {
    return screened(two & 0xffff0000u, pass) | (screened(two << 16, pass) >> 16);
  }
  static __device__ __forceinline__ void store4out(uint16_t *p, f32x4 v) {
    *reinterpret_cast<u32x2 *>(p) = u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
  }
};

// fp32 arithmetic: v_mfma_f32_32x32x2_f32 on rows of 64 floats (T = uint16_t: bf16 rows, converted
// on the way into LDS), for what StepF32 below cannot do.  An operand register holds one k index per half-wave: step s of the
// logits pairs channels s and 32 + s, step e of the second product keys (e, hh = 0) and (e, hh = 1).
template <typename T>
struct StepF32Whole {
  typedef T elem;
  static constexpr int kDepth = 1, kReq = 8, kHalf = 8192;
  static constexpr bool kParts = false;
  struct Q { float f[32]; };
  uint32_t kbase, kx, vrd[2];
  int rrow;
  __device__ __forceinline__ void init(int lane) {
    const int l32 = lane & 31, hh = lane >> 5;
    rrow = lane >> 4;
    // LDS chunk c of row r holds chunk c ^ (r & 15) of K and c ^ 8*((r>>2)&1) of V
    kbase = l32 * 256;
    kx = 16 * ((8 * hh) ^ (l32 & 15));
    vrd[0] = hh * 1024 + ((l32 * 4) ^ (hh * 128));
    vrd[1] = hh * 1024 + ((l32 * 4 + 128) ^ (hh * 128));
  }
  __device__ static __forceinline__ f32x4 load4(const float *p) { return *reinterpret_cast<const f32x4 *>(p); }
  __device__ static __forceinline__ f32x4 load4(const uint16_t *p) {
    const u32x2 u = *reinterpret_cast<const u32x2 *>(p);
    return f32x4{bf16_lo(u[0]), bf16_hi(u[0]), bf16_lo(u[1]), bf16_hi(u[1])};
  }
  __device__ __forceinline__ void load_q(Q &q, const char *base, int64_t rowB, int tok, int lane, float mul) const {
    const T *row = reinterpret_cast<const T *>(base + (int64_t)tok * rowB) + 32 * (lane >> 5);
#pragma unroll
    for (int s = 0; s < 8; s++) {
      const f32x4 v = load4(row + 4 * s);
#pragma unroll
      for (int e = 0; e < 4; e++) q.f[4 * s + e] = v[e] * mul;
    }
  }
  // one request: 4 rows of 256 bytes; chunk = 16-byte chunk of the row (4 elements)
  __device__ static __forceinline__ void request(const char *row, int chunk, unsigned char *dst, uint32_t lds, int lane) {
    if (sizeof(T) == 4) {
      const char *src = row + 16 * chunk;
      asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(lds), "v"(src) : "memory", "m0");
    } else {
      *reinterpret_cast<f32x4 *>(dst + 16 * lane) = load4(reinterpret_cast<const T *>(row) + 4 * chunk);
    }
  }
  static __device__ __forceinline__ uint32_t place(int tok, int64_t) { return (uint32_t)tok; }
  __device__ __forceinline__ void issue_k(const char *base, int64_t rowB, const uint32_t (&at)[kReq], unsigned char *dst, uint32_t lds, int lane) const {
    const int ln = opaque(lane);              // (chunk numbers: put together here, not kept)
#pragma unroll
    for (int it = 0; it < kReq; it++)
      request(base + (int64_t)at[it] * rowB, (ln & 15) ^ ((4 * it + (ln >> 4)) & 15), dst + it * 1024, lds + it * 1024, lane);
  }
  __device__ __forceinline__ void issue_v(const char *base, int64_t rowB, const uint32_t (&at)[kReq], unsigned char *dst, uint32_t lds, int lane) const {
    const int ln = opaque(lane);
#pragma unroll
    for (int it = 0; it < kReq; it++)
      request(base + (int64_t)at[it] * rowB, (ln & 15) ^ (8 * (it & 1)), dst + it * 1024, lds + it * 1024, lane);
  }
  template <int NT>
  __device__ __forceinline__ void logits(const Q (&q)[NT], const unsigned char *slot, f32x16 (&s)[NT]) const {
#pragma unroll
    for (int nt = 0; nt < NT; nt++) s[nt] = f32x16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < 8; c++) {
      const f32x4 k4 = *reinterpret_cast<const f32x4 *>(slot + kbase + (kx ^ (16 * c)));
#pragma unroll
      for (int e = 0; e < 4; e++)
#pragma unroll
        for (int nt = 0; nt < NT; nt++) s[nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(k4[e], q[nt].f[4 * c + e], s[nt], 0, 0, 0);
    }
  }
  template <int NT, bool LO>
  __device__ __forceinline__ void weigh(const f32x16 (&w)[NT], const unsigned char *slot, f32x16 (&o)[NT][2], int) const {
#pragma unroll
    for (int e = 0; e < 16; e++)
#pragma unroll
      for (int dt = 0; dt < 2; dt++) {
        const float v = *reinterpret_cast<const float *>(slot + vrd[dt] + (8 * (e >> 2) + (e & 3)) * 256);
#pragma unroll
        for (int nt = 0; nt < NT; nt++) o[nt][dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(v, w[nt][e], o[nt][dt], 0, 0, 0);
      }
  }
  static __device__ __forceinline__ uint32_t screen(uint32_t one, int pass) { return screened(one, pass); }
  static __device__ __forceinline__ void store4out(float *p, f32x4 v) { *reinterpret_cast<f32x4 *>(p) = v; }
  static __device__ __forceinline__ void store4out(uint16_t *p, f32x4 v) {
    *reinterpret_cast<u32x2 *>(p) = u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
  }
};

constexpr float kBf16Max = 0x1.fep127f;
// Values e and e + 1 of eight as sums of up to three bf16 numbers each, the next the rounding of what those before leave: all 24
// bits of a value between 2^-103, below which the last parts may be subnormal, and kBf16Max, which the first part must not exceed.
// (Rows of values about 2^-112 are still as exact as others, of 2^-116 to 2e-6, of 2^-124 to 6e-4; with fp32 products 3e-7 throughout.)
template <int P>
__device__ __forceinline__ void split_pair(const float (&x)[8], bf16x8 (&p)[P], int e) {
  float a = x[e], b = x[e + 1];
#pragma unroll
  for (int i = 0; i < P; i++) {
    const uint32_t u = pack_bf16(a, b);
    const bf16x2 pk = __builtin_bit_cast(bf16x2, u);
    p[i][e] = pk[0];
    p[i][e + 1] = pk[1];
    if (i + 1 < P) {
      a -= bf16_lo(u);
      b -= bf16_hi(u);
    }
  }
}
template <int P>
__device__ __forceinline__ void split8(const float (&x)[8], bf16x8 (&p)[P]) {
#pragma unroll
  for (int e = 0; e < 8; e += 2) split_pair(x, p, e);
}

// fp32 precision from v_mfma_f32_32x32x16_bf16: each value in three bf16 parts (a row's of bf16 in one), and of the nine products
// of parts the six that count, smallest first.  The three left out are together at most 2^-24 of the whole (2^-27.5 rms of random
// values), as much as one rounding of the product; the error of the rows is smaller than with fp32 products, which round more often.
// That is 192 cycles of the matrix pipe for 16 k where v_mfma_f32_32x32x2_f32 takes 512.  (64 queries a step would share K's and V's
// parts, but the parts of 64 rows of Q leave too few registers: 30 are spilled.)
// A value that is not finite, or that bf16 rounds to infinity, has parts that are NaN.  K: the logits of a step that has some are
// formed once more, from whole values (walk_keys).  Q: load_q takes other parts.  V: rows whose sums are not finite are computed once
// more from whole values (walk_not_finite on Whole).
template <typename T>
struct StepF32 : StepF32Whole<T> {
  typedef StepF32Whole<T> Whole;
  static constexpr bool kParts = true;
  static constexpr int KP = sizeof(T) == 4 ? 3 : 1;      // parts of a value of K or V
  struct Q { bf16x8 f[4][3]; };                          // [channels 8 s .. of this half][part]
  __device__ __forceinline__ void load_q(Q &q, const char *base, int64_t rowB, int tok, int lane, float mul) const {
    const T *row = reinterpret_cast<const T *>(base + (int64_t)tok * rowB) + 32 * (lane >> 5);
    float top = 0.f;
    auto load8 = [&](const T *from, float (&x)[8]) {
#pragma unroll
      for (int c = 0; c < 2; c++) {
        const f32x4 v = Whole::load4(from + 4 * c);
#pragma unroll
        for (int e = 0; e < 4; e++) x[4 * c + e] = v[e] * mul;
      }
    };
#pragma unroll
    for (int s = 0; s < 4; s++) {
      float x[8];
      load8(row + 8 * s, x);
#pragma unroll
      for (int e = 0; e < 8; e++) top = max_abs(top, x[e]);
      split8(x, q.f[s]);
    }
    // Values whose first part would not be finite: the largest bf16 number in front, or, for one that is not finite itself, nothing
    // but the last part, which is multiplied with a key's first part alone.
    if (__builtin_expect(__any(!(top < kBf16Max)), 0)) {
      row += opaque(0);
#pragma unroll
      for (int s = 0; s < 4; s++) {
        float x[8];
        load8(row + 8 * s, x);
#pragma unroll
        for (int e = 0; e < 8; e++) {
          const float size = __builtin_fabsf(x[e]);
          if (!(size < kBf16Max)) {
            const float most = size < INFINITY ? __builtin_copysignf(kBf16Max, x[e]) : 0.f, rest = x[e] - most;
            const __bf16 mid = (__bf16)(size < INFINITY ? rest : 0.f);
            q.f[s][0][e] = (__bf16)most;
            q.f[s][1][e] = mid;
            q.f[s][2][e] = (__bf16)(rest - (float)mid);
          }
        }
      }
    }
  }
  // c += a b of values in KP and 3 parts.  between(m): what is to stand behind product m of kProducts; the fences keep it there,
  // since the scheduler would put the vector instructions first and the products, which then wait for each other, behind them
  // (28x28, 7x7 blocks 24.3 -> 23.7 us a call, 16x16 14.8 -> 14.1; large grids, bound by their transfers, as before).
  static constexpr int kProducts = KP == 3 ? 6 : 3;
  template <class F>
  static __device__ __forceinline__ void product(const bf16x8 (&a)[KP], const bf16x8 (&b)[3], f32x16 &c, F between) {
    int m = 0;
#pragma unroll
    for (int order = 2; order >= 0; order--)
#pragma unroll
      for (int i = 0; i < KP; i++)
        if (order - i >= 0) {
          c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[order - i], c, 0, 0, 0);
          between(m++);
          __builtin_amdgcn_sched_barrier(0);
        }
  }
  // pairs [from, to) of the four of x that stand behind product m
  template <int P>
  static __device__ __forceinline__ void split_behind(int m, const float (&x)[8], bf16x8 (&p)[P], int from, int to) {
#pragma unroll
    for (int i = 0; i < to - from; i++)
      if (i * kProducts / (to - from) == m) split_pair(x, p, 2 * (from + i));
  }
  template <int NT>
  __device__ __forceinline__ void logits(const Q (&q)[NT], const unsigned char *slot, f32x16 (&s)[NT]) const {
    static_assert(NT == 1, "32 queries");
    const uint32_t kx = (uint32_t)opaque((int)this->kx);     // (eight addresses otherwise live through the walk)
    float x[4][8];
#pragma unroll
    for (int c = 0; c < 8; c++) {
      const f32x4 k4 = *reinterpret_cast<const f32x4 *>(slot + this->kbase + (kx ^ (16 * c)));
#pragma unroll
      for (int e = 0; e < 4; e++) x[c >> 1][4 * (c & 1) + e] = k4[e];
    }
    s[0] = f32x16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    bf16x8 k[2][KP];
    split8(x[0], k[0]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < 4; t++)
      product(k[t & 1], q[0].f[t], s[0], [&](int m) {
        if (t < 3) split_behind(m, x[t < 3 ? t + 1 : 3], k[(t + 1) & 1], 0, 4);
      });
  }
  // The logits from whole values, with key l32's row read from memory: its slot may be the next step's already.
  __device__ __forceinline__ void whole_logits(const Q &q, const char *row, int lane, f32x16 &s) const {
    const T *k = reinterpret_cast<const T *>(row) + 32 * (lane >> 5);
    s = f32x16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < 8; c++) {
      const f32x4 k4 = Whole::load4(k + 4 * c);
#pragma unroll
      for (int e = 0; e < 4; e += 2) {
        uint32_t p[3];
#pragma unroll
        for (int i = 0; i < 3; i++) {         // (opaque: put together here, not kept through the walk)
          const bf16x8 &f = q.f[c >> 1][i];
          p[i] = (uint32_t)opaque(__builtin_bit_cast(int, bf16x2{f[4 * (c & 1) + e], f[4 * (c & 1) + e + 1]}));
        }
        s = __builtin_amdgcn_mfma_f32_32x32x2f32(k4[e], bf16_lo(p[0]) + (bf16_lo(p[1]) + bf16_lo(p[2])), s, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_32x32x2f32(k4[e + 1], bf16_hi(p[0]) + (bf16_hi(p[1]) + bf16_hi(p[2])), s, 0, 0, 0);
      }
    }
  }
  struct V { float x[4][8]; };                // [2 sp + dt]
  __device__ __forceinline__ void load_v(V &v, const unsigned char *slot) const {
    auto &x = v.x;
#pragma unroll
    for (int g = 0; g < 4; g++)
#pragma unroll
      for (int e = 0; e < 8; e++)
        x[g][e] = *reinterpret_cast<const float *>(slot + this->vrd[g & 1] + (16 * (g >> 1) + 8 * (e >> 2) + (e & 3)) * 256);
  }
  __device__ __forceinline__ void weigh(const f32x16 &w, const V &vv, f32x16 (&o)[2]) const {
    const auto &x = vv.x;
    float y[2][8];                            // weights: [sp]
#pragma unroll
    for (int e = 0; e < 16; e++) y[e >> 3][e & 7] = w[e];
    bf16x8 pw[2][3], v[2][KP];
    split8(y[0], pw[0]);
    split8(x[0], v[0]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int g = 0; g < 4; g++)
      product(v[g & 1], pw[g >> 1], o[g & 1], [&](int m) {
        if (g < 3) split_behind(m, x[g < 3 ? g + 1 : 3], v[(g + 1) & 1], 0, 4);
        if (g < 2) split_behind(m, y[1], pw[1], 2 * g, 2 * g + 2);
      });
  }
};

// LDS of a wave: the K ring, the V ring, then 1 KB for tokens in flight (four steps' worth, 256 bytes
// each) and 128 bytes of key codes.  After the walk the rings hold the wave's partial output.
constexpr int kWaveRings = 16384, kWaveAux = 1024 + 128, kWaveLds = kWaveRings + kWaveAux;
constexpr int kWindowMl = 4 * 2 * 64 * 4;                    // (max, sum) per wave and query
constexpr int kWindowLds = 4 * kWaveLds + kWindowMl;         // two workgroups per CU
constexpr float kNoMax = -1e30f;
constexpr float kLargeSum = 1e30f;                           // a sum beyond this may be about to leave fp32's range

// State of 32*NT queries: running reference m (log2 units), sum l (this half-wave's keys), output.
template <class S, int NT>
struct WaveAcc {
  typename S::Q q[NT];
  f32x16 o[NT][2];
  float m[NT], l[NT];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int nt = 0; nt < NT; nt++) {
      m[nt] = kNoMax;
      l[nt] = 0.f;
#pragma unroll
      for (int e = 0; e < 16; e++) { o[nt][0][e] = 0.f; o[nt][1][e] = 0.f; }
    }
  }
  // The reference is the first step's maximum and normally stays: a weight is exp2 of how far a logit
  // lies above it, and neither fp32 nor bf16 lose anything on weights up to 2^100.  A wave whose sums
  // then turn out too large (or not finite) walks its keys once more and keeps the reference at the
  // largest logit so far: weights are then at most 1, whatever the values they multiply.
  __device__ __forceinline__ bool exceeds(float limit) const {
    float big = 0.f;
#pragma unroll
    for (int nt = 0; nt < NT; nt++) {
      big = max_abs(big, l[nt]);
#pragma unroll
      for (int e = 0; e < 16; e++) big = max_abs(max_abs(big, o[nt][0][e]), o[nt][1][e]);
    }
    return __any(!(big < limit));
  }
  __device__ __forceinline__ void reference(const f32x16 &s, int nt, float c) {
    float a = fmaxf(s[0], s[1]), b = fmaxf(s[2], s[3]);
#pragma unroll
    for (int e = 4; e < 16; e += 4) {
      a = fmaxf(fmaxf(a, s[e]), s[e + 1]);
      b = fmaxf(fmaxf(b, s[e + 2]), s[e + 3]);
    }
    const float top = half_swap_max(fmaxf(a, b)) * c;
    if (__any(top > m[nt])) {
      const float m_new = fmaxf(m[nt], top);
      const float alpha = __builtin_amdgcn_exp2f(m[nt] - m_new);
      m[nt] = m_new;
      l[nt] *= alpha;
#pragma unroll
      for (int e = 0; e < 16; e++) { o[nt][0][e] *= alpha; o[nt][1][e] *= alpha; }
    }
  }
  // logits -> weights, whose sum it gives back
  __device__ __forceinline__ float weights(f32x16 &s, int nt, float c) {
    float l0 = 0.f, l1 = 0.f;
#pragma unroll
    for (int e = 0; e < 16; e += 2) {
      s[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e], c, -m[nt]));
      s[e + 1] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e + 1], c, -m[nt]));
      l0 += s[e];
      l1 += s[e + 1];
    }
    l[nt] += l0 + l1;
    return l0 + l1;
  }
};

// n steps of a wave with two ring slots and 64 queries, software-pipelined: while the weights of one half of the
// queries are taken and multiplied with V, the logits of the other half (of the next step) are formed, a
// matrix instruction to every seven vector instructions, so that one wave keeps both pipes busy.  (Phase
// after phase, two waves on a SIMD took the sum of their vector and matrix time: they fall into step.)
// FIXED: fix() has something to do in every step, not only in the first and the last.  Arguments as for
// walk_keys below.
template <class S, bool RING, bool FIXED, class KeyToken, class KeyEntry, class FixToken, class Fix>
__device__ __forceinline__ void walk_keys_pipelined(const S &st, WaveAcc<S, 2> &a, const char *kb, const char *vb, int64_t rowB,
                                                    unsigned char *wsm, int n, float c, bool careful, int lane, KeyToken key_token,
                                                    KeyEntry key_entry, FixToken fix_token, Fix fix) {
  static_assert(S::kDepth == 2, "two slots per ring");
  constexpr int R = S::kReq, TL = RING ? 1 : 0;
  if (n <= 0) return;
  const uint32_t lds = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)((__attribute__((address_space(3))) unsigned char *)wsm));
  n = __builtin_amdgcn_readfirstlane(n);
  constexpr int kV = 2 * S::kHalf;            // V ring behind the K ring
  int *const ring = reinterpret_cast<int *>(wsm + kWaveRings);
  auto request_tokens = [&](int i) {
    const int32_t *src = key_entry(i);
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, off"
                 :: "s"(__builtin_amdgcn_readfirstlane(lds + kWaveRings + (uint32_t)(i & 3) * 256u)), "v"(src) : "memory", "m0");
  };
  constexpr int rpr = 32 / R;                 // rows per request
  // places of K's and, one step behind, V's next rows
  uint32_t tk[R], tv[R];
  auto tokens = [&](int i) {
    const uint32_t t = S::place(RING ? fix_token(i, lane & 31, ring[(i & 3) * 64 + (lane & 31)]) : key_token(i), rowB);
#pragma unroll
    for (int it = 0; it < R; it++) {
      tv[it] = tk[it];
      tk[it] = __shfl(t, it * rpr + st.rrow);
    }
  };
  auto issue_k = [&](int slot) { const int o = slot * S::kHalf; st.issue_k(kb, rowB, tk, wsm + o, lds + o, lane); };
  auto issue_v = [&](int slot, const uint32_t (&t)[R]) { const int o = kV + slot * S::kHalf; st.issue_v(vb, rowB, t, wsm + o, lds + o, lane); };

  // order of requests: K0; K1 V0; K2 V1; then at the end of step i K(i+3) V(i+2)
  if (RING) {
#pragma unroll
    for (int i = 0; i < 4; i++) request_tokens(i);
    wait_vm<1>();
  }
  tokens(0);
  issue_k(0);
  if (n > 1) {
    tokens(1);
    issue_k(1);
    issue_v(0, tv);
  } else {
    issue_v(0, tk);
  }
  f32x16 s0, s1;                              // logits of queries 0..31 and 32..63
  typename S::K kf;
  typename S::V vf;
  // the output product behind: none yet
  bf16x8 open = {};
  vf.f[1][0] = vf.f[1][1] = open;
  f32x4 l0 = {0.f, 0.f, 0.f, 0.f}, l1 = l0;   // sums since the reference was last raised
  // the first step's logits; then K2 takes its slot
  if (n > 1) wait_vm<2 * R>();
  else wait_vm<R>();
  st.load_k(kf, wsm);
  s0 = st.product(kf, a.q[0]);
  fix(0, 0, s0);
  a.reference(s0, 0, c);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  if (n > 2) {
    tokens(2);
    issue_k(0);
    if (RING) request_tokens(4);
    issue_v(1, tv);
  } else if (n > 1) {
    issue_v(1, tk);
  }
  // a higher reference for half nt, whose output product is not the open one
  auto take_sums = [&](int nt, f32x4 &l) {
    a.l[nt] += S::row_sum(l, lane);
    l = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  auto raise = [&](int nt, const f32x16 &s) {
    take_sums(nt, nt ? l1 : l0);
    a.reference(s, nt, c);
  };
  // step i, whose V is in slot `odd`; `odd` = i & 1 is a constant at each place of use
  auto step = [&](auto first_c, int i, int odd) {
    constexpr bool first = decltype(first_c)::value;
    const int rem = n - 1 - i;
    // K of step i + 1 and V of step i.  Behind them: K of step i + 2 (and a token request), V of step i + 1.
    if (rem >= 2) wait_vm<2 * R + TL>();
    else if (rem == 1) wait_vm<R>();
    else wait_vm<0>();
    const bool special = FIXED || careful || first || rem <= 1;
    const unsigned char *vslot = wsm + kV + odd * S::kHalf;
    st.load_v(vf, vslot, 0);
    st.template half_step<true>(s0, c, -a.m[0], l0, a.o[0], l1, a.o[1], open, vf, vslot, kf, a.q[1], s1);
    const bool rest = first && st.exact > 0;
    if (rest) a.l[0] += st.add_rest(s0, vslot, a.o[0], lane);
    if (special) {
      fix(i, 1, s1);
      if (careful || first) raise(1, s1);
    }
    st.load_k(kf, wsm + (odd ^ 1) * S::kHalf);      // (behind the last step: what the slot holds, not used)
    st.template half_step<false>(s1, c, -a.m[1], l1, a.o[1], l0, a.o[0], open, vf, vslot, kf, a.q[0], s0);
    if (rest) a.l[1] += st.add_rest(s1, vslot, a.o[1], lane);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // both slots have been read
    if (rem >= 3) {
      tokens(i + 3);
      issue_k(odd ^ 1);
      if (RING) request_tokens(i + 5);
      issue_v(odd, tv);
    } else if (rem == 2) {
      issue_v(odd, tk);
    }
    if (special && rem > 0) {
      fix(i + 1, 0, s0);
      if (careful) raise(0, s0);
    }
  };
  // (the first step by itself: what only it does, in the loop behind a branch, made 100 x 100 patches 97 -> 100 us)
  step(std::true_type{}, 0, 0);
  for (int i = 1; i < n; i += 2) {
    step(std::false_type{}, i, 1);
    if (i + 1 < n) step(std::false_type{}, i + 1, 0);
  }
#pragma unroll
  for (int dt = 0; dt < 2; dt++) a.o[1][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf.f[1][dt], open, a.o[1][dt], 0, 0, 0);
  st.add_weights(l1, open);
  take_sums(0, l0);
  take_sums(1, l1);
  wait_vm<0>();                               // (token requests past the end)
}

// n steps of a wave.  key_token(i): token of key `lane & 31` of step i; with RING the tokens are
// read from memory instead: key_entry(i) is where that token stands, fix_token(i, row, tok) the last
// word on it.  fix(i, nt, s) edits the logits of step i and issues exactly E stores, screen(v) the 32 rows of V in
// LDS.  Vector memory requests complete in issue order, so the waits count how many younger ones may still be in flight.
struct Unscreened {
  __device__ __forceinline__ void operator()(unsigned char *) const {}
};
template <class S, int NT, bool WITH_V, bool RING, bool LO, int E, class KeyToken, class KeyEntry, class FixToken, class Fix,
          class Screen = Unscreened>
__device__ __forceinline__ void walk_keys(const S &st, WaveAcc<S, NT> &a, const char *kb, const char *vb, int64_t rowB,
                                          unsigned char *wsm, int n, float c, bool careful, int lane, KeyToken key_token,
                                          KeyEntry key_entry, FixToken fix_token, Fix fix, Screen screen = Screen()) {
  // (without V the K ring takes the whole space: twice the slots)
  constexpr int D = WITH_V ? S::kDepth : 2 * S::kDepth, R = S::kReq, TL = RING ? 1 : 0;
  if (n <= 0) return;
  const uint32_t lds = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)((__attribute__((address_space(3))) unsigned char *)wsm));
  n = __builtin_amdgcn_readfirstlane(n);
  constexpr int kV = D * S::kHalf;            // V ring behind the K ring
  int *const ring = reinterpret_cast<int *>(wsm + kWaveRings);
  auto request_tokens = [&](int i) {
    const int32_t *src = key_entry(i);
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, off"
                 :: "s"(__builtin_amdgcn_readfirstlane(lds + kWaveRings + (uint32_t)(i & 3) * 256u)), "v"(src) : "memory", "m0");
  };
  constexpr int rpr = 32 / R;                 // rows per request
  uint32_t at[R];                             // where the rows of this lane's requests stand
  auto tokens = [&](int i) {
    const int rrow = R > 4 ? opaque(st.rrow) : st.rrow;      // (fp32: eight lane numbers otherwise live through the walk)
    if (RING) {
      // (lane l of each half turns the token of key l into its row's place)
      const uint32_t t = S::place(fix_token(i, lane & 31, ring[(i & 3) * 64 + (lane & 31)]), rowB);
#pragma unroll
      for (int it = 0; it < R; it++) at[it] = __shfl(t, it * rpr + rrow);
    } else {
      const uint32_t t = S::place(key_token(i), rowB);
#pragma unroll
      for (int it = 0; it < R; it++) at[it] = __shfl(t, it * rpr + rrow);
    }
  };
  auto issue_k = [&](int slot) { const int o = slot * S::kHalf; st.issue_k(kb, rowB, at, wsm + o, lds + o, lane); };
  auto issue_v = [&](int slot) { const int o = kV + slot * S::kHalf; if (WITH_V) st.issue_v(vb, rowB, at, wsm + o, lds + o, lane); };

  if (RING) {
#pragma unroll
    for (int i = 0; i <= D; i++) request_tokens(i);
    wait_vm<1>();
  }
#pragma unroll
  for (int i = 0; i < D; i++)
    if (i < n) {
      tokens(i);
      issue_k(i);
      if (RING && i == D - 1) request_tokens(D + 1);
      issue_v(i);
    }
  constexpr int kNext = D == 2 ? 2 * R : 0;   // requests of the step behind (two slots)
  // slot: i % D, a constant at each place of use
  auto step = [&](int i, int slot) {
    const int rem = n - 1 - i;                // steps behind this one
    // K of step i.  Behind it with two slots: V of step i, the stores of the step before, K and V
    // of the next step and, in the ring, one token request; with one slot: V of step i.  (Without V:
    // K of up to D - 1 further steps and at least one step's stores.)
    if (WITH_V) {
      constexpr int kStored = D == 2 ? E : 0;
      if (i == 0) {
        if (rem >= D - 1) wait_vm<R + kNext>();
        else wait_vm<R>();
      } else if (rem >= D) wait_vm<R + kNext + kStored + (D - 1) * TL>();
      else if (D == 2 && rem == 1) wait_vm<R + kNext + kStored>();
      else wait_vm<R + kStored>();
    } else {
      const int behind = rem < D - 1 ? rem : D - 1;
      if (i == 0) {
        if (behind == 3) wait_vm<3 * R>();
        else if (behind == 2) wait_vm<2 * R>();
        else if (behind == 1) wait_vm<R>();
        else wait_vm<0>();
      } else {
        if (behind == 3) wait_vm<3 * R + E>();
        else if (behind == 2) wait_vm<2 * R + E>();
        else if (behind == 1) wait_vm<R + E>();
        else wait_vm<E>();
      }
    }
    f32x16 s[NT];
    st.template logits<NT>(a.q, wsm + slot * S::kHalf, s);
#pragma unroll
    for (int nt = 0; nt < NT; nt++) fix(i, nt, s[nt]);
    if (rem >= D) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the slot has been read
      tokens(i + D);
      issue_k(slot);
      if (RING) request_tokens(i + D + 2);
    }
    float before[NT], sum[NT];
#pragma unroll
    for (int nt = 0; nt < NT; nt++) {
      if (careful || i == 0) a.reference(s[nt], nt, c);
      before[nt] = a.l[nt];
      sum[nt] = a.weights(s[nt], nt, c);
    }
    // Parts: where a logit is NaN, which whole values may make an infinity, the step's once more.  (Asked of the sum of weights, behind
    // V's reads: 28x28, 7x7 blocks 23.67 -> 23.86 us, 64x64, four images 267 -> 268; asked of the logits, which holds the next K back,
    // 1 to 3 % more.  With one infinite key a head 27 and 269; a second walk on whole values for the rows that see it, 42 and 415.)
    auto mend = [&]() {
      if constexpr (S::kParts) {
        if (!__builtin_expect(__any(sum[0] != sum[0]), 0)) return;
        const int tok = RING ? fix_token(i, lane & 31, ring[(i & 3) * 64 + (lane & 31)]) : key_token(i);
        st.whole_logits(a.q[0], kb + (int64_t)tok * rowB, lane, s[0]);
        fix(i, 0, s[0]);                      // (stores more than are counted: a wait then waits for more, not for less)
        a.l[0] = before[0];
        if (careful || i == 0) a.reference(s[0], 0, c);
        a.weights(s[0], 0, c);
      }
    };
    if (!WITH_V) mend();
    if (WITH_V) {
      // V of step i.  Behind it: the next step (two slots), this step's stores, K of step i + D
      if (rem >= D) wait_vm<kNext + E + R + (D - 1) * TL>();
      else if (D == 2 && rem == 1) wait_vm<kNext + E>();
      else wait_vm<E>();
      screen(wsm + kV + slot * S::kHalf);
      if constexpr (S::kParts) {
        typename S::V v;
        st.load_v(v, wsm + kV + slot * S::kHalf);
        __builtin_amdgcn_sched_barrier(0);
        mend();
        st.weigh(s[0], v, a.o[0]);
      } else {
        st.template weigh<NT, LO>(s, wsm + kV + slot * S::kHalf, a.o, lane);
      }
      if constexpr (S::kDepth == 2 && NT == 2)
        if (slot == 0 && i == 0 && st.exact > 0)
#pragma unroll
          for (int nt = 0; nt < NT; nt++) st.add_rest(s[nt], wsm + kV, a.o[nt], lane);
      if (rem >= D) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        issue_v(slot);
      }
    }
  };
  for (int i = 0; i < n; i += D) {
    step(i, 0);
    if (D > 1 && i + 1 < n) step(i + 1, 1);
    if (D > 2 && i + 2 < n) step(i + 2, 2);
    if (D > 3 && i + 3 < n) step(i + 3, 3);
  }
  wait_vm<0>();                               // (token requests past the end)
}

// n steps of a wave whose output sums are not finite after a careful walk: a row gets what the keys it sees give,
// infinities of one sign as such, of both signs and NaN as NaN.  The walks above let more in: a pair that is masked and
// a key number past the end have weight 0, and 0 times inf is NaN.  Three passes: which output values see +inf or NaN
// (weights 1 and 0, V 1 where it is that), which see -inf or NaN, then the output with the finite values of V.
// hide(i, nt, s): -inf in place of the logits of step i that do not count.
template <class S, int NT, bool RING, bool LO, class KeyToken, class KeyEntry, class FixToken, class Hide>
__device__ __forceinline__ void walk_not_finite(const S &st, WaveAcc<S, NT> &a, const char *kb, const char *vb, int64_t rowB,
                                                unsigned char *wsm, int n, float c, int lane, KeyToken key_token,
                                                KeyEntry key_entry, FixToken fix_token, Hide hide) {
  uint32_t sees[2][NT] = {};                  // bit 16 dt + e
#pragma unroll 1
  for (int pass = 0; pass < 3; pass++) {
    a.clear();
    walk_keys<S, NT, true, RING, LO, 0>(
      st, a, kb, vb, rowB, wsm, n, c, true, lane, key_token, key_entry, fix_token,
      [&](int i, int nt, f32x16 &s) {
        if (pass < 2)
#pragma unroll
          for (int e = 0; e < 16; e++) s[e] = 0.f;
        hide(i, nt, s);
      },
      [&](unsigned char *v) {
#pragma unroll
        for (int i = 0; i < S::kHalf / 1024; i++) {
          uint4 *const x = reinterpret_cast<uint4 *>(v + 1024 * i + 16 * lane);
          const uint4 u = *x;
          *x = uint4{S::screen(u.x, pass), S::screen(u.y, pass), S::screen(u.z, pass), S::screen(u.w, pass)};
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      });
    if (pass == 2) break;
#pragma unroll
    for (int nt = 0; nt < NT; nt++) {
      uint32_t bits = 0;
#pragma unroll
      for (int e = 0; e < 16; e++) bits |= (a.o[nt][0][e] > 0.f ? 1u << e : 0u) | (a.o[nt][1][e] > 0.f ? 0x10000u << e : 0u);
      sees[0][nt] = pass == 0 ? bits : sees[0][nt];
      sees[1][nt] = pass == 0 ? 0u : bits;
    }
  }
#pragma unroll
  for (int nt = 0; nt < NT; nt++)
#pragma unroll
    for (int dt = 0; dt < 2; dt++)
#pragma unroll
      for (int e = 0; e < 16; e++) {
        const uint32_t bit = 1u << (16 * dt + e);
        a.o[nt][dt][e] += sees[0][nt] & bit ? INFINITY : 0.f;
        a.o[nt][dt][e] += sees[1][nt] & bit ? -INFINITY : 0.f;
      }
}

// ... of a step that works on parts: the queries (lane l32: token tok) from whole values
template <class S, bool RING, class... Args>
__device__ __forceinline__ void whole_rows(const S &st, WaveAcc<S, 1> &a, const char *qb, const char *kb, const char *vb, int64_t rowB,
                                           int tok, float scale, unsigned char *wsm, int n, float c, int lane, Args &&...args) {
  typedef typename S::Whole W;
  WaveAcc<W, 1> b;
  static_cast<const W &>(st).load_q(b.q[0], qb, rowB, tok, lane, scale);
  walk_not_finite<W, 1, RING, false>(st, b, kb, vb, rowB, wsm, n, c, lane, args...);
  a.o[0][0] = b.o[0][0];
  a.o[0][1] = b.o[0][1];
  a.m[0] = b.m[0];
  a.l[0] = b.l[0];
}

// a query tile's walk: pipelined where there are two slots
template <class S, int NT, bool RING, bool FIXED, class... Args>
__device__ __forceinline__ void window_walk(const S &st, WaveAcc<S, NT> &a, Args &&...args) {
  if constexpr (S::kDepth == 2 && NT == 2) walk_keys_pipelined<S, RING, FIXED>(st, a, args...);
  else walk_keys<S, NT, true, RING, false, 0>(st, a, args...);
}

// 16 channels of a row, o[at .. at+7] of the two half-waves' lanes, times inv, as bf16: the lane of half hh has channels
// 4*hh + 0..3 and 8 + 4*hh + 0..3 and gets, to store 16 bytes at once, channels 8*hh + 0..7.
__device__ __forceinline__ u32x4 row_pieces(const f32x16 &o, int at, float inv) {
  uint32_t u[4];
#pragma unroll
  for (int i = 0; i < 4; i++) u[i] = pack_bf16(o[at + 2 * i] * inv, o[at + 2 * i + 1] * inv);
  const auto x = __builtin_amdgcn_permlane32_swap(u[0], u[2], false, false), y = __builtin_amdgcn_permlane32_swap(u[1], u[3], false, false);
  return u32x4{x[0], y[0], x[1], y[1]};
}

// A wave's state -> LDS: output rows of 64 floats in its rings (16-byte chunk c of row r at c ^ (r & 15)),
// (max, sum) in ml.
template <class S, int NT>
__device__ __forceinline__ void park_state(const WaveAcc<S, NT> &a, unsigned char *wsm, float *ml, int lane) {
  const int l32 = lane & 31, hh = lane >> 5;
#pragma unroll
  for (int nt = 0; nt < NT; nt++) {
    const int row = 32 * nt + l32;
#pragma unroll
    for (int dt = 0; dt < 2; dt++)
#pragma unroll
      for (int ig = 0; ig < 4; ig++) {
        const f32x4 v = {a.o[nt][dt][4 * ig], a.o[nt][dt][4 * ig + 1], a.o[nt][dt][4 * ig + 2], a.o[nt][dt][4 * ig + 3]};
        *reinterpret_cast<f32x4 *>(wsm + row * 256 + 16 * ((8 * dt + 2 * ig + hh) ^ (row & 15))) = v;
      }
    const float l = half_swap_sum(a.l[nt]);
    if (hh == 0) {
      ml[2 * row] = a.m[nt];
      ml[2 * row + 1] = l;
    }
  }
}
__device__ __forceinline__ f32x4 parked(const unsigned char *smem, int w, int row, int chunk) {
  return *reinterpret_cast<const f32x4 *>(smem + w * kWaveLds + row * 256 + 16 * (chunk ^ (row & 15)));
}

// ------------------------------------------------------------------------------------------
// The global rows: workgroup `id` takes a chunk of kClsChunk keys for a group of global tokens of one
// head, 32 keys a step and wave, all rows of the group against the same K and V rows (which are
// read once however many global tokens there are).  Leaves the raw logits and one softmax partial
// (max, sum, weighted V sum) per row and chunk.  bf16: a group is 16 rows, in the operand's columns
// twice, so that the second product gets every weight as bf16 head and bf16 rest (and the rest of that).
// ------------------------------------------------------------------------------------------
struct GlobalRows {
  const void *q, *k, *v;
  int64_t sb, sh, st;      // strides in elements
  float scale;
  float *logits;           // [B, H, G, T] or NULL
  float *partials;         // [B, H*G, nchunks, 66]
  double nat;              // natural units of a step's exponents: what one of them is as a logit
};
template <class S> constexpr int global_group_rows() { return S::kDepth == 2 ? 16 : 32; }
// (a step's exponent is q.k * c with c = scale * log2(e) rounded to fp32; fp32 rows are scaled before)
template <class S>
inline GlobalRows global_rows(const ns_attn_desc &d, const void *q, const void *k, const void *v, float *logits, float *partials) {
  const double nat = S::kDepth == 2 ? (double)d.scale / (double)(d.scale * kLog2e) : 1.0 / (double)kLog2e;
  return GlobalRows{q, k, v, d.q_stride_b, d.q_stride_h, d.q_stride_t, d.scale, logits, partials, nat};
}

template <class S, bool WITH_V, bool LOGITS>
__device__ __forceinline__ void global_rows_chunk(const GlobalRows &p, int heads, int G, int T, int groups, int nchunks,
                                                  int id, unsigned char *smem, int wave, int lane) {
  typedef typename S::elem elem;
  constexpr bool kBf16 = S::kDepth == 2;
  constexpr int GR = global_group_rows<S>();
  const int chunk = id % nchunks, hg = id / nchunks, grp = hg % groups, bh = hg / groups;
  const int b = bh / heads, h = bh - b * heads;
  const int l32 = lane & 31, hh = lane >> 5;
  const char *qb = reinterpret_cast<const char *>(static_cast<const elem *>(p.q) + b * p.sb + h * p.sh);
  const char *kb = reinterpret_cast<const char *>(static_cast<const elem *>(p.k) + b * p.sb + h * p.sh);
  const char *vb = WITH_V ? reinterpret_cast<const char *>(static_cast<const elem *>(p.v) + b * p.sb + h * p.sh) : nullptr;
  const int64_t rowB = p.st * (int64_t)sizeof(elem);
  unsigned char *wsm = smem + wave * kWaveLds;
  S st;
  st.init(lane);
  WaveAcc<S, 1> a;
  a.clear();
  const int col = l32 & (GR - 1), g = grp * GR + col;
  st.load_q(a.q[0], qb, rowB, min(g, G - 1), lane, p.scale);
  const float c = kBf16 ? p.scale * kLog2e : kLog2e, lmul = kBf16 ? p.scale : 1.f;
  const int j0 = chunk * kClsChunk + 32 * wave;
  const int left = min(T - chunk * kClsChunk, kClsChunk);           // keys of this chunk
  const int steps = (left + 31) / 32, n = steps > wave ? (steps - wave + 3) / 4 : 0;
  // (the second set of columns and the rows past G write nothing)
  const bool writes = LOGITS && l32 < GR && g < G;
  float *lrow = LOGITS ? p.logits + ((size_t)(b * heads + h) * G + min(g, G - 1)) * T : nullptr;
  auto key_token = [&](int i) { return min(j0 + 128 * i + l32, T - 1); };
  auto no_entry = [](int) { return (const int32_t *)nullptr; };
  auto as_is = [](int, int, int t) { return t; };
  auto hide = [&](int i, int, f32x16 &s) {
    const int jb = j0 + 128 * i + 4 * hh;
    if (j0 + 128 * i + 32 > T)
#pragma unroll
      for (int e = 0; e < 16; e++) s[e] = jb + 8 * (e >> 2) + (e & 3) < T ? s[e] : -INFINITY;
  };
  for (bool careful = false;; careful = true) {
    walk_keys<S, 1, WITH_V, false, kBf16, LOGITS ? 16 : 0>(
      st, a, kb, vb, rowB, wsm, n, c, careful, lane, key_token, no_entry, as_is,
      [&](int i, int nt, f32x16 &s) {
        const int jb = j0 + 128 * i + 4 * hh;
        // (keys past the end are copies of the last one: their lanes store its logit once more)
        if (LOGITS && writes)
#pragma unroll
          for (int e = 0; e < 16; e++) store4(lrow + min(jb + 8 * (e >> 2) + (e & 3), T - 1), s[e] * lmul);
        hide(i, nt, s);
      });
    if (!a.exceeds(careful ? INFINITY : kLargeSum)) break;
    if (careful) {
      if constexpr (WITH_V && kBf16) walk_not_finite<S, 1, false, true>(st, a, kb, vb, rowB, wsm, n, c, lane, key_token, no_entry, as_is, hide);
      else if constexpr (WITH_V) whole_rows<S, false>(st, a, qb, kb, vb, rowB, min(g, G - 1), p.scale, wsm, n, c, lane, key_token, no_entry, as_is, hide);
      break;
    }
    a.clear();
  }
  float *ml = reinterpret_cast<float *>(smem + 4 * kWaveLds);
  park_state(a, wsm, ml + wave * 128, lane);
  __syncthreads();
  // thread = (row, 16-byte chunk of the output)
  for (int t = wave * 64 + lane; t < GR * 16; t += 256) {
    const int row = t >> 4, ch = t & 15, gr = grp * GR + row;
    if (gr >= G) continue;
    float M = ml[2 * row], L = 0.f;
#pragma unroll
    for (int w = 1; w < 4; w++) M = fmaxf(M, ml[w * 128 + 2 * row]);
    f32x4 O = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < 4; w++) {
      const float f = __builtin_amdgcn_exp2f(ml[w * 128 + 2 * row] - M);
      L = __builtin_fmaf(f, ml[w * 128 + 2 * row + 1], L);
      if (WITH_V) {
        f32x4 v = parked(smem, w, row, ch);
        if (kBf16) v += parked(smem, w, row + 16, ch);
#pragma unroll
        for (int e = 0; e < 4; e++) O[e] = __builtin_fmaf(f, v[e], O[e]);
      }
    }
    float *rec = p.partials + (((size_t)(b * heads + h) * G + gr) * nchunks + chunk) * kClsPartialFloats;
    // The record's maximum is a logit, M an exponent: what rounding the one to fp32 leaves goes into the sums.
    // (Left out, a log-sum-exp near 500 is off by a whole unit in the last place, 3e-5.)
    const double m = (double)M * p.nat;
    const float mr = (float)m, f0 = __builtin_amdgcn_exp2f((float)((m - (double)mr) * 1.4426950408889634));
    L *= f0;
#pragma unroll
    for (int e = 0; e < 4; e++) O[e] *= f0;
    if (ch == 0) {
      rec[0] = mr;
      rec[1] = L;
    }
    if (WITH_V) {
      *reinterpret_cast<f32x2 *>(rec + 2 + 4 * ch) = f32x2{O[0], O[1]};
      *reinterpret_cast<f32x2 *>(rec + 4 + 4 * ch) = f32x2{O[2], O[3]};
    }
  }
}

__device__ __forceinline__ void unpack8(const u32x4 &u, float (&x)[8]) {
  x[0] = bf16_lo(u[0]); x[1] = bf16_hi(u[0]); x[2] = bf16_lo(u[1]); x[3] = bf16_hi(u[1]);
  x[4] = bf16_lo(u[2]); x[5] = bf16_hi(u[2]); x[6] = bf16_lo(u[3]); x[7] = bf16_hi(u[3]);
}
// ------------------------------------------------------------------------------------------
// One global row in bf16 on the vector ALU, workgroup `id` = (head, chunk): lane = (key slot, 8-channel slice), 8 lanes
// per key row, all of a wave's 128 rows of K and then of V on their way at once.  For a single row the matrix
// instructions above are work for 15 or 31 padding columns.  Bound: HBM.  Past the caches (non-temporal
// loads): 0.7 % of a whole call with 16x16 blocks on 256x256.
// ------------------------------------------------------------------------------------------
constexpr int kScanLds = 4 * 64 * 4 + 16;    // bytes
__device__ __forceinline__ void global_row_chunk(const GlobalRows &p, int H, int T_, int nchunks, int id, unsigned char *smem,
                                                 int tid) {
  constexpr int kSteps = kClsChunk / (4 * 8);   // 4 waves x 8 keys per wave-step
  const int chunk = id % nchunks, bh = id / nchunks, b = bh / H, h = bh - b * H;
  const int wave = tid >> 6, lane = tid & 63, slot = lane >> 3, sub = lane & 7;
  const int64_t head = b * p.sb + h * p.sh + sub * 8;
  const uint16_t *k = static_cast<const uint16_t *>(p.k) + head, *v = static_cast<const uint16_t *>(p.v) + head;
  float (*const osum)[64] = reinterpret_cast<float (*)[64]>(smem);
  float *const red = reinterpret_cast<float *>(smem + 4 * 64 * 4);

  float q8[8];
  unpack8(*reinterpret_cast<const u32x4 *>(static_cast<const uint16_t *>(p.q) + head), q8);
#pragma unroll
  for (int e = 0; e < 8; e++) q8[e] *= p.scale;
  const int key0 = chunk * kClsChunk + wave * (kSteps * 8) + slot;
  u32x4 row[kSteps];                       // (clamped, not skipped: a branch would wait for each load)
#pragma unroll
  for (int i = 0; i < kSteps; i++)
    row[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(k + (int64_t)min(key0 + i * 8, T_ - 1) * p.st));
  float s[kSteps];
  float mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < kSteps; i++) {
    float k8[8];
    unpack8(row[i], k8);
    row[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(v + (int64_t)min(key0 + i * 8, T_ - 1) * p.st));
    float acc = 0.f;
#pragma unroll
    for (int e = 0; e < 8; e++) acc = __builtin_fmaf(q8[e], k8[e], acc);
    acc += __shfl_xor(acc, 1);
    acc += __shfl_xor(acc, 2);
    acc += __shfl_xor(acc, 4);
    s[i] = key0 + i * 8 < T_ ? acc : -INFINITY;
    mx = fmaxf(mx, s[i]);
  }
  mx = fmaxf(mx, __shfl_xor(mx, 8));
  mx = fmaxf(mx, __shfl_xor(mx, 16));
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  if (lane == 0) red[wave] = mx;
  __syncthreads();
  const float M = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));   // finite: chunk non-empty
  __syncthreads();
  float l = 0.f;
  float o8[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < kSteps; i++) {
    const bool in = key0 + i * 8 < T_;
    const float pr = __builtin_amdgcn_exp2f((s[i] - M) * kLog2e);
    float v8[8];
    unpack8(row[i], v8);
    l += pr;
#pragma unroll
    for (int e = 0; e < 8; e++) o8[e] = __builtin_fmaf(pr, in ? v8[e] : 0.f, o8[e]);
  }
  // (stores behind the loads: waiting for a load also waits for every older store)
  if (p.logits) {
    float *lrow = p.logits + ((size_t)b * H + h) * T_;
#pragma unroll
    for (int i = 0; i < kSteps; i++)
      if (sub == 0 && key0 + i * 8 < T_) lrow[key0 + i * 8] = s[i];
  }
  // across the 8 key slots of the wave (not across channel slices)
#pragma unroll
  for (int sft = 8; sft < 64; sft <<= 1) {
    l += __shfl_xor(l, sft);
#pragma unroll
    for (int e = 0; e < 8; e++) o8[e] += __shfl_xor(o8[e], sft);
  }
  if (lane == 0) red[wave] = l;
  if (slot == 0) {
#pragma unroll
    for (int e = 0; e < 8; e++) osum[wave][sub * 8 + e] = o8[e];
  }
  __syncthreads();
  float *rec = p.partials + (((size_t)b * H + h) * nchunks + chunk) * kClsPartialFloats;
  if (tid == 0) {
    rec[0] = M;
    rec[1] = (red[0] + red[1]) + (red[2] + red[3]);
  }
  if (tid < 64) rec[2 + tid] = (osum[0][tid] + osum[1][tid]) + (osum[2][tid] + osum[3][tid]);
}

// ------------------------------------------------------------------------------------------
// One launch: a workgroup owns a query tile, whose keys the four waves share out step by step; the waves' partial
// states are merged through LDS.  Others own chunks of the global rows.  Bound at small sizes by the latency of the few steps a wave walks, at larger ones by the
// instruction issue of the steps while both waves of a SIMD are there, and by how often only one is
// (100x100 grid, 16 heads, 2 images, five global tokens: 95 us, matrix pipes 23 % busy, vector ALUs
// 41 %, 1.4 waves per SIMD, a quarter of a wave's time in waits).
// ------------------------------------------------------------------------------------------
struct WindowParams {
  GlobalRows r;            // q, k, v, strides, scale; logits and partials for the global rows
  void *out;
  int64_t osb, osh, ost;
  WindowGeom g;
};

template <class S, int NT, bool LISTS, bool MASK, int KS>
__device__ __forceinline__ void window_attention(const WindowParams &p, unsigned char *smem) {
  typedef typename S::elem elem;
  constexpr int QT = 32 * NT;
  constexpr bool kBf16 = S::kDepth == 2;
  const WindowGeom &g = p.g;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int gid = (int)blockIdx.x - g.rows_at;
  if (gid >= 0 && gid < g.row_wgs) {
    if (p.r.logits)
      global_rows_chunk<S, true, true>(p.r, g.heads, g.n_global, g.tokens, g.global_groups, g.nchunks, gid, smem, wave, lane);
    else
      global_rows_chunk<S, true, false>(p.r, g.heads, g.n_global, g.tokens, g.global_groups, g.nchunks, gid, smem, wave, lane);
    return;
  }
  const int bid = (int)blockIdx.x - g.tiles_at;
  if (bid < 0 || bid >= 8 * g.per_xcd) return;       // (the rows' workgroups are filled up to a multiple of 8)
  // waves part, part + 1, .. part + KS - 1 share a tile
  const int part = wave & (KS - 1), id = window_tile_id(g, bid) * (4 / KS) + wave / KS;
  WindowTile<LISTS, QT> w;
  // (a wave without a tile takes part in the barrier below and touches no memory: with an empty tile
  // there is no query slot, hence no token to look up)
  const bool live = id < g.tiles && w.init(g, id, lane);
  if (!live) {
    if (KS == 4 || KS == 1) return;            // (with KS = 4 the whole workgroup returns)
    w.b = w.h = w.qcnt = 0;
  }
  const int l32 = lane & 31, hh = lane >> 5;
  const int64_t head = w.b * p.r.sb + w.h * p.r.sh, rowB = p.r.st * (int64_t)sizeof(elem);
  const char *qb = reinterpret_cast<const char *>(static_cast<const elem *>(p.r.q) + head);
  const char *kb = reinterpret_cast<const char *>(static_cast<const elem *>(p.r.k) + head);
  const char *vb = reinterpret_cast<const char *>(static_cast<const elem *>(p.r.v) + head);
  unsigned char *wsm = smem + wave * kWaveLds;
  float *ml = reinterpret_cast<float *>(smem + 4 * kWaveLds);
  S st;
  st.init(lane);
  if constexpr (kBf16) st.exact = part == 0 ? min(g.n_global, 8) : 0;
  WaveAcc<S, NT> a;
  a.clear();
  if (KS != 2 || live) {
  const int steps = (w.nkeys + 31) / 32, n = steps > part ? (steps - part + KS - 1) / KS : 0;
  const float inv_block = 1.f / (float)g.block;
  uint32_t qcode[NT];
#pragma unroll
  for (int nt = 0; nt < NT; nt++) {
    st.load_q(a.q[nt], qb, rowB, w.query(g, 32 * nt + l32), lane, p.r.scale);
    if (MASK) qcode[nt] = w.query_code(g, 32 * nt + l32, inv_block);
  }
  uint32_t *const codes = reinterpret_cast<uint32_t *>(wsm + kWaveRings + 1024);
  auto key0 = [&](int i) { return 32 * (KS * i + part); };       // first key of this wave's step i
  // (squares of several blocks: a query may see none of a step's keys, so only a first step with the
  // global tokens in it gives a reference)
  const float c = kBf16 ? p.r.scale * kLog2e : kLog2e;
  auto key_token = [&](int i) { return w.key(g, key0(i) + l32); };
  auto key_entry = [&](int i) { return w.key_entry(g, key0(i) + l32); };
  auto fix_token = [&](int i, int row, int t) { return key0(i) + row < g.n_global ? key0(i) + row : t; };
  auto hide = [&](int i, int nt, f32x16 &s) {
    if (MASK) {
      if (nt == 0) {
        codes[l32] = w.key_code(g, key0(i) + l32, inv_block);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      }
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        const uint4 kc = *reinterpret_cast<const uint4 *>(codes + 8 * q4 + 4 * hh);
        const uint32_t k4[4] = {kc.x, kc.y, kc.z, kc.w};
#pragma unroll
        for (int e = 0; e < 4; e++) s[4 * q4 + e] = (k4[e] & ~qcode[nt]) == 0 ? s[4 * q4 + e] : -INFINITY;
      }
    } else if (key0(i) + 32 > w.nkeys) {
      const int jb = key0(i) + 4 * hh;
#pragma unroll
      for (int e = 0; e < 16; e++) s[e] = jb + 8 * (e >> 2) + (e & 3) < w.nkeys ? s[e] : -INFINITY;
    }
  };
  for (bool careful = MASK && part != 0;; careful = true) {
    window_walk<S, NT, LISTS, MASK>(st, a, kb, vb, rowB, wsm, n, c, careful, lane, key_token, key_entry, fix_token, hide);
    if (!a.exceeds(careful ? INFINITY : kLargeSum)) break;
    if (careful) {
      if constexpr (kBf16) {
        walk_not_finite<S, NT, LISTS, false>(st, a, kb, vb, rowB, wsm, n, c, lane, key_token, key_entry, fix_token, hide);
      } else {
        whole_rows<S, LISTS>(st, a, qb, kb, vb, rowB, w.query(g, l32), p.r.scale, wsm, n, c, lane, key_token, key_entry, fix_token, hide);
      }
      break;
    }
    a.clear();
  }
  }
  elem *ob = static_cast<elem *>(p.out) + w.b * p.osb + w.h * p.osh;
  if (KS == 1) {
    // lane (query, hh) owns channels 32*dt + 8*ig + 4*hh + 0..3
#pragma unroll
    for (int nt = 0; nt < NT; nt++) {
      const float inv = 1.f / half_swap_sum(a.l[nt]);
      if (32 * nt + l32 >= w.qcnt) continue;
      elem *row = ob + (int64_t)w.query(g, 32 * nt + l32) * p.ost + 4 * hh;
#pragma unroll
      for (int dt = 0; dt < 2; dt++)
#pragma unroll
        for (int ig = 0; ig < 4; ig++)
          S::store4out(row + 32 * dt + 8 * ig, f32x4{a.o[nt][dt][4 * ig] * inv, a.o[nt][dt][4 * ig + 1] * inv,
                                                     a.o[nt][dt][4 * ig + 2] * inv, a.o[nt][dt][4 * ig + 3] * inv});
    }
    return;
  }
  park_state(a, wsm, ml + wave * 128, lane);
  __syncthreads();
  // merge in wave order, normalise, store: 16 lanes per row, 4 KS rows of the tile per pass
  const int w0 = wave & ~(KS - 1);             // first wave of this tile
#pragma unroll
  for (int ps = 0; ps < QT / (4 * KS); ps++) {
    const int row = 4 * KS * ps + 4 * part + (lane >> 4), ch = lane & 15;
    float M = ml[w0 * 128 + 2 * row], L = 0.f;
#pragma unroll
    for (int x = 1; x < KS; x++) M = fmaxf(M, ml[(w0 + x) * 128 + 2 * row]);
    f32x4 O = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < KS; x++) {
      const float f = __builtin_amdgcn_exp2f(ml[(w0 + x) * 128 + 2 * row] - M);     // 0 for a wave without keys
      L = __builtin_fmaf(f, ml[(w0 + x) * 128 + 2 * row + 1], L);
      const f32x4 v = parked(smem, w0 + x, row, ch);
#pragma unroll
      for (int e = 0; e < 4; e++) O[e] = __builtin_fmaf(f, v[e], O[e]);
    }
    const float inv = 1.f / L;
    if (row < w.qcnt) S::store4out(ob + (int64_t)w.query(g, row) * p.ost + 4 * ch, O * inv);
  }
}

// Mean length of a side of the squares' key rectangles.
inline double mean_reach(int grid, int side, int block) {
  double sum = 0;
  int n = 0;
  for (int i = 0; i * side < grid; i++, n++) sum += std::min((i + 1) * side + block, grid) - std::max(i * side - block, 0);
  return sum / n;
}

// What a launch with `ks` waves per tile costs, in steps of one wave: the mean walk of a wave and what its start
// and end cost (3 to 4.2 steps), times the workgroups that share a CU: the first takes 1.07 us a step (it has nobody
// to hide its latencies behind), every further one adds 0.65.
struct WindowCost {
  double tiles, steps;     // tiles that exist, mean 32-key steps of a tile
  bool fp32;               // steps of 32 queries on parts: longer ones, so that a start is 1.1 to 2 of them
  double of(int ks) const {
    const double per_cu = tiles * ks / 4.0 / device_cu_count();
    return 0.65 * (std::max(per_cu, 1.0) + 0.65) * (std::max(steps / ks, 1.0) + (fp32 ? (ks == 4 ? 1.95 : (ks == 2 ? 1.2 : 1.1)) : (ks == 4 ? 4.2 : (ks == 2 ? 3.7 : 3.0))));
  }
  // Waves per tile.  One wave per tile does the least work (no merge, one start), four fill the chip when there
  // are few tiles and shorten the walk when it is long.  (Measured with each forced over 88 grids of 14 to
  // 248 a side, 8 to 32 heads: the choice takes 0.7 % more than the best on average, 15 % more at worst - 20x33, 8x8 blocks, 16 heads,
  // two waves 15.1 us, four 13.1 -, 12 % with 24x24 blocks on 100x60.  Squares of several blocks take longer a step, for their
  // masks, than this says - 245x245, 2x2 blocks: 174 us, not 98 -, but by about the same factor for each split: of eight
  // such grids in bf16 the choice is the best on seven and 3 % off on one.  fp32, 41 grids of 14 to 64 a side: 1.1 % more than the best, 11 % at
  // worst - 23x27, 8x8 blocks, four images, two waves 56.3 us, four 50.6 -; with bf16's starts 6.6 %: 28x28, 7x7 blocks, two images 42.1 -> 34.6,
  // 36x21 47.8 -> 35.8, 44x44, 8x8 blocks 87 -> 74.  The other rows of the fp32 kernel take the same starts, against bf16's, of 14 to 18 grids:
  // pruned ones 2.9 % more than the best against 3.7, bf16 rows 2.0 against 7.5, pruned bf16 rows 4.3 against 3.9; at worst 22 %, with either -
  // 40x40, 16x16 blocks, 60 % left, two waves 61 us, four 51.)
  int split() const { return of(4) <= of(2) && of(4) <= of(1) ? 4 : (of(2) <= of(1) ? 2 : 1); }
};
inline WindowCost window_cost(const ns_attn_desc &d, int qt) {
  const int side = d.block > 4 ? d.block : d.block * (8 / d.block);
  const int nh = d.grid_h / side, nw = d.grid_w / side, eh = d.grid_h % side, ew = d.grid_w % side;
  const double full = d.coords ? (double)(d.tokens - d.n_global) / ((double)d.grid_h * d.grid_w) : 1.0;
  auto runs = [&](int h, int w) { return std::ceil(full * h * w / qt); };
  const double per_image = (double)nh * nw * runs(side, side) + nw * runs(eh, side) + nh * runs(side, ew) + runs(eh, ew);
  return WindowCost{per_image * d.batch * d.heads,
                    (full * mean_reach(d.grid_h, side, d.block) * mean_reach(d.grid_w, side, d.block) + d.n_global) / 32.0 + 0.5, qt == 32};
}

// The geometry on the host; qt = queries per tile, rows_per_group = global rows that one global
// workgroup handles (0: no global rows in this launch).  Workgroups to launch, or -1.
inline long long window_geometry(const AttnArgs &a, int qt, int rows_per_group, int nchunks, WindowGeom &g, int &ks) {
  const ns_attn_desc &d = a.d;
  const bool lists = d.coords != nullptr;
  g.grid_h = d.grid_h; g.grid_w = d.grid_w; g.block = d.block; g.n_global = d.n_global; g.tokens = d.tokens;
  g.heads = d.heads;
  g.side = lists || d.block > 4 ? d.block : d.block * (8 / d.block);
  g.nbh = (d.grid_h + g.side - 1) / g.side;
  g.nbw = (d.grid_w + g.side - 1) / g.side;
  g.cap = d.block * d.block;
  g.tpb = (g.side * g.side + qt - 1) / qt;
  g.lists = a.geom.lists; g.counts = a.geom.counts;
  const long long per_image = (long long)g.nbh * g.nbw * g.tpb, tiles = per_image * d.batch * d.heads;
  const int groups = rows_per_group ? (d.n_global + rows_per_group - 1) / rows_per_group : 0;
  const long long live = (long long)d.batch * d.heads * groups * nchunks;
  if (tiles > 0x7ffffff0LL || live > 0x7ffffff0LL) return -1;
  g.tiles_per_image = (int)per_image;
  g.tiles = (int)tiles;
  ks = a.split ? a.split : window_cost(d, qt).split();
  g.per_xcd = (int)((tiles * ks + 31) / 32);
  g.global_groups = groups;
  g.nchunks = nchunks;
  // The chunks of the global rows come last, where they fill what the last round of tiles leaves idle (against first,
  // whole calls: 100x100, 8x8 blocks, two images, five global tokens 104.0 -> 100.6 us, fp32 64x64 110.7 -> 104.0).  Where all
  // workgroups fit the chip at once there is no such round and a chunk takes longest: first (28x28, 7x7 blocks,
  // 13.4 us, last 14.5).
  const long long tile_wgs = 8LL * g.per_xcd, wgs = tile_wgs + (live + 7) / 8 * 8;
  const bool first = wgs <= 2LL * device_cu_count();
  g.row_wgs = (int)live;
  g.rows_at = first ? 0 : (int)tile_wgs;
  g.tiles_at = first ? (int)(wgs - tile_wgs) : 0;
  return wgs > 0x7fffffffLL ? -1 : wgs;
}

// The launch arguments; logits, partials: of the global rows, NULL partials = patch queries only
template <class S, int NT>
inline long long window_params(const AttnArgs &a, float *logits, float *partials, WindowParams &p, int &ks) {
  const ns_attn_desc &d = a.d;
  p.r = global_rows<S>(d, a.q, a.k, a.v, logits, partials);
  p.out = a.out;
  p.osb = d.out_stride_b; p.osh = d.out_stride_h; p.ost = d.out_stride_t;
  return window_geometry(a, 32 * NT, partials ? global_group_rows<S>() : 0, cls_num_chunks(d.tokens), p.g, ks);
}

}  // namespace ns
