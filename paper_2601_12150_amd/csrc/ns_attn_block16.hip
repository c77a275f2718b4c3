// bf16 MFMA neighbourhood attention for blocks whose side is a multiple of 16: the queries of a block
// share every key tile (gfx950).
//
// All queries of a block have the same keys, the rectangle that the (clipped) 3x3 blocks around it cover.  So queries are
// numbered in raster order within their block, keys in raster order within the rectangle, and short blocks at the right
// and bottom edge leave no holes on either side: a workgroup of 4 waves owns 256 consecutive queries of a block, wave w
// 64 of them, and walks the keys in tiles of 64.  The key tiles pass through a 4-slot LDS ring (direct global -> LDS
// transfers, a quarter of each issued by every wave, XOR-swizzled) and every wave uses every one of them: one fetch from
// L2 instead of four.  One s_barrier per key tile makes the tile after next visible to all and frees the slot that the
// next transfer overwrites.
//
// A tile is two pipelined steps of 32 keys (StepBf16::half_step in ns_window.h): while the weights of one half of the
// queries are taken and multiplied with V, the logits of the other half are formed, across the barrier too, so tiles t
// and t + 1 have landed when t is worked on.  The exponent reference is the global tokens' largest logit and is not raised
// tile by tile, which makes the weights element-wise; a query tile whose sums leave the safe range is redone with a
// running maximum.  Bound: the power that the matrix instructions, the exponentials and the fragment reads take
// together - the clock falls from 2.4 to 1.7 GHz under this loop, so that what counts is the work in a tile, not how
// well it overlaps.  Measured against squares of 16x16 filled up with copies, tiles whose sums and products the compiler
// scheduled (whole calls, 16 heads): 245x245 with 64x64 blocks 6995 -> 5647 us, of which 15 % are the copies, 256x256
// with 16x16 blocks 627 -> 606.
#include "ns_window.h"

namespace ns {

namespace {

struct BlockParams {
  GlobalRows r;         // q, k, v, strides, scale; logits and partials for the global rows
  uint16_t *out;
  int64_t osb, osh, ost;
  float c;              // scale * log2(e)
  int grid_h, grid_w, block, nbh, nbw;   // blocks per side: ceil(grid / block)
  int heads;
  int parts;            // workgroups per block: ceil(block^2 / 256)
  int inner, rim;       // blocks of an image with all eight neighbours, other blocks
  int images;           // batch * heads
  int inner_xcd, rim_xcd;   // workgroups of either kind per XCD
  int n_global;         // G leading global tokens, 1 .. 8 (their K and V rows sit in LDS)
  int tokens, nchunks;
  int row_wgs, row_xcd; // workgroups that own a chunk of a head's global rows; per XCD
};

typedef bf16x8 __attribute__((address_space(3))) *lds_bf16x8_ptr;

constexpr uint32_t kSlot = 16384;     // one key tile: K [64][64] bf16, then V [64][64] bf16
constexpr uint32_t kVOff = 8192;
constexpr int kSlots = 4;
constexpr uint32_t kK0Row = kSlots * kSlot;        // k_0 in the first 128 bytes of a 1 KB transfer
constexpr uint32_t kV0Row = kSlots * kSlot + 1024; // v_0 likewise
constexpr int kBlockLds = kSlots * kSlot + 2048;

#define NS_U(x) __builtin_amdgcn_readfirstlane(x)

constexpr float kMasked = -INFINITY;  // logit of a key number past the end: below any other, times any scale

// grid: 8 XCDs x (row_xcd + inner_xcd + rim_xcd) workgroups of 256 threads, each 256 queries of a block or a chunk of the
// global rows.  ROWS: 0: no global rows, 1: one, 2: several.
template <int ROWS>
__global__ __launch_bounds__(256, 2) void attn_block16_kernel(BlockParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, wave = NS_U(tid >> 6), lane = tid & 63;
  const int l32 = lane & 31, hh = lane >> 5;

  // Workgroups are dealt round-robin to the 8 XCDs.  Each XCD takes a contiguous range of the inner blocks (neighbours
  // share most of their key tiles) and after them one of the rim's, which have fewer keys and fill the chip's last round
  // (245x245, 64x64 blocks: an inner block's workgroup takes a sixth of the launch).
  int img, R, C, part;
  {
    int i = (int)blockIdx.x >> 3;
    // The chunks of the global rows, a few microseconds each, come last: they fill what the last round of tiles leaves
    // idle (against a launch of their own, 16 heads: 256x256, 16x16 blocks 612 -> 598 us a call, 96x96 102 -> 94, 128x128
    // with 64x64 blocks and five global tokens 1030 -> 1007).  (Spread among the tiles, so that their loads run beside products, they put launches of whole rounds of tiles
    // into another round: 128x128, 64x64 blocks, five global tokens, 1056 -> 1192 us.)
    if (ROWS && i >= p.inner_xcd + p.rim_xcd) {
      const int id = ((int)blockIdx.x & 7) * p.row_xcd + i - p.inner_xcd - p.rim_xcd;
      if (id >= p.row_wgs) return;
      if (ROWS == 1) global_row_chunk(p.r, p.heads, p.tokens, p.nchunks, id, smem, tid);
      else if (p.r.logits) global_rows_chunk<StepBf16, true, true>(p.r, p.heads, p.n_global, p.tokens, 1, p.nchunks, id, smem, wave, lane);
      else global_rows_chunk<StepBf16, true, false>(p.r, p.heads, p.n_global, p.tokens, 1, p.nchunks, id, smem, wave, lane);
      return;
    }
    const bool rim = i >= p.inner_xcd;
    i = rim ? ((int)blockIdx.x & 7) * p.rim_xcd + i - p.inner_xcd : ((int)blockIdx.x & 7) * p.inner_xcd + i;
    const int per = (rim ? p.rim : p.inner) * p.parts;
    if (i >= per * p.images) return;
    img = NS_U(i / per);
    i -= img * per;
    int blk = NS_U(i / p.parts);
    part = i - blk * p.parts;
    if (!rim) {
      R = blk / (p.nbw - 2);
      C = 1 + blk - R * (p.nbw - 2);
      R += 1;
    } else {
      // the top row, the ends of the middle rows, the bottom row
      const int ends = min(p.nbw, 2), mid = max(p.nbh - 2, 0) * ends;
      const int b2 = blk - p.nbw, b3 = b2 - mid;
      R = b2 < 0 ? 0 : (b3 < 0 ? 1 + b2 / ends : p.nbh - 1);
      C = b2 < 0 ? blk : (b3 < 0 ? (b2 % ends ? p.nbw - 1 : 0) : b3);
    }
    R = NS_U(R);
    C = NS_U(C);
  }
  const int b = NS_U(img / p.heads), h = img - b * p.heads;
  // the block's queries
  const int r0 = R * p.block, c0 = C * p.block;
  const int bw = min(p.block, p.grid_w - c0), qn = min(p.block, p.grid_h - r0) * bw;
  if (part * 256 >= qn) return;
  // the rectangle of its keys
  const int kr0 = max(r0 - p.block, 0), kc0 = max(c0 - p.block, 0);
  const int kw = min(c0 + 2 * p.block, p.grid_w) - kc0, nk = (min(r0 + 2 * p.block, p.grid_h) - kr0) * kw;
  const int steps = (nk + 63) >> 6;
  const int q0 = part * 256 + wave * 64, qcnt = NS_U(min(qn - q0, 64));     // this wave's queries, if any

  const int64_t head = b * p.r.sb + h * p.r.sh;
  const char *qb = reinterpret_cast<const char *>(static_cast<const uint16_t *>(p.r.q) + head);
  const char *kb = reinterpret_cast<const char *>(static_cast<const uint16_t *>(p.r.k) + head);
  const char *vb = reinterpret_cast<const char *>(static_cast<const uint16_t *>(p.r.v) + head);
  char *ob = reinterpret_cast<char *>(p.out + b * p.osb + h * p.osh);

  const uint32_t lds_base = (uint32_t)(size_t)((__attribute__((address_space(3))) unsigned char *)smem);

  const uint32_t rowB = (uint32_t)p.r.st * 2u;
  // token of a query slot (slots past the end repeat the last one) and of a key number (likewise)
  auto query = [&](int i) {
    const int s = q0 + min(i, qcnt - 1), r = div_small(s, 1.f / (float)bw);
    return p.n_global + (r0 + r) * p.grid_w + c0 + s - r * bw;
  };
  auto key = [&](int j) {
    j = min(j, nk - 1);
    const int r = div_small(j, 1.f / (float)kw);
    return p.n_global + (kr0 + r) * p.grid_w + kc0 + j - r * kw;
  };
  StepBf16 st;
  st.init(lane);

  // ---- transfers.  This wave moves rows 16*wave .. +15 of a tile, two requests of 8 rows each for K and for V; a lane
  // follows the places of its two rows: 64 keys on are `down` rows of the rectangle and `right` columns.
  const int right = 64 % kw;
  const uint32_t step_off = (uint32_t)((64 / kw) * p.grid_w + right) * rowB, wrap_off = (uint32_t)(p.grid_w - kw) * rowB;
  int col[2];
  uint32_t at[2];
#pragma unroll
  for (int j = 0; j < 2; j++) {
    const int i = 16 * wave + 8 * j + (lane >> 3), r = div_small(i, 1.f / (float)kw);
    col[j] = i - r * kw;
    at[j] = (uint32_t)(p.n_global + (kr0 + r) * p.grid_w + kc0 + col[j]) * rowB;
  }
  int issued = 0;
  auto issue_next = [&]() {
    if (issued == steps - 1 && (nk & 63))        // the last tile of a ragged rectangle repeats its last key
#pragma unroll
      for (int j = 0; j < 2; j++) at[j] = (uint32_t)key(64 * issued + 16 * wave + 8 * j + (lane >> 3)) * rowB;
    const uint32_t dst = lds_base + (uint32_t)(issued & (kSlots - 1)) * kSlot + (uint32_t)wave * 2048u;
#pragma unroll
    for (int j = 0; j < 2; j++) dma16(kb, at[j] + st.kch[j], dst + j * 1024);
#pragma unroll
    for (int j = 0; j < 2; j++) dma16(vb, at[j] + st.vch, dst + kVOff + j * 1024);
    issued++;
#pragma unroll
    for (int j = 0; j < 2; j++) {
      col[j] += right;
      at[j] += step_off;
      const bool wrap = col[j] >= kw;
      col[j] -= wrap ? kw : 0;
      at[j] += wrap ? wrap_off : 0u;
    }
  };

  // ---- register state of this wave's query tile
  StepBf16::Q qf[2];
  f32x16 o[2][2];       // [query half][channels 32 dt ..]
  float m[2], l[2];
  auto load_tile = [&]() {
    st.load_q(qf[0], qb, rowB, query(l32), lane, 0.f);
    st.load_q(qf[1], qb, rowB, query(32 + l32), lane, 0.f);
    // (arrived: a load that the compiler takes to be pending at the key loop's head would put a wait for every transfer
    // in flight into each iteration)
#pragma unroll
    for (int s = 0; s < 4; s++) asm volatile("" : "+v"(qf[0].f[s]), "+v"(qf[1].f[s]));
  };
  // The state the global token gives a query tile: m = its logit (the fixed exponent reference),
  // l = 1, O = v_0; k_0 and v_0 sit in LDS.  The k_0 fragment is that of a key tile whose rows
  // are all k_0, so every register of its product with Q is q . k_0.  Further global tokens
  // (rows 1 .. G-1 of the same LDS areas) are added one by one with a running maximum, so the
  // reference becomes the largest of the global tokens' logits.
  auto init_tile = [&]() {
    for (int g = 0; g < p.n_global; g++) {
      StepBf16::K kg;
#pragma unroll
      for (int s = 0; s < 4; s++) kg.f[s] = *(lds_bf16x8_ptr)(smem + kK0Row + 128 * g + 64 * hh + 16 * s);
      float pg[2];
#pragma unroll
      for (int nt = 0; nt < 2; nt++) {
        const f32x16 s = st.product(kg, qf[nt]);
        const float sg = s[0] * p.c;
        if (g == 0) {
          m[nt] = sg;
          l[nt] = hh == 0 ? 1.f : 0.f;
          continue;
        }
        const float m_new = fmaxf(m[nt], sg), alpha = __builtin_amdgcn_exp2f(m[nt] - m_new);
        pg[nt] = __builtin_amdgcn_exp2f(sg - m_new);
        m[nt] = m_new;
        l[nt] = __builtin_fmaf(l[nt], alpha, hh == 0 ? pg[nt] : 0.f);
#pragma unroll
        for (int e = 0; e < 16; e++) { o[nt][0][e] *= alpha; o[nt][1][e] *= alpha; }
      }
#pragma unroll
      for (int dt = 0; dt < 2; dt++)
#pragma unroll
        for (int ig = 0; ig < 4; ig++) {
          const u32x2 v2 = *(u32x2 __attribute__((address_space(3))) *)(smem + kV0Row + 128 * g + 64 * dt + 16 * ig + 8 * hh);
          const bf16x4 v4 = __builtin_bit_cast(bf16x4, v2);
#pragma unroll
          for (int e = 0; e < 4; e++)
#pragma unroll
            for (int nt = 0; nt < 2; nt++)
              o[nt][dt][4 * ig + e] = g == 0 ? (float)v4[e] : __builtin_fmaf(pg[nt], (float)v4[e], o[nt][dt][4 * ig + e]);
        }
    }
  };
  // normalise and store; returns whether a weight overflowed the fixed reference (then some sum or
  // output is not finite).  Lane (query, hh) stores channels 32*dt + 16*ig + 8*hh + 0..7.
  auto finish_tile = [&]() {
    float big = max_abs(max_abs(0.f, l[0]), l[1]);
#pragma unroll
    for (int i = 0; i < 16; i++)
      big = max_abs(max_abs(max_abs(max_abs(big, o[0][0][i]), o[0][1][i]), o[1][0][i]), o[1][1][i]);
    const bool bad = __any(!(big < 1e30f));
#pragma unroll
    for (int nt = 0; nt < 2; nt++) {
      const float inv = 1.f / half_swap_sum(l[nt]);
      char *row = ob + (size_t)query(32 * nt + l32) * (size_t)(p.ost * 2) + 16 * hh;
#pragma unroll
      for (int dt = 0; dt < 2; dt++)
#pragma unroll
        for (int ig = 0; ig < 2; ig++) {
          const u32x4 u = row_pieces(o[nt][dt], 8 * ig, inv);
          if (32 * nt + l32 < qcnt) *reinterpret_cast<u32x4 *>(row + 64 * dt + 32 * ig) = u;
        }
    }
    return bad;
  };
  // register e of a product is key 8*(e/4) + 4*hh + e%4 of the 32 from number j on
  auto mask_keys = [&](f32x16 &s, int j) {
#pragma unroll
    for (int e = 0; e < 16; e++) s[e] = j + 8 * (e >> 2) + 4 * hh + (e & 3) < nk ? s[e] : kMasked;
  };

  // ---- prologue: the first four key tiles are requested, the first two have landed
  if (wave == 0) {
    // the global tokens' rows, 8 lanes x 16 bytes each: LDS row r = token min(r, G-1)
    const uint32_t goff = (uint32_t)min(lane >> 3, p.n_global - 1) * rowB + 16u * (lane & 7);
    dma16(kb, goff, lds_base + kK0Row);
    dma16(vb, goff, lds_base + kV0Row);
  }
#pragma unroll
  for (int i = 0; i < kSlots; i++)
    if (i < steps) issue_next();
  if (steps >= kSlots) wait_vm<8>();           // k_0, v_0, tiles 0 and 1
  else wait_vm<0>();
  __syncthreads();
  const bool live = qcnt > 0;                  // (a wave without queries only moves its share of the tiles)
  const unsigned char *slot = smem;
  f32x4 ls[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  f32x16 s0, s1;                               // logits of queries 0..31 and 32..63
  StepBf16::K kf;
  StepBf16::V vf;
  bf16x8 open = {};                            // the output product behind: none yet
  vf.f[1][0] = vf.f[1][1] = open;
  if (live) {
    load_tile();                               // consumed at once: no load is pending at the loop head
    init_tile();
    st.load_k(kf, slot);
    s0 = st.product(kf, qf[0]);
    if (steps == 1) mask_keys(s0, 0);
  }
  for (int t = 0; t < steps; t++) {
    const unsigned char *next = smem + ((t + 1) & (kSlots - 1)) * kSlot;
    if (live) {
      const bool last = 64 * (t + 1) > nk, last_next = 64 * (t + 2) > nk;
      st.load_v(vf, slot + kVOff, 0);
      st.template half_step<true>(s0, p.c, -m[0], ls[0], o[0], ls[1], o[1], open, vf, slot + kVOff, kf, qf[1], s1);
      if (last) mask_keys(s1, 64 * t);
      st.load_k(kf, slot + 4096);
      st.template half_step<false>(s1, p.c, -m[1], ls[1], o[1], ls[0], o[0], open, vf, slot + kVOff, kf, qf[0], s0);
      if (last) mask_keys(s0, 64 * t + 32);
      st.load_v(vf, slot + kVOff + 4096, 0);
      st.template half_step<true>(s0, p.c, -m[0], ls[0], o[0], ls[1], o[1], open, vf, slot + kVOff + 4096, kf, qf[1], s1);
      if (last) mask_keys(s1, 64 * t + 32);
      st.load_k(kf, next);                     // (behind the last tile: what the slot holds, not used)
      st.template half_step<false>(s1, p.c, -m[1], ls[1], o[1], ls[0], o[0], open, vf, slot + kVOff + 4096, kf, qf[0], s0);
      if (last_next) mask_keys(s0, 64 * (t + 1));
    }
    // tile t+2: this wave's share has landed (its share of tile t+3 may still be in flight)
    if (t + 3 < steps) wait_vm<4>();
    else wait_vm<0>();
    __syncthreads();   // ... and everybody's; and everybody is done with tile t, whose slot tile t+4 takes
    if (issued < steps) issue_next();
    slot = next;
  }
  bool bad = false;
  if (live) {
#pragma unroll
    for (int dt = 0; dt < 2; dt++) o[1][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf.f[1][dt], open, o[1][dt], 0, 0, 0);
    st.add_weights(ls[1], open);
#pragma unroll
    for (int nt = 0; nt < 2; nt++) l[nt] += StepBf16::row_sum(ls[nt], lane);
    bad = finish_tile();
  }
  // (the ring is free behind the last barrier: each wave takes a slot of it below)
  if (!bad) return;

  // ---- a weight overflowed in this wave's query tile (its stored rows are not finite): once
  // more with a running maximum, fragments straight from global memory, V staged through LDS
  const uint32_t mine = (uint32_t)wave * kSlot;
  load_tile();
  init_tile();
  for (int t = 0; t < steps; t++) {
    StepBf16::K kt[2];
#pragma unroll
    for (int mt = 0; mt < 2; mt++) st.load_q(kt[mt], kb, rowB, key(64 * t + 32 * mt + l32), lane, 0.f);
#pragma unroll
    for (int it = 0; it < 8; it++)
      dma16(vb, (uint32_t)key(64 * t + 8 * it + (lane >> 3)) * rowB + st.vch, lds_base + mine + it * 1024);
    wait_vm<0>();               // also the K fragments above
#pragma unroll
    for (int nt = 0; nt < 2; nt++) {
      f32x16 s[2] = {st.product(kt[0], qf[nt]), st.product(kt[1], qf[nt])};
      if (64 * (t + 1) > nk) {
        mask_keys(s[0], 64 * t);
        mask_keys(s[1], 64 * t + 32);
      }
      float mx = fmaxf(s[0][0], s[1][0]);
#pragma unroll
      for (int e = 1; e < 16; e++) mx = fmaxf(fmaxf(mx, s[0][e]), s[1][e]);
      const float m_new = fmaxf(m[nt], half_swap_max(mx) * p.c);
      const float alpha = __builtin_amdgcn_exp2f(m[nt] - m_new);
      m[nt] = m_new;
      l[nt] *= alpha;
#pragma unroll
      for (int e = 0; e < 16; e++) { o[nt][0][e] *= alpha; o[nt][1][e] *= alpha; }
#pragma unroll
      for (int mt = 0; mt < 2; mt++) {
        bf16x8 w[2];
#pragma unroll
        for (int e = 0; e < 16; e += 2) {
          const uint32_t u = pack_bf16(__builtin_amdgcn_exp2f(__builtin_fmaf(s[mt][e], p.c, -m_new)),
                                       __builtin_amdgcn_exp2f(__builtin_fmaf(s[mt][e + 1], p.c, -m_new)));
          l[nt] += bf16_lo(u) + bf16_hi(u);
          const bf16x2 pk = __builtin_bit_cast(bf16x2, u);
          w[e >> 3][e & 7] = pk[0];
          w[e >> 3][(e & 7) + 1] = pk[1];
        }
#pragma unroll
        for (int sp = 0; sp < 2; sp++) {
          StepBf16::V v;
          st.load_v(v, smem + mine + 4096 * mt, sp);
#pragma unroll
          for (int dt = 0; dt < 2; dt++) o[nt][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v.f[sp][dt], w[sp], o[nt][dt], 0, 0, 0);
        }
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // V reads done before the next transfer into the slot
  }
  finish_tile();
}

}  // namespace

bool block16_attn_supported(const ns_attn_desc &d) {
  return d.dtype == NS_BF16 && d.head_dim == 64 && d.radius == 1 && d.n_global >= 1 && d.n_global <= 8 &&
         d.coords == nullptr && d.block >= 16 && d.block % 16 == 0 && d.scale > 0.f &&
         // tokens are addressed with 32-bit byte offsets from the (batch, head) base
         (long long)d.tokens * d.q_stride_t * 2 < 0x7fffffffLL &&
         (long long)d.tokens * d.out_stride_t * 2 < 0x7fffffffLL;
}

ns_status launch_attn_block16(const AttnArgs &a, float *logits, float *partials) {
  const ns_attn_desc &d = a.d;
  BlockParams p;
  p.r = global_rows<StepBf16>(d, a.q, a.k, a.v, logits, partials);
  p.out = static_cast<uint16_t *>(a.out);
  p.osb = d.out_stride_b; p.osh = d.out_stride_h; p.ost = d.out_stride_t;
  p.c = d.scale * kLog2e;
  p.grid_h = d.grid_h;
  p.grid_w = d.grid_w;
  p.block = d.block;
  p.nbh = (d.grid_h + d.block - 1) / d.block;
  p.nbw = (d.grid_w + d.block - 1) / d.block;
  p.parts = (d.block * d.block + 255) / 256;
  p.inner = std::max(p.nbh - 2, 0) * std::max(p.nbw - 2, 0);
  p.rim = p.nbh * p.nbw - p.inner;
  p.heads = d.heads;
  p.images = d.batch * d.heads;
  p.n_global = d.n_global;
  p.tokens = d.tokens;
  p.nchunks = cls_num_chunks(d.tokens);
  static_assert(8 <= global_group_rows<StepBf16>(), "the global rows of a head are one group");
  const long long inner = ((long long)p.images * p.inner * p.parts + 7) / 8, rim = ((long long)p.images * p.rim * p.parts + 7) / 8;
  const long long rows = partials ? (long long)p.images * p.nchunks : 0, wgs = 8 * (inner + rim + (rows + 7) / 8);
  if (wgs > 0x7fffffffLL) return fail(NS_ERR_UNSUPPORTED, "launch grid too large");
  p.inner_xcd = (int)inner;
  p.rim_xcd = (int)rim;
  p.row_wgs = (int)rows;
  p.row_xcd = (int)((rows + 7) / 8);
  typedef void (*kern_t)(BlockParams);
  const kern_t kern = !partials ? attn_block16_kernel<0> : (d.n_global == 1 ? attn_block16_kernel<1> : attn_block16_kernel<2>);
  const int lds = partials && d.n_global > 1 ? kWindowLds : kBlockLds;
  static_assert(kBlockLds <= kWindowLds && kScanLds <= kBlockLds, "LDS");
  const ns_status rs = reserve_lds_once(reinterpret_cast<const void *>(kern), lds);
  if (rs != NS_OK) return rs;
  hipLaunchKernelGGL(kern, dim3((unsigned)wgs), dim3(256), lds, a.stream, p);
  return check_launch("attn_block16_kernel");
}

}  // namespace ns
