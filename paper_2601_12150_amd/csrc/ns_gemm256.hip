// bf16 MFMA GEMM with a 256 x 256 workgroup tile for the linear maps of the transformer block
// (QKV, attention projection, MLP): C[m][n] = sum_k A[m][k] W[n][k] + bias[n], optional exact
// GELU, optional residual R[m][n].  A, W, R, C bf16 row-major, bias fp32, fp32 accumulation.
// Bound: bf16 MFMA, 2*M*N*K FLOP.
//
// Why this shape.  A wave that owns a 64x64 piece of the output reads 1 KB of fragments from LDS
// per 32 matrix-pipe cycles, which is exactly the LDS bandwidth of a CU at full MFMA rate; with
// a 128 x 128 piece per wave (8 x 8 MFMA tiles, 256 accumulator registers) it is half of that.
// v_mfma_f32_16x16x32_bf16 and not 32x32x16: the chip is limited by power under either (the clock falls from 2.4 to
// 1.7 GHz), and the smaller one takes less of it: products of random values from registers alone sustain 2.07 against 1.80 PFLOP/s,
// 1.94 where both operands change with every instruction.  Whole launches, 32x32x16 -> 16x16x32, us: 16385 x 3072 x 1024 91.0 ->
// 83.7, 16385 x 1024 x 4096 + residual 109.4 -> 100.3, 9832 x 4096 x 1024 + GELU 90.9 -> 84.5.
// So: 4 waves per workgroup, one per SIMD, each with up to 512 registers; 256 (n) x 256 (m) per
// workgroup; k in slices of 64 by direct global -> LDS transfers (rows of 128 bytes: a transfer then uses whole
// cache lines, which moves the same bytes in 3/4 of the time that 64-byte rows take).
//
// How far ahead.  With two slots per operand, requested as soon as the slice before is read, 64 KB
// per CU are on their way; under load a transfer takes longer than the slice it has (1.69 us a slice with every
// CU busy, where the MFMAs alone take 1.18 and the transfers alone 0.88).  The weights get a third slot
// (all 160 KB of LDS are then in use), and the token fragments of a whole slice are held in registers: they are read in
// the last k-step before and the first k-step of their slice, which frees their slot after a quarter of it.  So 112 KB are on
// their way: weights have two slices of time, tokens one and a half.  LDS reads and the issue of the
// transfers are placed between the MFMAs one by one.  The product is formed transposed (W rows as
// the A operand) as in the smaller kernel; the epilogue transposes each 32-token slab through
// LDS so that bias / GELU / residual / store work on 16-byte pieces of full output rows.
//
// Rows.  With M = 256 q + rem and 0 < rem <= 32 (a full-grid sequence: rem is the number of
// global tokens in the batch) the last row tile takes the extra rows as a ninth 32-row slab
// instead of opening a nearly empty tile row, which would cost a whole extra round on a launch
// that otherwise fills the chip exactly once; the slab's 32 MFMA tiles are shared out eight per
// wave.  Any other remainder gets a tile of its own whose waves only compute the slabs that
// hold rows.  Where M / 256 row tiles leave many CUs without work in the last round (a pruned
// sequence: 39 x 4 tiles on 256 CUs), tiles of 192 rows (three slabs per wave) are used instead
// when that shortens the launch.
//
// Measured (us, two slots per operand, 32x32x16 products and an epilogue that waits for each of its loads -> this): 16385 x 3072 x 1024
// 111 -> 84, 16385 x 1024 x 1024 + residual 49 -> 32, 16385 x 4096 x 1024 + GELU 177 -> 131, 16385 x 1024 x 4096 + residual 128 -> 100;
// 9832 rows: 70 -> 55, 31 -> 21, 113 -> 84, 89 -> 63.
#include "ns_gemm.h"
#include <type_traits>

namespace ns {

namespace {

struct Gemm256Params : GemmIo {
  int ntn, ntm;      // tiles along n and m
  int extended;      // the last row tile has 288 rows
  int n256;          // the first n256 rows of tiles have 256 token rows, the others 192 (three slabs per wave):
                     // the mix that fills the chip's rounds of workgroups best
  int batch;         // products of the same w, bias and r: a and c of the next one follow at these distances
  long long a_stride, c_stride;   // in elements
  PixelRows pix;
};

constexpr int kStageW = 256 * 128;           // bytes: 256 weight rows x 64 k
constexpr int kStageX = 256 * 128;           // 256 token rows x 64 k
constexpr int kGemmLds = 2 * kStageX + 3 * kStageW;
constexpr int kEpiWave = Epi<4>::kBytes;

// One wave's work on one workgroup tile.  NTJ: 32-row token slabs of its own 128 rows that this
// wave computes (0..4).  EXT: the tile has a ninth token slab (rows 256..287); this wave then
// also computes that slab against weight slabs 2*WM and 2*WM+1 of its n half, and every wave
// issues 9 instead of 8 token-row requests per k-slice.  NK: slices of k where there
// are only one or two, which are all requested at the start, else 0.
template <int NK, int NTJ, bool EXT, int WM, bool GELU, bool RES, bool PIX, int TM = 256>
__device__ __forceinline__ void gemm256_wave(const Gemm256Params &p, unsigned char *smem, int m0, int n0,
                                             int wave, int lane) {
  static_assert(TM == 256 || (TM == 192 && !EXT && NTJ <= 3), "192-row tiles: three slabs per wave, no ninth slab");
  constexpr int NT = NTJ > 0 ? NTJ : 1;
  constexpr int XREQ = EXT ? 9 : TM / 32;    // requests of 8 token rows per wave
  constexpr int WROWS = TM / 2;              // token rows per pair of waves
  constexpr int kSlots = EXT ? 2 : 3;        // LDS slots for weight slices; token slices have two
  constexpr int kX = EXT ? kStageX + 4096 : kStageX, kW = 2 * kX;   // bytes of a token slot; the weight slots lie behind
  static_assert(kW + kSlots * kStageW <= kGemmLds, "slots");
  const int l16 = lane & 15;
  const int wm = wave >> 1, wn = wave & 1;
  const uint32_t lds0 = (uint32_t)(size_t)((__attribute__((address_space(3))) unsigned char *)smem);
  const uint32_t rowB = (uint32_t)p.K * 2u;
  const char *ab = reinterpret_cast<const char *>(p.a);
  const char *wb = reinterpret_cast<const char *>(p.w);

  // ---- transfers.  A request moves 8 rows x 128 bytes: slot `lane` is row lane/8, physical
  // 16-byte chunk lane%8, which holds logical chunk (lane%8) ^ ((row >> 1) & 7), row counted
  // within the stage.  (The LDS has 64 banks and serves 16 lanes of a 16-byte read per clock: two
  // rows of 128 bytes span the banks once, so rows 2j and 2j+1 share a swizzle and the 16 rows
  // that 16 consecutive lanes read land on 16 different bank groups.)  Requests start at
  // multiples of 8 rows, so (row >> 1) & 7 = 4 * (request & 1) + lane/16.
  const int drow = lane >> 3;
  auto dchunk = [&](int req) { return 16u * ((lane & 7) ^ ((4 * (req & 1) + (drow >> 1)) & 7)); };
  const int wreq0 = wave * 8;                                        // weight requests: 8 per wave
  const int xreq0 = wave * XREQ;                                     // token requests
  const uint32_t woff[2] = {(uint32_t)(n0 + wreq0 * 8 + drow) * rowB + dchunk(0),
                            (uint32_t)(n0 + wreq0 * 8 + drow) * rowB + dchunk(1)};
  uint32_t xoff[XREQ];
#pragma unroll
  for (int j = 0; j < XREQ; j++) {
    const int m = min(m0 + (xreq0 + j) * 8 + drow, p.M - 1);         // rows past M repeat the last row
    xoff[j] = PIX ? pixel_chunk(p.pix, m, dchunk(xreq0 + j) >> 4) : (uint32_t)m * rowB + dchunk(xreq0 + j);
  }
  auto issue_w = [&](int kt, int slot, int j) {
    dma16(wb + (size_t)kt * 128 + (size_t)j * 8 * rowB, woff[j & 1], lds0 + kW + slot * kStageW + (wreq0 + j) * 1024);
  };
  auto issue_x = [&](int kt, int j) { dma16(ab + (PIX ? pixel_slice(p.pix, kt) : (size_t)kt * 128), xoff[j], lds0 + (kt & 1) * kX + (xreq0 + j) * 1024); };

  // ---- fragment reads: lane (row l16 of a 16-row tile, quarter lane/16) reads logical chunk 4*h + lane/16 of
  // half h of the slice, i.e. physical chunk (4*h + lane/16) ^ (l16 >> 1) (tiles start at multiples of 16 rows)
  unsigned char *wrd[2], *xrd[2];
#pragma unroll
  for (int h = 0; h < 2; h++) {
    const int ch = 16 * ((4 * h + (lane >> 4)) ^ (l16 >> 1));
    wrd[h] = smem + kW + (wn * 128 + l16) * 128 + ch;
    xrd[h] = smem + (wm * WROWS + l16) * 128 + ch;
  }
  const int eoff = (256 - wm * WROWS) * 128;           // from xrd to the ninth slab
  bf16x8 fw[2][4], fx[2][2 * NT], fe[2][2];
  f32x4 acc[8][2 * NT];   // [16 weights][16 tokens]: register e = n 4*(lane/16) + e, token l16
  f32x4 acce[4][2];       // weights 64*WM + 16*i, ninth slab's tokens 16*j

  // One quarter of a slice: half ks/2 of its k with weights 64*(ks & 1) .. + 63 of the wave's 128, i.e. the MFMAs of fragments
  // (fw[ks & 1], fx[ks >> 1]) with, spread between them, the LDS reads of
  // later fragments and the transfers of a later slice, so that neither the reads' latency nor the issue of the
  // transfers is exposed.  The fences keep this order: the scheduler would sink the reads below the MFMAs
  // that do not need them.  A weight fragment stays for all token fragments: an operand that does not change costs less power.
  //   ks 0: reads W(t, 1), X(t, half 1)           ks 1: reads W(t, 2); transfers X(t+2)
  //   ks 2: reads W(t, 3)                         ks 3: reads W(t+1, 0), X(t+1, half 0); transfers W(t+kSlots)
  constexpr int XF = 2 * (NTJ + (EXT ? 1 : 0));        // token fragments of half a slice
  auto read_w = [&](int ks, int slot, int i) {
    fw[ks & 1][i] = *(lds_bf16x8_ptr)(wrd[ks >> 1] + slot * kStageW + (4 * (ks & 1) + i) * 2048);
  };
  auto read_x = [&](int h, int kt, int tj) {
    if (tj < 2 * NTJ) fx[h][tj] = *(lds_bf16x8_ptr)(xrd[h] + (kt & 1) * kX + tj * 2048);
    else fe[h][tj - 2 * NTJ] = *(lds_bf16x8_ptr)(xrd[h] + (kt & 1) * kX + eoff + (tj - 2 * NTJ) * 2048);
  };
  auto kstep = [&](auto ks_c, auto read_c, auto move_c, int t, int slot, int slot_next) {
    constexpr int ks = decltype(ks_c)::value;
    constexpr bool kRead = decltype(read_c)::value, kMove = decltype(move_c)::value;
    constexpr int reads = !kRead ? 0 : 4 + (ks == 0 || ks == 3 ? XF : 0);
    constexpr int moves = !kMove ? 0 : (ks == 1 ? XREQ : (ks == 3 ? 8 : 0));
    constexpr int mfmas = 8 * NTJ, groups = mfmas > 0 ? mfmas : 1;
    auto read = [&](int i) {
      if (i < 4) read_w((ks + 1) & 3, ks == 3 ? slot_next : slot, i);
      else read_x(ks == 0 ? 1 : 0, ks == 0 ? t : t + 1, i - 4);
    };
    auto move = [&](int j) {
      if (ks == 1) issue_x(t + 2, j);
      else issue_w(t + kSlots, slot, j);
    };
#pragma unroll
    for (int i = 0; i < groups; i++) {
      // (reads early in the step, a transfer to every fourth MFMA)
#pragma unroll
      for (int r = 0; r < reads; r++)
        if ((2 * reads <= groups ? 2 * r : r * groups / reads) == i) read(r);
      // (asm: with the builtin, whose result may lie elsewhere than its accumulator, the compiler rotates the 256 registers through
      // moves in every slice.  It pads no hazard for asm: nothing but these products and reads from LDS, which the compiler
      // waits for, touches an operand inside the loop and in the slices behind it.  A test reads that off the built code.)
      if (mfmas > 0) {
        f32x4 &c = acc[4 * (ks & 1) + i / (2 * NT)][i % (2 * NT)];
        const bf16x8 &w = fw[ks & 1][i / (2 * NT)], &x = fx[ks >> 1][i % (2 * NT)];
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(w), "v"(x));
      }
#pragma unroll
      for (int j = 0; j < moves; j++)
        if (j * groups / moves == i) move(j);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (EXT && (ks & 1) == WM) {
      // The compiler keeps every accumulator of its own MFMAs in the 256 accumulator registers;
      // 8 of 64 + 8 do not fit and would be rotated through moves in every iteration.  These
      // are pinned to ordinary vector registers instead.  (Each is next touched two quarters later,
      // and read by other instructions only after the loop; the wait states cover a fragment or accumulator that a
      // vector instruction has just written.)
      asm volatile("s_nop 1");
#pragma unroll
      for (int i = 0; i < 4; i++)
#pragma unroll
        for (int j = 0; j < 2; j++) {
          f32x4 &c = acce[i][j];
          const bf16x8 &w = fw[ks & 1][i], &x = fe[ks >> 1][j];
          asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(w), "v"(x));
        }
    }
  };
  // every wave's reads so far have arrived, and so has what it has waited for
  auto meet = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
  using K0 = std::integral_constant<int, 0>;
  using K1 = std::integral_constant<int, 1>;
  using K2 = std::integral_constant<int, 2>;
  using K3 = std::integral_constant<int, 3>;
  using Yes = std::true_type;
  using No = std::false_type;

  // ---- main loop over slices of 64.  Requests stand in the queue in the order W(t+kSlots-1), X(t+1),
  // W(t+kSlots), X(t+2), ..; after the first k-step of slice t every wave has its X fragments and X(t+2) takes
  // their place, after the third the W fragments and W(t+kSlots) does.  Before the fourth, slice t+1 must have
  // landed for every wave; X(t+2) and (three slots) W(t+2) may still be on their way.
  const int nk = NK ? NK : p.K / 64;                   // at least 3 if not NK
  constexpr int kBehind = XREQ + (kSlots - 2) * 8;
#pragma unroll
  for (int s = 0; s < (NK ? NK : kSlots); s++) {
#pragma unroll
    for (int j = 0; j < 8; j++) issue_w(s, s, j);
    if (s < 2)
#pragma unroll
      for (int j = 0; j < XREQ; j++) issue_x(s, j);
  }
  // (cleared while the first transfers are on their way: 256 registers)
#pragma unroll
  for (int ti = 0; ti < 8; ti++)
#pragma unroll
    for (int tj = 0; tj < 2 * NT; tj++) {
      acc[ti][tj] = {0.f, 0.f, 0.f, 0.f};
      asm volatile("" : "+a"(acc[ti][tj]));   // (64 separate values: as copies of one zero the compiler moves them about behind the loop)
    }
#pragma unroll
  for (int i = 0; i < 4; i++)
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int e = 0; e < 4; e++) acce[i][j][e] = 0.f;
  // (their products are asm, for which the compiler pads no hazard: a matrix instruction right behind the vector instruction
  // that clears its accumulator reads what the register held before.  So they are cleared here, not next to it.)
  if (EXT)
#pragma unroll
    for (int i = 0; i < 4; i++) asm volatile("s_nop 1" : "+v"(acce[i][0]), "+v"(acce[i][1]));
  wait_vm<NK == 0 ? 8 + kBehind : (NK - 1) * (8 + XREQ)>();
  meet();
#pragma unroll
  for (int ti = 0; ti < 4; ti++) read_w(0, 0, ti);
#pragma unroll
  for (int tj = 0; tj < XF; tj++) read_x(0, 0, tj);
  // one slice; `ahead`: how many of the slices t+1 .. t+kSlots exist
  auto slice = [&](auto ahead_c, int t, int slot, int slot_next) {
    constexpr int ahead = decltype(ahead_c)::value;
    using More = std::integral_constant<bool, (ahead >= 2)>;
    using Next = std::integral_constant<bool, (ahead >= 1)>;
    kstep(K0{}, Yes{}, No{}, t, slot, slot_next);
    if (ahead >= 2) meet();
    kstep(K1{}, Yes{}, More{}, t, slot, slot_next);
    kstep(K2{}, Yes{}, No{}, t, slot, slot_next);
    if (ahead >= 1) {
      wait_vm<(ahead >= 2 ? kBehind : 0)>();
      meet();
    }
    kstep(K3{}, Next{}, std::integral_constant<bool, (ahead >= kSlots)>{}, t, slot, slot_next);
  };
  auto next = [&](int slot) { return slot + 1 == kSlots ? 0 : slot + 1; };
  int t = 0, slot = 0;
  if (NK == 0) {
    for (; t < nk - kSlots; t++) {
      const int slot_next = next(slot);
      slice(std::integral_constant<int, kSlots>{}, t, slot, slot_next);
      slot = slot_next;
    }
    if (kSlots == 3) {
      slice(K2{}, t, slot, next(slot));
      t++;
      slot = next(slot);
    }
  }
  if (NK != 1) {
    slice(K1{}, t, slot, next(slot));
    t++;
    slot = next(slot);
  }
  // (no transfer is on its way any more: what the epilogue starts with may be asked for)
  using E4 = Epi<4>;
  using E2 = Epi<2>;
  const int mw = m0 + wm * WROWS, nw = n0 + wn * 128, ne = nw + 64 * WM;   // ne: columns of the ninth slab
  f32x4 bias[2], biase[2];
  uint4 res[2][E4::PASSES] = {}, rese[E2::PASSES] = {};
  E4::load_bias(p, nw, lane, bias);
  if (EXT) E2::load_bias(p, ne, lane, biase);
  if (RES && NTJ > 0) E4::load_residual(p, mw, nw, lane, res[0]);
  slice(K0{}, t, slot, 0);
  // (the accumulators are final here: left to itself the compiler sinks the last products into the epilogue's slabs,
  // and their operands are spilled on the way; the first of these also waits for the last product)
#pragma unroll
  for (int ti = 0; ti < 8; ti++)
#pragma unroll
    for (int tj = 0; tj < 2 * NTJ; tj++) {
      if (ti == 0 && tj == 0) asm volatile("s_nop 15" : "+a"(acc[0][0]));
      else asm volatile("" : "+a"(acc[ti][tj]));
    }
  if (EXT)
#pragma unroll
    for (int i = 0; i < 4; i++) asm volatile("s_nop 15" : "+v"(acce[i][0]), "+v"(acce[i][1]));   // (their products are asm: no one else pads)
  __syncthreads();             // every wave is done with the stages: they become the epilogue's staging area

  // ---- epilogue, one 32-token slab at a time
  unsigned char *const ebuf[2] = {smem + wave * kEpiWave, smem + (4 + wave) * kEpiWave};
  static_assert(8 * kEpiWave <= kGemmLds, "two staged slabs per wave");
  auto stage = [&](int tj) {
#pragma unroll
    for (int j = 0; j < 2; j++) {
      if (tj < NTJ) {
        const f32x4 *tile[8];
#pragma unroll
        for (int i = 0; i < 8; i++) tile[i] = &acc[i][2 * tj + j];
        E4::stage(ebuf[tj & 1], tile, j, lane);
      } else if (EXT) {
        const f32x4 *tile[4];
#pragma unroll
        for (int i = 0; i < 4; i++) tile[i] = &acce[i][j];
        E2::stage(ebuf[tj & 1], tile, j, lane);
      }
    }
  };
  stage(0);
#pragma unroll
  for (int tj = 0; tj < NTJ; tj++)
    E4::template emit<GELU, RES>(p, ebuf[tj & 1], bias, res[tj & 1], mw + tj * 32, nw, lane, [&]() {
      if (RES && tj + 1 < NTJ) E4::load_residual(p, mw + (tj + 1) * 32, nw, lane, res[(tj + 1) & 1]);
      if (RES && EXT && tj + 1 == NTJ) E2::load_residual(p, m0 + 256, ne, lane, rese);
      stage(tj + 1);
    });
  if (EXT) E2::template emit<GELU, RES>(p, ebuf[NTJ & 1], biase, rese, m0 + 256, ne, lane, []() {});
}

// PIX: the token rows are patches, read from their pixels
template <int NK, bool GELU, bool RES, bool PIX = false>
__global__ __launch_bounds__(256) void gemm256_bf16_kernel(Gemm256Params p) {
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  // workgroups are dealt round-robin to the 8 XCDs; give each XCD a contiguous run of tiles (n
  // fastest) so that the tiles sharing token rows and the weight matrix meet in one L2
  const int total = p.ntn * p.ntm * p.batch;
  int bid = blockIdx.x;
  if (PIX && bid >= total) {
    cls_rows(p.pix, bid - total, p.N, tid);
    return;
  }
  const bool uniform = p.n256 == 0 || p.n256 == p.ntm;     // (a mix of tile heights keeps the launch order: tall tiles first)
  if (uniform && total % 8 == 0) bid = (bid & 7) * (total / 8) + (bid >> 3);
  int bm = bid / p.ntn;
  const int bn = bid - bm * p.ntn;
  if (p.batch > 1) {         // (the tall tiles of all products first)
    const int tall = p.batch * p.n256, per = bm < tall ? p.n256 : p.ntm - p.n256, x = bm < tall ? bm : bm - tall;
    const int z = __builtin_amdgcn_readfirstlane(x / per);
    p.a += z * p.a_stride;
    p.c += z * p.c_stride;
    bm = (bm < tall ? 0 : p.n256) + x - z * per;
  }
  const int tm = bm < p.n256 ? 256 : 192;
  const int m0 = bm < p.n256 ? bm * 256 : p.n256 * 256 + (bm - p.n256) * 192, n0 = bn * 256;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

  const bool ext = p.extended && bm == p.ntm - 1;
  const int wm = wave >> 1;
  const int wrows = tm >> 1;
  const int rows = min(p.M - (m0 + wm * wrows), wrows);   // may be <= 0
  const int ntj = __builtin_amdgcn_readfirstlane(rows <= 0 ? 0 : (rows + 31) / 32);
  if (ext) {   // the extended tile is full: 256 + (1..32) rows
    if (wm) gemm256_wave<NK, 4, true, 1, GELU, RES, PIX>(p, smem, m0, n0, wave, lane);
    else gemm256_wave<NK, 4, true, 0, GELU, RES, PIX>(p, smem, m0, n0, wave, lane);
    return;
  }
  if (tm == 192) {
    switch (ntj) {
      case 3: gemm256_wave<NK, 3, false, 0, GELU, RES, PIX, 192>(p, smem, m0, n0, wave, lane); break;
      case 2: gemm256_wave<NK, 2, false, 0, GELU, RES, PIX, 192>(p, smem, m0, n0, wave, lane); break;
      case 1: gemm256_wave<NK, 1, false, 0, GELU, RES, PIX, 192>(p, smem, m0, n0, wave, lane); break;
      default: gemm256_wave<NK, 0, false, 0, GELU, RES, PIX, 192>(p, smem, m0, n0, wave, lane); break;
    }
    return;
  }
  switch (ntj) {
    case 4: gemm256_wave<NK, 4, false, 0, GELU, RES, PIX>(p, smem, m0, n0, wave, lane); break;
    case 3: gemm256_wave<NK, 3, false, 0, GELU, RES, PIX>(p, smem, m0, n0, wave, lane); break;
    case 2: gemm256_wave<NK, 2, false, 0, GELU, RES, PIX>(p, smem, m0, n0, wave, lane); break;
    case 1: gemm256_wave<NK, 1, false, 0, GELU, RES, PIX>(p, smem, m0, n0, wave, lane); break;
    default: gemm256_wave<NK, 0, false, 0, GELU, RES, PIX>(p, smem, m0, n0, wave, lane); break;
  }
}

}  // namespace

bool gemm256_supported(int M, int N, int K) {
  return M >= 256 && N % 256 == 0 && K % 64 == 0 && K >= 64;
}

ns_status launch_gemm256(const uint16_t *a, const uint16_t *w, const float *bias, const uint16_t *r,
                         uint16_t *c, int M, int N, int K, bool gelu, hipStream_t s, int batch,
                         long long a_stride, long long c_stride, const PixelRows *pixels) {
  if (!gemm256_supported(M, N, K)) return fail(NS_ERR_UNSUPPORTED, "GEMM shape M=%d N=%d K=%d", M, N, K);
  if ((long long)M * K * 2 >= 0x7fffffffLL || (long long)N * K * 2 >= 0x7fffffffLL)
    return fail(NS_ERR_UNSUPPORTED, "GEMM operand beyond 2 GiB");
  Gemm256Params p{{a, w, r, bias, c, M, N, K}, N / 256, 0, 0, 0, batch, a_stride, c_stride, {}};
  if (pixels) p.pix = *pixels;
  const int q = M / 256, rem = M % 256;
  p.extended = (rem > 0 && rem <= 32) ? 1 : 0;
  p.ntm = (rem == 0 || p.extended) ? q : q + 1;
  p.n256 = p.ntm;
  {
    // Rows of tiles: a of 256 token rows, then b of 192, a*256 + b*192 >= M.  Workgroups start in
    // launch order, a CU takes the next one when it is free: the mix with the shortest makespan
    // (a 192-row tile costs 0.8 of a 256-row one: 12288 rows against 16384, launches of whole rounds of the one or the other, K x N 1024 x 3072
    // 69.2 and 86.4 us, 4096 x 1024 73.4 and 94.0, the most 0.84, 1024 x 1024, the least 0.72, 4096 x 4096).
    const int cus = device_cu_count();
    auto makespan = [&](long long na, long long nb) -> double {
      // na*ntn tiles of cost 1.0, then nb*ntn of cost 0.8, each given to the unit that is free first.
      // After the tall tiles n2 units are free at t2 and the other n1 one tile time earlier, at t1.
      const long long ta = na * p.ntn * batch;
      long long left = nb * p.ntn * batch;
      const long long n2 = ta % cus, n1 = cus - n2;
      double t1 = (double)(ta / cus), t2 = t1 + 1.0;
      double end = n2 ? t2 : t1;
      while (left > 0) {
        if (n2 == 0 || t1 <= t2) {
          left -= std::min(left, n1);
          t1 += 0.8;
          end = std::max(end, t1);
        } else {
          left -= std::min(left, n2);
          t2 += 0.8;
          end = std::max(end, t2);
        }
      }
      return end;
    };
    double best = makespan(p.ntm, 0);    // (the ninth slab of an extended tile is not counted: it is cheap)
    int best_a = p.ntm, best_b = 0;
    const int max_b = (M + 191) / 192;
    for (int nb = 1; nb <= max_b; nb++) {
      const long long covered = (long long)nb * 192;
      const int na = covered >= M ? 0 : (int)((M - covered + 255) / 256);
      const double t = makespan(na, nb);
      if (t < best - 1e-9) { best = t; best_a = na; best_b = nb; }
    }
    if (best_b > 0) { p.n256 = best_a; p.ntm = best_a + best_b; p.extended = 0; }
  }
  const long long wgs = (long long)p.ntm * p.ntn * batch + (pixels ? ((long long)batch * N + 255) / 256 : 0);
  if (wgs > 0x7fffffffLL) return fail(NS_ERR_UNSUPPORTED, "GEMM grid too large");
  typedef void (*kern_t)(Gemm256Params);
  // K = 64 and 128: the pipeline is three slices deep, they have instantiations without it (16385 x 1024: 10.8 and
  // 12.0 us, with residual 12.8 and 14.2)
#define NS_KERNS(NK)                                                                                                     \
  {gemm256_bf16_kernel<NK, false, false>, gemm256_bf16_kernel<NK, false, true>, gemm256_bf16_kernel<NK, true, false>,     \
   gemm256_bf16_kernel<NK, true, true>}
  static const kern_t kerns[3][4] = {NS_KERNS(0), NS_KERNS(1), NS_KERNS(2)};
#undef NS_KERNS
  const kern_t kern = pixels ? gemm256_bf16_kernel<0, false, true, true> : kerns[K >= 192 ? 0 : K / 64][(gelu ? 2 : 0) + (r ? 1 : 0)];
  const ns_status rs = reserve_lds_once(reinterpret_cast<const void *>(kern), kGemmLds);
  if (rs != NS_OK) return rs;
  hipLaunchKernelGGL(kern, dim3((unsigned)wgs), dim3(256), kGemmLds, s, p);
  return check_launch("gemm256_bf16_kernel");
}

}  // namespace ns
