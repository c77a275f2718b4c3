// bf16 MFMA GEMM with tiles of 128 (n) x 32 TJ (m), TJ = 2 .. 6, for linear maps whose 256 x 256 tiles leave CUs idle, and for
// N that 256 does not divide (gfx950).
//
// Bound: in a launch of one round of workgroups or less, the time of one tile: its K / 64 slices, each of which the matrix pipes
// take 128 TJ cycles for and the LDS 64 (4 + TJ) to read, and what comes before and after.  So the tiles are as small as lets
// all CUs work at once, a slice's transfers are requested four slices ahead (four LDS slots; the token rows of a tile are few, so
// that the weights' latency counts), the fragments of half a slice are read while the half before is multiplied, and there is one
// barrier a slice, between its halves: by then every wave has read all of it, so that the slot is free and what it
// waits for is the slice after.  A weight fragment stays for all token fragments, as in the larger kernel.
// Tiles of other heights than 128 rows let a launch that is a little too large for one round (4097 rows: 33 x 8 tiles of 128 rows) fit it.
// Measured, us, 256 x 256 tiles -> this: 449 x 1024 x 4096 + residual 53.6 -> 19.7, 1025 x 3072 x 1024 18.9 -> 12.2, 3137 x 1024 x 1024
// + residual 19.0 -> 11.9, 5184 x 1024 x 4096 + residual 55.7 -> 39.0; against an earlier kernel of 128 x 128 tiles, two slots and a wait for
// all transfers in every slice: 197 x 1024 x 4096 + residual 38 -> 20.
#include "ns_gemm.h"
#include <algorithm>
#include <type_traits>

namespace ns {

namespace {

struct Gemm128Params : GemmIo {
  int ntn, ntm;      // tiles along n and m
  int per_xcd;       // workgroups per XCD
  int batch;         // products of the same w, bias and r: a and c of the next one follow at these distances
  long long a_stride, c_stride;   // in elements
  PixelRows pix;
};

constexpr int kSlots = 4;
template <int TJ> constexpr int stage_bytes() { return TJ * 4096 + 16384; }   // 32 TJ token rows, 128 weight rows, 64 k each

// PIX: the token rows are patches, read from their pixels
template <int TJ, bool GELU, bool RES, bool PIX = false>
__global__ __launch_bounds__(256, 2) void gemm128_bf16_kernel(Gemm128Params p) {
  constexpr int kX = TJ * 4096, kStage = stage_bytes<TJ>(), kReq = 4 + TJ;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int l16 = lane & 15, wm = wave >> 1, wn = wave & 1;
  // workgroups are dealt round-robin to the 8 XCDs; each XCD gets a contiguous run of tiles, n fastest, so that the tiles that
  // share token rows meet in one L2
  if (PIX && (int)blockIdx.x >= 8 * p.per_xcd) {
    cls_rows(p.pix, (int)blockIdx.x - 8 * p.per_xcd, p.N, tid);
    return;
  }
  const int id = (int)(blockIdx.x & 7) * p.per_xcd + (int)(blockIdx.x >> 3), per = p.ntn * p.ntm;
  if (id >= per * p.batch) return;
  const int z = __builtin_amdgcn_readfirstlane(id / per), t0 = id - z * per;
  const int bm = __builtin_amdgcn_readfirstlane(t0 / p.ntn), m0 = bm * 32 * TJ, n0 = (t0 - bm * p.ntn) * 128;
  p.a += z * p.a_stride;
  p.c += z * p.c_stride;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const uint32_t lds0 = (uint32_t)(size_t)((__attribute__((address_space(3))) unsigned char *)smem);

  // ---- transfers: requests of 8 rows x 128 bytes; 16-byte chunk c of row r lies at chunk c ^ ((r >> 1) & 7), so that the 16
  // rows that 16 consecutive lanes read land on 16 different bank groups
  const uint32_t rowB = (uint32_t)p.K * 2u;
  const char *ab = reinterpret_cast<const char *>(p.a), *wb = reinterpret_cast<const char *>(p.w);
  const int drow = lane >> 3;
  auto dchunk = [&](int req) { return 16u * ((lane & 7) ^ ((4 * (req & 1) + (drow >> 1)) & 7)); };
  uint32_t woff[2], xoff[TJ];
#pragma unroll
  for (int j = 0; j < 2; j++) woff[j] = (uint32_t)(n0 + wave * 32 + drow) * rowB + dchunk(j);
#pragma unroll
  for (int j = 0; j < TJ; j++) {
    const int m = min(m0 + (wave * TJ + j) * 8 + drow, p.M - 1);     // rows past M repeat the last row
    xoff[j] = PIX ? pixel_chunk(p.pix, m, dchunk(wave * TJ + j) >> 4) : (uint32_t)m * rowB + dchunk(wave * TJ + j);
  }
  auto issue = [&](int kt, int j) {
    const uint32_t dst = lds0 + (uint32_t)(kt & (kSlots - 1)) * kStage;
    if (j < 4) dma16(wb + (size_t)kt * 128 + (size_t)j * 8 * rowB, woff[j & 1], dst + kX + (wave * 4 + j) * 1024);
    else dma16(ab + (PIX ? pixel_slice(p.pix, kt) : (size_t)kt * 128), xoff[j - 4], dst + (wave * TJ + j - 4) * 1024);
  };

  // ---- fragments of half a slice (32 k): lane (row l16, quarter lane/16) reads logical chunk 4*h + lane/16
  uint32_t frd[2];
#pragma unroll
  for (int h = 0; h < 2; h++) frd[h] = lds0 + l16 * 128 + 16 * ((4 * h + (lane >> 4)) ^ (l16 >> 1));
  bf16x8 fw[2][4], fx[2][TJ];
  auto read = [&](int h, int kt, int i) {
    const uint32_t at = frd[h] + (uint32_t)(kt & (kSlots - 1)) * kStage;
    if (i < 4) fw[h][i] = *(lds_bf16x8_ptr)(at + kX + (wn * 64 + i * 16) * 128);
    else fx[h][i - 4] = *(lds_bf16x8_ptr)(at + (wm * TJ + i - 4) * 16 * 128);
  };
  f32x4 acc[4][TJ];    // [16 weights][16 tokens]: register e = n 4*(lane/16) + e, token l16
#pragma unroll
  for (int i = 0; i < 4; i++)
#pragma unroll
    for (int j = 0; j < TJ; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto meet = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
  // slice kt has landed for every wave, with `behind` slices requested after it
  auto landed = [&](int behind) {
    if (behind >= 3) wait_vm<3 * kReq>();
    else if (behind == 2) wait_vm<2 * kReq>();
    else if (behind == 1) wait_vm<kReq>();
    else wait_vm<0>();
    meet();
  };
  // the products of one half, with the reads of the next half and, MOVE, the transfers of slice t + kSlots between them
  auto half = [&](auto h_c, auto read_c, auto move_c, int t) {
    constexpr int h = decltype(h_c)::value;
    constexpr bool kRead = decltype(read_c)::value, kMove = decltype(move_c)::value;
#pragma unroll
    for (int i = 0; i < 4 * TJ; i++) {
#pragma unroll
      for (int r = 0; r < 4 + TJ; r++)
        if (kRead && r * 2 * TJ / (4 + TJ) == i) read(1 - h, h ? t + 1 : t, r);
      acc[i / TJ][i % TJ] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[h][i / TJ], fx[h][i % TJ], acc[i / TJ][i % TJ], 0, 0, 0);
#pragma unroll
      for (int j = 0; j < kReq; j++)
        if (kMove && j * 4 * TJ / kReq == i) issue(t + kSlots, j);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  using H0 = std::integral_constant<int, 0>;
  using H1 = std::integral_constant<int, 1>;
  using Yes = std::true_type;
  using No = std::false_type;

  const int nk = p.K / 64;
#pragma unroll
  for (int s = 0; s < kSlots; s++)
    if (s < nk)
#pragma unroll
      for (int j = 0; j < kReq; j++) issue(s, j);
  landed(min(nk, kSlots) - 1);
#pragma unroll
  for (int i = 0; i < 4 + TJ; i++) read(0, 0, i);
  int t = 0;
  for (; t < nk - kSlots; t++) {
    half(H0{}, Yes{}, No{}, t);
    landed(2);
    half(H1{}, Yes{}, Yes{}, t);
  }
  for (; t < nk - 1; t++) {
    half(H0{}, Yes{}, No{}, t);
    landed(nk - 2 - t);
    half(H1{}, Yes{}, No{}, t);
  }
  // (no transfer is on its way any more: what the epilogue starts with may be asked for)
  const int mw = m0 + wm * 16 * TJ, nw = n0 + wn * 64;
  constexpr int kSlabs = (TJ + 1) / 2;
  using E = Epi<2>;
  using EH = Epi<2, 16>;               // the last half slab where TJ is odd
  f32x4 bias[2];
  uint4 res[2][E::PASSES] = {}, resh[EH::PASSES] = {};
  E::load_bias(p, nw, lane, bias);
  if (RES) E::load_residual(p, mw, nw, lane, res[0]);
  half(H0{}, Yes{}, No{}, t);
  half(H1{}, No{}, No{}, t);
  __syncthreads();                     // every wave is done with the stages: they become the epilogue's staging area
  unsigned char *const ebuf[2] = {smem + wave * E::kBytes, smem + (4 + wave) * E::kBytes};
  static_assert(8 * E::kBytes <= kSlots * kStage, "two staged slabs per wave");
  auto stage = [&](int s) {
#pragma unroll
    for (int j = 0; j < 2; j++)
      if (2 * s + j < TJ) {
        const f32x4 *tile[4];
#pragma unroll
        for (int i = 0; i < 4; i++) tile[i] = &acc[i][2 * s + j];
        E::stage(ebuf[s & 1], tile, j, lane);
      }
  };
  stage(0);
#pragma unroll
  for (int s = 0; s < kSlabs; s++) {
    auto then = [&]() {
      if (RES && s + 1 < kSlabs) {
        if (2 * s + 3 < TJ) E::load_residual(p, mw + (s + 1) * 32, nw, lane, res[(s + 1) & 1]);
        else EH::load_residual(p, mw + (s + 1) * 32, nw, lane, resh);
      }
      if (s + 1 < kSlabs) stage(s + 1);
    };
    if (2 * s + 1 < TJ) E::template emit<GELU, RES>(p, ebuf[s & 1], bias, res[s & 1], mw + s * 32, nw, lane, then);
    else EH::template emit<GELU, RES>(p, ebuf[s & 1], bias, resh, mw + s * 32, nw, lane, then);
  }
}

}  // namespace

bool gemm128_supported(int N, int K) { return N % 128 == 0 && K % 64 == 0 && K >= 64; }

ns_status launch_gemm128(const uint16_t *a, const uint16_t *w, const float *bias, const uint16_t *r,
                         uint16_t *c, int M, int N, int K, bool gelu, hipStream_t s, int tj, int batch,
                         long long a_stride, long long c_stride, const PixelRows *pixels) {
  if (!gemm128_supported(N, K)) return fail(NS_ERR_UNSUPPORTED, "GEMM needs N %% 128 == 0 and K %% 64 == 0 (N=%d K=%d)", N, K);
  if ((long long)M * K * 2 >= 0x7fffffffLL || (long long)N * K * 2 >= 0x7fffffffLL)
    return fail(NS_ERR_UNSUPPORTED, "GEMM operand beyond 2 GiB");
  Gemm128Params p{{a, w, r, bias, c, M, N, K}, N / 128, (M + 32 * tj - 1) / (32 * tj), 0, batch, a_stride, c_stride, {}};
  if (pixels) p.pix = *pixels;
  const long long tiles = (long long)p.ntn * p.ntm * batch, wgs = (tiles + 7) / 8 * 8;
  const long long cls = pixels ? ((long long)batch * N + 255) / 256 : 0;
  if (wgs + cls > 0x7fffffffLL) return fail(NS_ERR_UNSUPPORTED, "GEMM grid too large");
  p.per_xcd = (int)(wgs / 8);
  typedef void (*kern_t)(Gemm128Params);
#define NS_KERNS(TJ) \
  {gemm128_bf16_kernel<TJ, false, false>, gemm128_bf16_kernel<TJ, false, true>, gemm128_bf16_kernel<TJ, true, false>, gemm128_bf16_kernel<TJ, true, true>}
  static const kern_t kerns[5][4] = {NS_KERNS(2), NS_KERNS(3), NS_KERNS(4), NS_KERNS(5), NS_KERNS(6)};
#undef NS_KERNS
  static const kern_t pixel_kerns[5] = {gemm128_bf16_kernel<2, false, true, true>, gemm128_bf16_kernel<3, false, true, true>,
                                        gemm128_bf16_kernel<4, false, true, true>, gemm128_bf16_kernel<5, false, true, true>,
                                        gemm128_bf16_kernel<6, false, true, true>};
  const kern_t kern = pixels ? pixel_kerns[tj - 2] : kerns[tj - 2][(gelu ? 2 : 0) + (r ? 1 : 0)];
  const int lds = kSlots * (tj * 4096 + 16384);
  const ns_status rs = reserve_lds_once(reinterpret_cast<const void *>(kern), lds);
  if (rs != NS_OK) return rs;
  hipLaunchKernelGGL(kern, dim3((unsigned)(wgs + cls)), dim3(256), lds, s, p);
  return check_launch("gemm128_bf16_kernel");
}

}  // namespace ns
