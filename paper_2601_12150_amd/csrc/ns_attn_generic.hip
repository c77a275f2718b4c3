// Shape-generic neighbourhood attention in fp32 arithmetic (any block side, ragged blocks, pruned
// sequences, any strides, fp32 or bf16 storage), and the block-list builder for pruned sequences.
//
// Pattern: paper, "Memory-Efficiency Optimization" -- a patch query sees the patches of the
// 3x3 blocks around its own block plus the global token.
//
// One workgroup per tile of 32 queries, the tile's keys shared out over its four waves; products of fp32 values as six products of
// their bf16 parts on the matrix pipe (StepF32 in ns_window.h); the global rows' chunks ride in the same launch.
// Bound: at small sizes the chain of a wave's few steps, at large ones the transfers (a step of 32 keys and queries moves 16 KB into
// LDS: 9.3 TB/s on 64x64, four images); taking the parts is about 400 of a step's 580 vector instructions and stands between the products.
// Against v_mfma_f32_32x32x2_f32, which runs at the
// vector ALU's fp32 peak, us a call, 16 heads: 64x64 with 8x8 blocks, four images, 362 -> 270, one image 104 -> 80, 28x28 with 7x7 blocks 31.7
// -> 26, four images 75 -> 59; error of the rows against 64 bits 3.5e-7 -> 2.8e-7, with logits of +-60 1.3e-6 -> 0.98e-6.
#include "ns_window.h"

namespace ns {

namespace {

template <typename T, bool LISTS, bool MASK, int KS>
__global__ __launch_bounds__(256, 2) void attn_generic_kernel(WindowParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  window_attention<StepF32<T>, 1, LISTS, MASK, KS>(p, smem);
}

constexpr int kListRound = 4096;      // coordinates per round

// Pruned sequence: bucket the surviving patch tokens by block, preserving sequence order.
// grid (nblocks, B); each workgroup scans the image's coordinate list for its own block, 4096
// positions a round.  Bound: a chain of rounds; with 16 waves, and the next round's coordinates on their way while one is counted and
// placed, instead of four a round's instructions take a quarter of the time (9831 of 16384 patches, 8x8 blocks: 9.1 -> 5.6 us the
// launch).  That holds while all workgroups are on the chip at once, two of 16 waves a CU; beyond, where four waves fill it as well
// and each step of the prefix sum is done by fewer, four are faster (whole calls, us, 16 waves and four: 512 blocks 22.1 and 23.3, 529
// blocks 30.3 and 28.9, 1024 49.8 and 44.1, 16384 463 and 282).
template <int kListThreads>
__global__ __launch_bounds__(kListThreads) void block_lists_kernel(const int32_t *coords, int n_patch,
                                                          int n_global, int grid_h, int grid_w,
                                                          int block, int nbw, int nblocks, int cap,
                                                          int32_t *lists, int32_t *counts) {
  constexpr int kListWaves = kListThreads / 64, kListUnroll = kListRound / kListThreads;   // coordinates per thread and round
  static_assert(kListUnroll * kListWaves == 64, "one run per lane");
  const int blk = blockIdx.x, b = blockIdx.y;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int R = blk / nbw, C = blk - R * nbw;
  const int r0 = R * block, r1 = min(r0 + block, grid_h), c0 = C * block, c1 = min(c0 + block, grid_w);
  __shared__ int wcnt[2][kListUnroll * kListWaves];
  const int32_t *cb = coords + (size_t)b * n_patch;
  int32_t *lb = lists + ((size_t)b * nblocks + blk) * cap;
  int running = 0, flip = 0;
  uint32_t pc[kListUnroll];
  auto load = [&](int base) {
#pragma unroll
    for (int i = 0; i < kListUnroll; i++) pc[i] = (uint32_t)cb[min(base + kListThreads * i + tid, n_patch - 1)];
  };
  constexpr bool kAhead = kListUnroll <= 4;         // (16 of them ahead: 2 % more where the chip is full of workgroups)
  if (kAhead) load(0);
  for (int base = 0; base < n_patch; base += kListRound, flip ^= 1) {
    if (!kAhead) load(base);
    unsigned long long bal[kListUnroll];
#pragma unroll
    for (int i = 0; i < kListUnroll; i++) {
      const int r = (int)(pc[i] >> 16), c = (int)(pc[i] & 0xffffu);
      bal[i] = __ballot(base + kListThreads * i + tid < n_patch && r >= r0 && r < r1 && c >= c0 && c < c1);
      if (lane == 0) wcnt[flip][kListWaves * i + wave] = __popcll(bal[i]);
    }
    // the next round's coordinates, on their way while this one is counted and placed
    if (kAhead && base + kListRound < n_patch) load(base + kListRound);
    __syncthreads();
    // counts of the (group of kListThreads, wave) runs in sequence order: lane = run, prefix sum over the 64
    int pre = wcnt[flip][lane];
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) {
      const int up = __shfl_up(pre, s);
      pre += lane >= s ? up : 0;
    }
    const int total = __shfl(pre, 63);
    const int excl = pre - wcnt[flip][lane];
    if (total != 0)
#pragma unroll
      for (int i = 0; i < kListUnroll; i++) {
        const int off = running + __shfl(excl, kListWaves * i + wave) + __popcll(bal[i] & ((1ull << lane) - 1ull));
        if (((bal[i] >> lane) & 1) && off < cap) lb[off] = n_global + base + kListThreads * i + tid;
      }
    running += total;
  }
  if (tid == 0) counts[(size_t)b * nblocks + blk] = min(running, cap);
}

}  // namespace

ns_status launch_block_lists(const ns_attn_desc &d, int32_t *lists, int32_t *counts, hipStream_t s) {
  const int nbh = (d.grid_h + d.block - 1) / d.block, nbw = (d.grid_w + d.block - 1) / d.block;
  const dim3 grid(nbh * nbw, d.batch);
  const bool wide = (long long)nbh * nbw * d.batch <= 2LL * device_cu_count();
  const auto kern = wide ? block_lists_kernel<1024> : block_lists_kernel<256>;
  hipLaunchKernelGGL(kern, grid, dim3(wide ? 1024 : 256), 0, s, d.coords, d.tokens - d.n_global,
                     d.n_global, d.grid_h, d.grid_w, d.block, nbw, nbh * nbw, d.block * d.block,
                     lists, counts);
  return check_launch("block_lists_kernel");
}

template <typename T>
static ns_status launch_generic(const AttnArgs &a, float *logits, float *partials) {
  WindowParams p;
  int ks;
  const long long wgs = window_params<StepF32<T>, 1>(a, logits, partials, p, ks);
  if (wgs < 0) return fail(NS_ERR_UNSUPPORTED, "launch grid too large");
  const bool lists = a.d.coords != nullptr, mask = p.g.side > p.g.block;
  typedef void (*kern_t)(WindowParams);
#define NS_KERN(KS)                                                                                     \
  (lists ? attn_generic_kernel<T, true, false, KS>                                                      \
         : (mask ? attn_generic_kernel<T, false, true, KS> : attn_generic_kernel<T, false, false, KS>))
  const kern_t kern = ks == 4 ? NS_KERN(4) : (ks == 2 ? NS_KERN(2) : NS_KERN(1));
#undef NS_KERN
  const ns_status rs = reserve_lds_once(reinterpret_cast<const void *>(kern), kWindowLds);
  if (rs != NS_OK) return rs;
  hipLaunchKernelGGL(kern, dim3((unsigned)wgs), dim3(256), kWindowLds, a.stream, p);
  return check_launch("attn_generic_kernel");
}

ns_status launch_attn_generic(const AttnArgs &a, float *logits, float *partials) {
  return a.d.dtype == NS_F32 ? launch_generic<float>(a, logits, partials) : launch_generic<uint16_t>(a, logits, partials);
}

}  // namespace ns
