// bf16 MFMA neighbourhood attention for every problem without a kernel of its own for its size: small
// complete grids, block sides that are neither 2, 4, 8 nor a multiple of 16, many global tokens, and
// pruned sequences (paper, "Time-Efficiency Optimization": after pruning the mask is still evaluated
// on each survivor's original grid position) (gfx950).
//
// One workgroup per tile of 64 queries, the tile's keys shared out over its four waves; the global
// rows' chunks ride in the same launch (ns_window.h).
#include "ns_window.h"

namespace ns {

namespace {

template <bool LISTS, bool MASK, int KS>
__global__ __launch_bounds__(256, 2) void attn_mfma_ragged_kernel(WindowParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  window_attention<StepBf16, 2, LISTS, MASK, KS>(p, smem);
}

}  // namespace

bool ragged_attn_supported(const ns_attn_desc &d) {
  return d.dtype == NS_BF16 && d.head_dim == 64 && d.radius == 1 && d.n_global >= 1 &&
         d.scale > 0.f &&
         (long long)d.tokens * d.q_stride_t * 2 < 0x7fffffffLL &&
         (long long)d.tokens * d.out_stride_t * 2 < 0x7fffffffLL;
}

// (a step of the cost model is 1.05 to 1.2 us: 128 x 128 x 16 heads x 2 with 8x8 blocks 113 steps, 127 us; where the sweep is the
// alternative, many tiles, the upper end)
double ragged_attn_us(const ns_attn_desc &d) {
  const WindowCost c = window_cost(d, 64);
  return 1.2 * c.of(c.split()) + 6.0;
}

ns_status launch_attn_ragged(const AttnArgs &a, float *logits, float *partials) {
  WindowParams p;
  int ks;
  const long long wgs = window_params<StepBf16, 2>(a, logits, partials, p, ks);
  if (wgs < 0) return fail(NS_ERR_UNSUPPORTED, "launch grid too large");
  const bool lists = a.d.coords != nullptr, mask = p.g.side > p.g.block;
  if (lists && (!p.g.lists || !p.g.counts))
    return fail(NS_ERR_INVALID_ARG, "the list kernel was launched without block lists");
  typedef void (*kern_t)(WindowParams);
#define NS_KERN(KS)                                                                                     \
  (lists ? attn_mfma_ragged_kernel<true, false, KS>                                                     \
         : (mask ? attn_mfma_ragged_kernel<false, true, KS> : attn_mfma_ragged_kernel<false, false, KS>))
  const kern_t kern = ks == 4 ? NS_KERN(4) : (ks == 2 ? NS_KERN(2) : NS_KERN(1));
#undef NS_KERN
  const ns_status rs = reserve_lds_once(reinterpret_cast<const void *>(kern), kWindowLds);
  if (rs != NS_OK) return rs;
  hipLaunchKernelGGL(kern, dim3((unsigned)wgs), dim3(256), kWindowLds, a.stream, p);
  return check_launch("attn_mfma_ragged_kernel");
}

}  // namespace ns
