// Shared by the linear maps' kernels (ns_gemm256.hip, ns_gemm128.hip): C[m][n] = sum_k A[m][k] W[n][k] + bias[n], optional exact
// GELU, optional residual R[m][n].
#pragma once
#include "ns_common.h"

namespace ns {

struct GemmIo {
  const uint16_t *a, *w, *r;
  const float *bias;
  uint16_t *c;
  int M, N, K;
};

typedef bf16x8 __attribute__((address_space(3))) *lds_bf16x8_ptr;

// Rows that are patches of an image, read from its pixels: byte offset of 16-byte chunk `chunk` (of the eight of a slice of 64
// columns) of patch m, and of slice kt.
__device__ __forceinline__ uint32_t pixel_chunk(const PixelRows &p, int m, uint32_t chunk) {
  const int r = div_small(m, 1.f / (float)p.grid_w), c = m - r * p.grid_w;
  return (((uint32_t)r << p.lside) + (chunk >> p.lchunks)) * p.row_bytes + ((uint32_t)c << (p.lside + 1)) +
         16u * (chunk & ((1u << p.lchunks) - 1u));
}
__device__ __forceinline__ size_t pixel_slice(const PixelRows &p, int kt) {
  const int ls = 2 * p.lside - 6;              // log2 of a channel's slices; a slice is 8 >> lchunks rows of pixels
  return (size_t)(kt >> ls) * p.plane_bytes + (size_t)((kt & ((1 << ls) - 1)) << (3 - p.lchunks)) * p.row_bytes;
}
// x[b, 0, :] = cls + pos, the row in front of an image's patches: workgroup `wg` of those that do this
__device__ __forceinline__ void cls_rows(const PixelRows &p, int wg, int dim, int tid) {
  const long long t = (long long)wg * 256 + tid;
  if (t >= (long long)p.images * dim) return;
  const int b = (int)(t / dim), d = (int)(t - (long long)b * dim);
  const float v = bf16_lo((uint32_t)p.cls[d]) + bf16_lo((uint32_t)p.pos[d]);
  p.x[b * p.image_stride + d] = (uint16_t)(pack_bf16(v, 0.f) & 0xffffu);
}

// ---- epilogue of NS slabs of 32 weights x TOK tokens: accumulators -> LDS (fp32, [token][32*NS n]) -> lanes that
// own 8 consecutive n of one token: + bias, GELU, + residual, one 16-byte store.  A wave has its SIMD to itself here, so
// every latency it waits for is lost: the next slab is staged (two buffers) and its residual rows are requested before
// this one is finished, the staged values are read four passes ahead, and nothing is loaded behind a store that
// would have to be waited for with it (one in-order counter).  Lanes past the last row, whose inputs repeat it, store
// its values once more, to the same place: no branch around the stores.  Against an epilogue that staged, loaded and read each
// slab and pass in turn (32 LDS latencies and four drained stores a tile; whole calls): 16385 x 1024 x 1024 + residual 38.0 -> 36.7 us,
// 16385 x 4096 x 1024 + GELU 153 -> 148; 9832 rows: 26.0 -> 24.0 and 100 -> 96, x 3072 x 1024 63 -> 61; K = 4096 as before.
template <int NS, int TOK = 32>
struct Epi {
  static constexpr int LPT = NS * 4;                          // lanes per token row
  static constexpr int TPP = 64 / LPT, PASSES = TOK / TPP;    // tokens per pass
  static constexpr int AHEAD = PASSES < 4 ? PASSES : 4;
  static constexpr int kRow = NS * 128 + 16;                  // bytes per staged output row: 32 * NS floats + 16 pad
  static constexpr int kBytes = TOK * kRow;
  static __device__ __forceinline__ int col(int nbase, int lane) { return nbase + 8 * (lane & (LPT - 1)); }
  static __device__ __forceinline__ size_t at(const GemmIo &p, int mbase, int nbase, int ps, int lane) {
    return (size_t)min(mbase + TPP * ps + lane / LPT, p.M - 1) * p.N + col(nbase, lane);
  }
  static __device__ __forceinline__ void load_bias(const GemmIo &p, int nbase, int lane, f32x4 (&b)[2]) {
    b[0] = *reinterpret_cast<const f32x4 *>(p.bias + col(nbase, lane));
    b[1] = *reinterpret_cast<const f32x4 *>(p.bias + col(nbase, lane) + 4);
  }
  static __device__ __forceinline__ void load_residual(const GemmIo &p, int mbase, int nbase, int lane, uint4 (&res)[PASSES]) {
#pragma unroll
    for (int ps = 0; ps < PASSES; ps++) res[ps] = *reinterpret_cast<const uint4 *>(p.r + at(p, mbase, nbase, ps, lane));
  }
  // half: tokens 0..15 or 16..31 of the slab.  (A row of the staging area is four banks further than the one before: 16
  // lanes write 64 different banks.)
  static __device__ __forceinline__ void stage(unsigned char *ebuf, const f32x4 *(&tile)[2 * NS], int half, int lane) {
#pragma unroll
    for (int ti = 0; ti < 2 * NS; ti++)
      *reinterpret_cast<f32x4 *>(ebuf + (16 * half + (lane & 15)) * kRow + (16 * ti + 4 * (lane >> 4)) * 4) = *tile[ti];
  }
  // finishes the slab staged in ebuf; `then` is called when the first values have been asked for
  template <bool GELU, bool RES, class F>
  static __device__ __forceinline__ void emit(const GemmIo &p, const unsigned char *ebuf, const f32x4 (&b)[2],
                                              const uint4 (&res)[PASSES], int mbase, int nbase, int lane, F then) {
    const unsigned char *src = ebuf + lane / LPT * kRow + 32 * (lane & (LPT - 1));
    f32x4 v[AHEAD][2];
    auto fetch = [&](int ps, f32x4 (&x)[2]) {
      x[0] = *reinterpret_cast<const f32x4 *>(src + TPP * kRow * ps);
      x[1] = *reinterpret_cast<const f32x4 *>(src + TPP * kRow * ps + 16);
    };
#pragma unroll
    for (int i = 0; i < AHEAD; i++) fetch(i, v[i]);
    then();
    auto pass = [&](int ps, f32x4 (&x)[2], const uint4 &r4) {
      float o[8];
#pragma unroll
      for (int i = 0; i < 8; i++) o[i] = x[i >> 2][i & 3] + b[i >> 2][i & 3];
      fetch(min(ps + AHEAD, PASSES - 1), x);
      if (GELU) gelu_erf8(o);
      if (RES) {
        o[0] += bf16_lo(r4.x); o[1] += bf16_hi(r4.x); o[2] += bf16_lo(r4.y); o[3] += bf16_hi(r4.y);
        o[4] += bf16_lo(r4.z); o[5] += bf16_hi(r4.z); o[6] += bf16_lo(r4.w); o[7] += bf16_hi(r4.w);
      }
      const uint4 u = {pack_bf16(o[0], o[1]), pack_bf16(o[2], o[3]), pack_bf16(o[4], o[5]), pack_bf16(o[6], o[7])};
      *reinterpret_cast<uint4 *>(p.c + at(p, mbase, nbase, ps, lane)) = u;
    };
    if (RES) {
#pragma unroll
      for (int ps = 0; ps < PASSES; ps++) pass(ps, v[ps % AHEAD], res[ps]);
    } else {
#pragma unroll 1
      for (int ps = 0; ps < PASSES; ps += AHEAD)
#pragma unroll
        for (int i = 0; i < AHEAD; i++) pass(ps + i, v[i], res[0]);
    }
  }
};

}  // namespace ns
