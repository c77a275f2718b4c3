// Internal helpers shared by the HIP translation units of libnsattn.so.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include "../../include/nsattn.h"

namespace ns {

// ---- error reporting -------------------------------------------------------
ns_status fail(ns_status code, const char *fmt, ...);
ns_status check_launch(const char *what);   // hipGetLastError -> NS_ERR_HIP

// ---- bf16 <-> fp32 on the device ------------------------------------------
typedef __bf16 bf16_t;
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf16_lo(uint32_t packed) { return __uint_as_float(packed << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t packed) { return __uint_as_float(packed & 0xffff0000u); }

// round-to-nearest-even pack of two floats into two bf16 (v_cvt_pk_bf16_f32 on gfx950)
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  f32x2 v = {lo, hi};
  bf16x2 r = __builtin_convertvector(v, bf16x2);
  return __builtin_bit_cast(uint32_t, r);
}

constexpr float kLog2e = 1.4426950408889634f;

// GELU with the Gaussian error function, 0.5 x (1 + erf(x / sqrt 2)), written so that the
// cancellation for negative x never happens: with E = erfc(|x| / sqrt 2) / 2,
//   gelu(x) = max(x, 0) - |x| E,   E = exp2(P(|x|)),
// where P is a polynomial of degree 8 fitted to log2 E (weighted least squares, reweighted until the largest error of
// |x| E is smallest, on [0, 6.5]; it falls for every larger |x|, so that E goes to 0 there).  Evaluated in fp32, |x| E is within 6.5e-8
// of the true value for all x, and E to 4e-7 of itself up to |x| = 1, 1.1e-6 up to 2, 3.8e-6 up to 3, 2e-3 up to 6.5 (the rational
// approximation 7.1.26 of Abramowitz & Stegun times exp(-x^2 / 2): 2.1e-7; 7e-7, 3.3e-6, 5.2e-5, 5e-3).
// Beyond 6.5, outside the fit, E falls too fast: by 2 % at 7, 19 % at 8, and from 10 on nothing of it is left (the rational form:
// 0.7 %, 1 %, 2 %).  What is lost there is below 6e-13 in the result, less than the form's error anywhere else; a
// polynomial that keeps the tail to 4 % as well has degree 10, and its two further instructions per value take 3.5 % of the MLP's
// first product (16385 x 4096 x 1024: 148 -> 153 us).
// 11 vector instructions per value, one of them transcendental; the rational form has 13 and two.
constexpr float kGelu[9] = {-0.999999646325079f, -1.1511218255590818f, -0.4590842402002178f, -0.05284321485882337f,
                            0.007533510192487715f, -0.00047641503734017864f, -5.32491038671624e-05f,
                            1.2904940425108796e-05f, -7.46200327314319e-07f};
__device__ __forceinline__ float gelu_erf(float x) {
  const float ax = __builtin_fabsf(x);
  float q = kGelu[8];
#pragma unroll
  for (int i = 7; i >= 0; i--) q = __builtin_fmaf(q, ax, kGelu[i]);
  return __builtin_fmaf(-ax, __builtin_amdgcn_exp2f(q), __builtin_fmaxf(x, 0.f));
}
// The same for eight values, stage by stage, so that the eight dependency chains are interleaved: a wave that
// has its SIMD to itself otherwise waits out every link.  The empty asm statements between the
// stages keep the compiler from putting the chains back one after the other.
__device__ __forceinline__ void stage8(float (&a)[8]) {
  asm volatile("" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7]));
}
__device__ __forceinline__ void gelu_erf8(float (&o)[8]) {
  float q[8], r[8];
#pragma unroll
  for (int i = 0; i < 8; i++) q[i] = __builtin_fmaf(kGelu[8], __builtin_fabsf(o[i]), kGelu[7]);
  stage8(q);
#pragma unroll
  for (int c = 6; c >= 0; c--) {
#pragma unroll
    for (int i = 0; i < 8; i++) q[i] = __builtin_fmaf(q[i], __builtin_fabsf(o[i]), kGelu[c]);
    stage8(q);
  }
#pragma unroll
  for (int i = 0; i < 8; i++) q[i] = __builtin_amdgcn_exp2f(q[i]);
  stage8(q);
#pragma unroll
  for (int i = 0; i < 8; i++) r[i] = __builtin_fmaxf(o[i], 0.f);
  stage8(r);
#pragma unroll
  for (int i = 0; i < 8; i++) o[i] = __builtin_fmaf(-__builtin_fabsf(o[i]), q[i], r[i]);
  stage8(o);
}
constexpr float kLn2 = 0.6931471805599453f;

// ---- block lists of a pruned sequence: lists[b][blk][slot] is the token, counts[b][blk] the fill
struct BlockGeom {
  const int32_t *lists;    // [B, nbh*nbw, block*block] or nullptr
  const int32_t *counts;   // [B, nbh*nbw]              or nullptr
};

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// ---- device helpers shared by the MFMA kernels ------------------------------
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// A value the compiler can no longer trace back: what is computed from it stays where it is written
// instead of being hoisted out of a loop into registers that live for the whole kernel.
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// a / d for 0 <= a < 2^21 with inv = 1.f / d: the quotient's fraction is at least 0.5 / d away from an
// integer after adding 0.5, more than the two roundings can move it
__device__ __forceinline__ int div_small(int a, float inv) { return (int)(((float)a + 0.5f) * inv); }

// max(a, |b|), NaN if either is (v_maximum3_f32): fmaxf drops a NaN, and a check for overflow must see +inf - inf
__device__ __forceinline__ float max_abs(float a, float b) { return __builtin_elementwise_maximum(a, __builtin_fabsf(b)); }

// max / sum of a value over the two half-waves (lane l and lane l ^ 32); both lanes get it
__device__ __forceinline__ float half_swap_max(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_swap_sum(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// ... over the rows of 16 lanes (lane l and lane l ^ 16)
__device__ __forceinline__ float row_swap_max(float x) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float row_swap_sum(float x) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// x of another lane of the same 16 (DPP control CTRL)
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, 0xf, 0xf, true));
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppMirror8 = 0x141, kDppMirror16 = 0x140;
// max / sum over the wave, in every lane
__device__ __forceinline__ float wave_max(float x) {
  x = fmaxf(x, dpp<kDppXor1>(x));
  x = fmaxf(x, dpp<kDppXor2>(x));
  x = fmaxf(x, dpp<kDppMirror8>(x));
  x = fmaxf(x, dpp<kDppMirror16>(x));
  return half_swap_max(row_swap_max(x));
}
__device__ __forceinline__ float wave_sum(float x) {
  x += dpp<kDppXor1>(x);
  x += dpp<kDppXor2>(x);
  x += dpp<kDppMirror8>(x);
  x += dpp<kDppMirror16>(x);
  return half_swap_sum(row_swap_sum(x));
}
// 16 bytes per lane, global -> LDS, no registers: LDS address = lds + 16 * lane.  Issued as asm
// so that the compiler does not guard later LDS reads with a full vmcnt(0) wait (it cannot tell
// one tile's transfer from the next tile's, which is still in flight); the kernels order and
// count their memory requests themselves (wait_vm).
__device__ __forceinline__ void dma16(const char *base, uint32_t voff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(lds), "v"(voff), "s"(base) : "memory", "m0");
}
// 4 / 16 bytes per lane to global memory, issued from asm so that each is exactly one request
__device__ __forceinline__ void store4(void *ptr, float v) {
  asm volatile("global_store_dword %0, %1, off" :: "v"(ptr), "v"(v) : "memory");
}
// (a store of more than 8 bytes reads its data after it has been issued: two wait states before a vector instruction
// may write these registers, which the compiler cannot know of)
__device__ __forceinline__ void store16(void *ptr, u32x4 v) {
  asm volatile("global_store_dwordx4 %0, %1, off\n\ts_nop 2" :: "v"(ptr), "v"(v) : "memory");
}
// at most N vector memory requests of this wave still in flight (they complete in issue order)
template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

// ---- host helpers -------------------------------------------------------------
// Compute units of the current device (256 if the query fails).  Thread-safe; looked up once.
int device_cu_count();
// hipFuncSetAttribute(MaxDynamicSharedMemorySize) for a kernel that wants more than 64 KB of LDS;
// every kernel is set up once per process (thread-safe).  `slot` tells the kernels of a file apart.
ns_status reserve_lds_once(const void *kernel, int bytes);


// ---- launchers implemented in the individual .hip files --------------------
struct AttnArgs {
  ns_attn_desc d;
  const void *q, *k, *v;
  void *out;
  BlockGeom geom;
  hipStream_t stream;
  int kernel;            // the patch-query kernel chosen for this call (ns_api.hip: PatchKernel)
  int split = 0;         // waves per query tile of the window kernels: 1, 2 or 4, or 0: by size
};

// ns_attn_forward with one more knob: reuse_lists = the per-block token lists that an earlier call
// with the same descriptor, coords contents and workspace left in the workspace are still valid
// (a stack of blocks after its pruning stage), so they are not rebuilt.  scores != NULL: also the
// importance scores [B, T-G] (needs cls_logits), merged and scored in one launch.
ns_status attn_forward_impl(const ns_attn_desc *desc, const void *q, const void *k, const void *v, void *out,
                            float *cls_logits, float *cls_lse, float *scores, void *workspace,
                            size_t workspace_bytes, void *stream, bool reuse_lists);

// the descriptor checks of ns_attn_forward alone (status and message as that call would give)
ns_status attn_validate(const ns_attn_desc *desc);

// cls_scores behind its validation: shared by the entry point that takes a workspace and the one
// that brings its own scratch memory
ns_status cls_scores_impl(const ns_attn_desc *desc, const void *q, const void *k, float *scores,
                          void *workspace, size_t workspace_bytes, void *stream);

ns_status launch_block_lists(const ns_attn_desc &d, int32_t *lists, int32_t *counts, hipStream_t s);
// partials != NULL: the launch also computes the global rows' chunk records [B, H*G, cls_num_chunks, 66] and,
// with logits, their raw logits [B,H,G,T]
ns_status launch_attn_generic(const AttnArgs &a, float *logits, float *partials);
bool sweep_attn_supported(const ns_attn_desc &d);    // 8x8 blocks: key tiles shared along a row of blocks
// cls_partials != NULL: the kernel also computes the global query's row, [B,H,4*nbh,66] partial records
// (sweep_cls_chunks of them per head-image) and, with cls_logits, its raw logits [B,H,T]
ns_status launch_attn_sweep(const AttnArgs &a, float *cls_logits, float *cls_partials);
inline int sweep_cls_chunks(const ns_attn_desc &d) { return 4 * ((d.grid_h + 7) / 8); }
bool block16_attn_supported(const ns_attn_desc &d);  // blocks of 16 and its multiples: key tiles shared by a block's query tiles
ns_status launch_attn_block16(const AttnArgs &a, float *logits, float *partials);
bool ragged_attn_supported(const ns_attn_desc &d);   // bf16, head_dim 64: any complete grid or pruned sequence
ns_status launch_attn_ragged(const AttnArgs &a, float *logits, float *partials);
double ragged_attn_us(const ns_attn_desc &d);         // what its launch takes on a complete grid, roughly

// global-query (CLS) row: per-chunk partials, then a combine.
constexpr int kClsChunk = 512;                      // keys per workgroup of the row kernel
inline int cls_num_chunks(int tokens) { return (tokens + kClsChunk - 1) / kClsChunk; }
// partial record per (b, h, chunk): m, l, o[64]
constexpr int kClsPartialFloats = 2 + 64;
// v: NULL for scoring, which wants logits; else of a bf16 problem, logits or NULL
ns_status launch_cls_row(const ns_attn_desc &d, const void *q, const void *k, const void *v,
                         float *logits /* [B,H,G,T] */, float *partials, hipStream_t s);
ns_status launch_cls_combine(const ns_attn_desc &d, const float *partials, void *out, float *lse,
                             bool with_v, hipStream_t s, int nchunks = 0 /* 0: cls_num_chunks(tokens) */);
// lse given directly, or (lse == nullptr) recomputed from the row kernel's partials
// launch_cls_combine and the scoring of all patches in one launch (lse may be NULL)
ns_status launch_cls_combine_scores(const ns_attn_desc &d, const float *partials, void *out, float *lse,
                                    const float *logits, float *scores, hipStream_t s, int nchunks = 0);
ns_status launch_cls_scores(int B, int H, int T, int G, const float *logits, const float *lse,
                            const float *partials, int nchunks, float *scores, hipStream_t s);

// Where the rows of a product's first operand are patches of 8, 16, 32 pixels a side and it is read from the pixels themselves: a patch's row
// of pixels is then whole 16-byte pieces, and 64 columns of the matrix are whole rows of pixels.  The launch also writes the row in
// front of every image's patches.
struct PixelRows {
  int grid_w, lside, lchunks;           // patches in a row; log2 of a patch's side and of its 16-byte pieces a row
  int images;
  uint32_t row_bytes;                   // of the image
  size_t plane_bytes;                   // of a channel
  const uint16_t *cls, *pos;
  uint16_t *x;
  long long image_stride;               // of x, in elements
};

// linear map with fused epilogue, 256 x 256 workgroup tiles (ns_gemm256.hip); batch: so many of them with the
// same weights, bias and residual in one launch, rows and results at the given distances in elements
bool gemm256_supported(int M, int N, int K);
ns_status launch_gemm256(const uint16_t *a, const uint16_t *w, const float *bias, const uint16_t *r,
                         uint16_t *c, int M, int N, int K, bool gelu, hipStream_t s, int batch = 1,
                         long long a_stride = 0, long long c_stride = 0, const PixelRows *pixels = nullptr);
// ... with tiles of 128 x 32 tj, tj = 2 .. 6 (ns_gemm128.hip)
bool gemm128_supported(int N, int K);
ns_status launch_gemm128(const uint16_t *a, const uint16_t *w, const float *bias, const uint16_t *r,
                         uint16_t *c, int M, int N, int K, bool gelu, hipStream_t s, int tj, int batch = 1,
                         long long a_stride = 0, long long c_stride = 0, const PixelRows *pixels = nullptr);

// ws: topk_select_workspace_bytes(B, N) bytes, 16-byte aligned (nothing for short score rows)
size_t topk_select_workspace_bytes(int B, int N);
ns_status launch_topk_select(int B, int N, int k, const float *scores, const int32_t *coords_in,
                             int32_t *kept, int32_t *coords_out, void *ws, hipStream_t s);
ns_status launch_gather_rows(int B, int N, int k, int G, size_t row_bytes, const void *x,
                             const int32_t *kept, void *y, hipStream_t s);

}  // namespace ns
