// The global (CLS) query's attention row and the importance scores derived from it.
//
// Paper, "Memory-Efficiency Optimization": the global token attends to every token.
// Paper, "Time-Efficiency Optimization": a per-token importance score is read off the
// global token's attention weights; here: softmax weight of CLS on each patch key, averaged
// over heads.
//
// A few queries against T keys are a bandwidth problem, so the rows are cut into chunks of 512
// keys: cls_row_kernel streams K (and V) once, writes the raw logits and one softmax
// partial (max, sum, weighted V sum) per row and chunk; cls_combine_kernel merges the partials in
// chunk order; cls_scores_kernel turns logits + log-sum-exp into head-averaged weights.
#include "ns_window.h"

namespace ns {

namespace {

// 8 consecutive elements of a row as floats
__device__ __forceinline__ void load_row8(const float *p, float (&x)[8]) {
  const f32x4 a = *reinterpret_cast<const f32x4 *>(p), b = *reinterpret_cast<const f32x4 *>(p + 4);
#pragma unroll
  for (int e = 0; e < 4; e++) { x[e] = a[e]; x[4 + e] = b[e]; }
}
__device__ __forceinline__ void load_row8(const uint16_t *p, float (&x)[8]) { unpack8(*reinterpret_cast<const u32x4 *>(p), x); }

// One global token and K only (scoring without an attention output): grid (chunks, H, B), 256
// threads, lane = (key slot, 8-channel slice), 8 lanes per key row, every load of a wave's 128 keys
// in flight at once.  Bound: HBM.  For a single row the matrix instructions of the kernel below
// are work for 15 or 31 padding columns: 2 x 16384 keys x 16 heads bf16 took 13.9 us here and
// 16.4 us there, 4 x 9825 x 24 fp32 43 against 57 us.
//
// LEAN: a logit is stored as soon as it is known, and fewer loads are in flight; bf16 then takes 42 registers instead
// of 71, eight workgroups per CU instead of seven.  All loads first is faster by itself (2 x 16384 keys 21.8
// against 23.0 us, 8 x 16384 59.6 against 63.5), the eighth workgroup where it saves a round of workgroups (60000 keys,
// 1888 workgroups: 40.4 against 35.4 us; 4 x 9825 x 24 heads, 1920: 38.0 against 33.8; 2 x 60000: 62.6 against 58.6).
template <typename T, bool LEAN>
__global__ __launch_bounds__(256) void cls_scan_kernel(const T *q, const T *k, int64_t sb, int64_t sh, int64_t st,
                                                       int T_, int H, float scale, float *logits, float *partials,
                                                       int nchunks) {
  constexpr int kSteps = kClsChunk / (4 * 8);   // 4 waves x 8 keys per wave-step
  const int chunk = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int slot = lane >> 3, sub = lane & 7;
  const T *kb = k + b * sb + h * sh + sub * 8;
  __shared__ float red[4];

  float q8[8];
  load_row8(q + b * sb + h * sh + sub * 8, q8);
#pragma unroll
  for (int e = 0; e < 8; e++) q8[e] *= scale;
  const int key0 = chunk * kClsChunk + wave * (kSteps * 8) + slot;
  float *lrow = logits + ((size_t)b * H + h) * T_;
  float s[kSteps];
  float mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < kSteps; i++) {
    const int key = key0 + i * 8;
    float k8[8];
    load_row8(kb + (int64_t)min(key, T_ - 1) * st, k8);    // (clamped, not skipped: a branch would wait for each load)
    float acc = 0.f;
#pragma unroll
    for (int e = 0; e < 8; e++) acc = __builtin_fmaf(q8[e], k8[e], acc);
    // sum the 8 channel slices of the row (all lanes of the slot end up with the logit)
    acc += __shfl_xor(acc, 1);
    acc += __shfl_xor(acc, 2);
    acc += __shfl_xor(acc, 4);
    s[i] = key < T_ ? acc : -INFINITY;
    mx = fmaxf(mx, s[i]);
    if (LEAN && sub == 0 && key < T_) lrow[key] = acc;
  }
  if (!LEAN)
#pragma unroll
    for (int i = 0; i < kSteps; i++)
      if (sub == 0 && key0 + i * 8 < T_) lrow[key0 + i * 8] = s[i];
  mx = fmaxf(mx, __shfl_xor(mx, 8));
  mx = fmaxf(mx, __shfl_xor(mx, 16));
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  if (lane == 0) red[wave] = mx;
  __syncthreads();
  const float M = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));   // finite: chunk non-empty
  __syncthreads();
  float l = 0.f;
#pragma unroll
  for (int i = 0; i < kSteps; i++) l += __builtin_amdgcn_exp2f((s[i] - M) * kLog2e);
#pragma unroll
  for (int sft = 8; sft < 64; sft <<= 1) l += __shfl_xor(l, sft);
  if (lane == 0) red[wave] = l;
  __syncthreads();
  if (tid == 0) {
    float *rec = partials + (((size_t)b * H + h) * nchunks + chunk) * kClsPartialFloats;
    rec[0] = M;
    rec[1] = (red[0] + red[1]) + (red[2] + red[3]);
  }
}

// grid (chunks * groups of global rows * H * B): one workgroup per chunk of 512 keys and group of
// global rows of a head (ns_window.h).  Bound: HBM, K (and V) are read once.
template <class S, bool WITH_V, bool LOGITS>
__global__ __launch_bounds__(256, 2) void cls_row_kernel(GlobalRows p, int heads, int G, int T_, int groups, int nchunks) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  global_rows_chunk<S, WITH_V, LOGITS>(p, heads, G, T_, groups, nchunks, blockIdx.x, smem,
                                       __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), threadIdx.x & 63);
}

__device__ __forceinline__ void store_out(float *p, float x) { *p = x; }
__device__ __forceinline__ void store_out(uint16_t *p, float x) { *p = (uint16_t)(pack_bf16(x, 0.f) & 0xffffu); }

// grid (H*G, B), 1024 threads: thread (group g = tid/64, channel d = tid%64).  First the maximum
// over all records, then group g sums the records g, g+16, g+32, ... weighted against that maximum
// (no running maximum: the loads do not depend on each other and eight are kept in flight - the
// records were written by other workgroups, so every load is a long trip), and the sixteen groups
// are added in group order.  The order of operations is fixed, so the result is deterministic.
constexpr int kCombineThreads = 1024, kCombineGroups = kCombineThreads / 64;
template <typename T, bool WITH_V>
__device__ __forceinline__ void cls_combine_body(int hg, int b, const float *partials, int nchunks, int H, int G,
                                                 T *out, int64_t osb, int64_t osh, int64_t ost, float *lse) {
  const int tid = threadIdx.x, g = tid >> 6, d = tid & 63;
  const int h = hg / G, gq = hg - h * G;
  const float *rec = partials + ((size_t)b * H * G + hg) * nchunks * kClsPartialFloats;
  __shared__ float sm[kCombineGroups], sl[kCombineGroups], so[kCombineGroups][64];
  float M = -INFINITY;
  for (int c = tid; c < nchunks; c += kCombineThreads) M = fmaxf(M, rec[(size_t)c * kClsPartialFloats]);
#pragma unroll
  for (int sft = 1; sft < 64; sft <<= 1) M = fmaxf(M, __shfl_xor(M, sft));
  if (d == 0) sm[g] = M;
  __syncthreads();
  M = sm[0];
#pragma unroll
  for (int i = 1; i < kCombineGroups; i++) M = fmaxf(M, sm[i]);   // finite: there is at least one record with a key
  float L = 0.f, O = 0.f;
#pragma unroll 8
  for (int c = g; c < nchunks; c += kCombineGroups) {
    const float *r = rec + (size_t)c * kClsPartialFloats;
    const float w = __builtin_amdgcn_exp2f((r[0] - M) * kLog2e);   // 0 for a record without keys
    L = __builtin_fmaf(r[1], w, L);
    if (WITH_V) O = __builtin_fmaf(r[2 + d], w, O);
  }
  if (d == 0) sl[g] = L;
  so[g][d] = O;
  __syncthreads();
  if (g != 0) return;
  float Lt = 0.f, Ot = 0.f;
#pragma unroll
  for (int i = 0; i < kCombineGroups; i++) {
    Lt += sl[i];
    Ot += so[i][d];
  }
  if (WITH_V) store_out(out + b * osb + h * osh + gq * ost + d, Ot / Lt);
  if (lse && d == 0) lse[(size_t)b * H * G + hg] = M + __builtin_amdgcn_logf(Lt) * kLn2;
}

template <typename T, bool WITH_V>
__global__ __launch_bounds__(kCombineThreads) void cls_combine_kernel(const float *partials, int nchunks, int H,
                                                                      int G, T *out, int64_t osb, int64_t osh,
                                                                      int64_t ost, float *lse) {
  cls_combine_body<T, WITH_V>(blockIdx.x, blockIdx.y, partials, nchunks, H, G, out, osb, osh, ost, lse);
}

// Workgroup `blk` of image b scores THREADS / GROUPS patches: thread = (patch, group of rows).  H counts the global
// rows of an image (heads x global tokens): the score is the mean over all of them, every fourth row summed by itself and the four sums
// added in order, so that it does not depend on the launch.  lse given directly, or recomputed per row from the (max, sum) of the partial records.
// Bound: latency, of the records and then of a thread's share of the logits, which come from other XCDs' L2s: hence four groups and up to
// eight loads on their way.  (A thread per patch that went through all rows: 80 rows, 2 x 10000 patches, 12.3 us the launch, this 7.7.)
// Where that many threads are more than the chip holds at once, a thread takes a patch's rows alone.
constexpr int kRowSums = 4;
template <int THREADS, int GROUPS>
__device__ __forceinline__ void cls_scores_body(int blk, int b, const float *logits, const float *lse,
                                                const float *partials, int nchunks, int H, int T_, int G,
                                                float *scores) {
  constexpr int nthreads = THREADS, kPatches = THREADS / GROUPS, kOwn = kRowSums / GROUPS;
  __shared__ float s_lse[1024], s_part[GROUPS > 1 ? GROUPS : 1][GROUPS > 1 ? kPatches : 1];
  const int tid = threadIdx.x;
  if (lse) {
    for (int h = tid; h < H; h += nthreads) s_lse[h] = lse[(size_t)b * H + h];
  } else {
    // 16 lanes per head: each merges every 16th record, then the 16 are merged pairwise (fixed order)
    const int sub = tid & 15;
    for (int h = tid >> 4; h < H; h += nthreads >> 4) {
      const float *rec = partials + ((size_t)b * H + h) * nchunks * kClsPartialFloats;
      float M = -INFINITY, L = 0.f;
      for (int c = sub; c < nchunks; c += 16) {
        const float mc = rec[c * kClsPartialFloats], lc = rec[c * kClsPartialFloats + 1];
        const float Mn = fmaxf(M, mc);
        L = L * __builtin_amdgcn_exp2f((M - Mn) * kLog2e) + lc * __builtin_amdgcn_exp2f((mc - Mn) * kLog2e);
        M = Mn;
      }
#pragma unroll
      for (int sft = 1; sft < 16; sft <<= 1) {
        const float Mo = __shfl_xor(M, sft), Lo = __shfl_xor(L, sft);
        const float Mn = fmaxf(M, Mo);
        // a lane without records has M = -inf, L = 0: its weight is exp2(-inf) = 0 unless both are
        // empty, which cannot happen for all 16 (there is at least one record)
        const float wa = Mn == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((M - Mn) * kLog2e);
        const float wb = Mn == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((Mo - Mn) * kLog2e);
        // both lanes of a pair must add in the same order to agree bit for bit
        const bool lowl = (sub & sft) == 0;
        L = lowl ? L * wa + Lo * wb : Lo * wb + L * wa;
        M = Mn;
      }
      if (sub == 0) s_lse[h] = M + __builtin_amdgcn_logf(L) * kLn2;
    }
  }
  __syncthreads();
  const int N = T_ - G, g = tid / kPatches, lj = tid % kPatches, j = blk * kPatches + lj;
  const float *row = logits + (size_t)b * H * T_ + G + min(j, N - 1);
  auto weight = [&](int h) { return __builtin_amdgcn_exp2f((row[(size_t)h * T_] - s_lse[h]) * kLog2e); };
  float acc[kOwn] = {};
  int h = g;
  if (kOwn > 1)
#pragma unroll 2
    for (; h + kRowSums <= H; h += kRowSums)
#pragma unroll
      for (int i = 0; i < kOwn; i++) acc[i] += weight(h + i);
#pragma unroll 8
  for (int i = 0; h < H; h += GROUPS, i++) {
    const float w = weight(h);
#pragma unroll
    for (int j = 0; j < kOwn; j++) acc[j] += kOwn == 1 || i == j ? w : 0.f;
  }
  static_assert(kOwn == 1 || GROUPS == 1, "sums in the order of their rows");
  if (GROUPS > 1) {
    s_part[g][lj] = acc[0];
    __syncthreads();
    if (g != 0) return;
  }
  if (j >= N) return;
  float sum = acc[0];
#pragma unroll
  for (int i = 1; i < kRowSums; i++) sum += GROUPS > 1 ? s_part[i % GROUPS][lj] : acc[i % kOwn];
  scores[(size_t)b * N + j] = sum / (float)H;
}

// grid (ceil(N / (THREADS / GROUPS)), B)
template <int THREADS, int GROUPS>
__global__ __launch_bounds__(THREADS) void cls_scores_kernel(const float *logits, const float *lse, const float *partials, int nchunks,
                                                             int H, int T_, int G, float *scores) {
  cls_scores_body<THREADS, GROUPS>(blockIdx.x, blockIdx.y, logits, lse, partials, nchunks, H, T_, G, scores);
}

// Both in one launch, grid (H + ceil(N / (1024 / GROUPS)), B), 1024 threads: the first H workgroups of an image
// merge the records of one global row each (output row and log-sum-exp), the others score 1024 / GROUPS
// patches each, with the log-sum-exps they derive from the records themselves.
template <typename T, int GROUPS>
__global__ __launch_bounds__(kCombineThreads) void cls_combine_scores_kernel(const float *partials, int nchunks,
                                                                             int heads, int G, T *out, int64_t osb,
                                                                             int64_t osh, int64_t ost, float *lse,
                                                                             const float *logits, int T_,
                                                                             float *scores) {
  const int H = heads * G;
  if ((int)blockIdx.x < H)
    cls_combine_body<T, true>(blockIdx.x, blockIdx.y, partials, nchunks, heads, G, out, osb, osh, ost, lse);
  else
    cls_scores_body<kCombineThreads, GROUPS>(blockIdx.x - H, blockIdx.y, logits, nullptr, partials, nchunks, H, T_, G, scores);
}

}  // namespace

template <class S, bool WITH_V, bool LOGITS>
static ns_status launch_rows(const ns_attn_desc &d, const void *q, const void *k, const void *v, float *logits, float *partials,
                             hipStream_t s) {
  const GlobalRows p = global_rows<S>(d, q, k, v, logits, partials);
  const int nch = cls_num_chunks(d.tokens), groups = (d.n_global + global_group_rows<S>() - 1) / global_group_rows<S>();
  const long long wgs = (long long)nch * groups * d.heads * d.batch;
  if (wgs > 0x7fffffffLL) return fail(NS_ERR_UNSUPPORTED, "launch grid too large");
  const auto kern = cls_row_kernel<S, WITH_V, LOGITS>;
  const ns_status rs = reserve_lds_once(reinterpret_cast<const void *>(kern), kWindowLds);
  if (rs != NS_OK) return rs;
  hipLaunchKernelGGL(kern, dim3((unsigned)wgs), dim3(256), kWindowLds, s, p, d.heads, d.n_global, d.tokens, groups, nch);
  return check_launch("cls_row_kernel");
}

ns_status launch_cls_row(const ns_attn_desc &d, const void *q, const void *k, const void *v,
                         float *logits, float *partials, hipStream_t s) {
  const dim3 grid(cls_num_chunks(d.tokens), d.heads, d.batch), blk(256);
  const bool single = d.n_global == 1;
  if (v)     // several rows in bf16, a positive scale, 32-bit row offsets (the sweep, where it is forced on them)
    return logits ? launch_rows<StepBf16, true, true>(d, q, k, v, logits, partials, s)
                  : launch_rows<StepBf16, true, false>(d, q, k, v, logits, partials, s);
  if (!single) {
    if (d.dtype == NS_F32) return launch_rows<StepF32<float>, false, true>(d, q, k, v, logits, partials, s);
    // (the bf16 step wants a positive scale and 32-bit row offsets)
    if (d.scale > 0.f && (long long)d.tokens * d.q_stride_t * 2 < 0x7fffffffLL)
      return launch_rows<StepBf16, false, true>(d, q, k, v, logits, partials, s);
    return launch_rows<StepF32<uint16_t>, false, true>(d, q, k, v, logits, partials, s);
  }
  if (d.dtype == NS_F32) {
    hipLaunchKernelGGL((cls_scan_kernel<float, false>), grid, blk, 0, s, static_cast<const float *>(q), static_cast<const float *>(k),
                       d.q_stride_b, d.q_stride_h, d.q_stride_t, d.tokens, d.heads, d.scale, logits, partials, (int)grid.x);
  } else {
    const long long wgs = (long long)grid.x * d.heads * d.batch, seven = 7LL * device_cu_count(), eight = 8LL * device_cu_count();
    const bool lean = (wgs + seven - 1) / seven > (wgs + eight - 1) / eight;
    hipLaunchKernelGGL((lean ? cls_scan_kernel<uint16_t, true> : cls_scan_kernel<uint16_t, false>), grid, blk, 0, s,
                       static_cast<const uint16_t *>(q), static_cast<const uint16_t *>(k), d.q_stride_b, d.q_stride_h,
                       d.q_stride_t, d.tokens, d.heads, d.scale, logits, partials, (int)grid.x);
  }
  return check_launch("cls_scan_kernel");
}

ns_status launch_cls_combine(const ns_attn_desc &d, const float *partials, void *out, float *lse,
                             bool with_v, hipStream_t s, int nchunks) {
  const int nch = nchunks > 0 ? nchunks : cls_num_chunks(d.tokens);
  dim3 grid(d.heads * d.n_global, d.batch), blk(kCombineThreads);
  if (d.dtype == NS_F32) {
    if (with_v)
      hipLaunchKernelGGL((cls_combine_kernel<float, true>), grid, blk, 0, s, partials, nch, d.heads,
                         d.n_global, static_cast<float *>(out), d.out_stride_b, d.out_stride_h, d.out_stride_t, lse);
    else
      hipLaunchKernelGGL((cls_combine_kernel<float, false>), grid, blk, 0, s, partials, nch, d.heads,
                         d.n_global, static_cast<float *>(out), d.out_stride_b, d.out_stride_h, d.out_stride_t, lse);
  } else {
    if (with_v)
      hipLaunchKernelGGL((cls_combine_kernel<uint16_t, true>), grid, blk, 0, s, partials, nch,
                         d.heads, d.n_global, static_cast<uint16_t *>(out), d.out_stride_b, d.out_stride_h,
                         d.out_stride_t, lse);
    else
      hipLaunchKernelGGL((cls_combine_kernel<uint16_t, false>), grid, blk, 0, s, partials, nch,
                         d.heads, d.n_global, static_cast<uint16_t *>(out), d.out_stride_b, d.out_stride_h,
                         d.out_stride_t, lse);
  }
  return check_launch("cls_combine_kernel");
}

// Four threads to a patch shorten a launch whose workgroups, of 1024 threads then, are all on the chip at once (two a CU).  More of them
// take a second round, each of them deriving the log-sum-exps anew: a thread per patch, eight workgroups a CU, is faster from there on.
// (cls_scores, 16 heads, four images, four threads to a patch against one: 32768 patches each, 512 workgroups, 53.4 us against 52.9; 33000
// patches 55.9 against 53.0; one head, one image of 262144 27.5 against 21.3.  80 rows, 16384 patches, 64 workgroups 36.6 against 40.9.)
static bool one_round_of_1024(long long wgs) { return wgs <= 2LL * device_cu_count(); }

ns_status launch_cls_combine_scores(const ns_attn_desc &d, const float *partials, void *out, float *lse,
                                    const float *logits, float *scores, hipStream_t s, int nchunks) {
  const int nch = nchunks > 0 ? nchunks : cls_num_chunks(d.tokens);
  const int N = d.tokens - d.n_global, H = d.heads * d.n_global;
  const bool four = one_round_of_1024((long long)(H + (N + 255) / 256) * d.batch);
  const int patches = four ? kCombineThreads / 4 : kCombineThreads;
  dim3 grid(H + (N + patches - 1) / patches, d.batch), blk(kCombineThreads);
#define NS_LAUNCH(T, GROUPS)                                                                                                  \
  hipLaunchKernelGGL((cls_combine_scores_kernel<T, GROUPS>), grid, blk, 0, s, partials, nch, d.heads, d.n_global,              \
                     static_cast<T *>(out), d.out_stride_b, d.out_stride_h, d.out_stride_t, lse, logits, d.tokens, scores)
  if (d.dtype == NS_F32) {
    if (four) NS_LAUNCH(float, 4);
    else NS_LAUNCH(float, 1);
  } else {
    if (four) NS_LAUNCH(uint16_t, 4);
    else NS_LAUNCH(uint16_t, 1);
  }
#undef NS_LAUNCH
  return check_launch("cls_combine_scores_kernel");
}

ns_status launch_cls_scores(int B, int H, int T, int G, const float *logits, const float *lse,
                            const float *partials, int nchunks, float *scores, hipStream_t s) {
  const dim3 grid((T - G + 255) / 256, B);
  if (one_round_of_1024((long long)grid.x * B))
    hipLaunchKernelGGL((cls_scores_kernel<1024, 4>), grid, dim3(1024), 0, s, logits, lse, partials, nchunks, H * G, T, G, scores);
  else
    hipLaunchKernelGGL((cls_scores_kernel<256, 1>), grid, dim3(256), 0, s, logits, lse, partials, nchunks, H * G, T, G, scores);
  return check_launch("cls_scores_kernel");
}

}  // namespace ns
