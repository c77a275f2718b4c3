// Ranking and compaction (paper, "Time-Efficiency Optimization": rank the tokens by
// importance, discard the lowest-scoring proportion, shorten the sequence).
//
// Exact k-th largest score on an order-preserving integer image of the floats, then an
// in-index-order compaction, so the kept indices come out ascending and exact ties resolve to
// the lower index.
//   topk_select_reg_kernel: rows of up to 32768 scores, one launch.  Every workgroup selects from all keys of its
//     image, held in registers, by 11-bit digits (radix select) until at most 256 candidates are left, which are ranked
//     against each other, and places its share of the outputs: latency-bound, a score row is 64 - 128 KB.
//   topk_digit_pass_kernel / topk_place_kernel: longer rows, several
//     workgroups per image, four 8-bit digit passes (radix select), one launch each.
// gather_rows_kernel: copies the kept token rows (and the global rows) with 16-byte accesses.
#include "ns_common.h"
#include <algorithm>

namespace ns {

namespace {

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;

// larger float <=> larger key; -0.0 and +0.0 map to the same key
__device__ __forceinline__ uint32_t order_key(float x) {
  const uint32_t u = __float_as_uint(x + 0.0f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Adds the digits of the wave's candidate lanes to the wave's histogram.  Clustered scores put
// most lanes of a wave into the same few bins, where one LDS atomic per lane would serialise;
// so the first bins are peeled off with one add of a lane count each, and only what is left
// (digits that are spread out, hence rarely colliding) goes through per-lane atomics.
__device__ __forceinline__ void wave_histogram_add(uint32_t *h, bool cand, uint32_t digit, int lane) {
  unsigned long long rem = __ballot(cand);
#pragma unroll 1
  for (int it = 0; it < 2 && rem; it++) {
    const int leader = __ffsll((long long)rem) - 1;
    const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)digit, leader);
    const unsigned long long same = __ballot(cand && digit == d0) & rem;
    if (lane == leader) atomicAdd(&h[d0], (uint32_t)__popcll(same));
    rem &= ~same;
  }
  if ((rem >> lane) & 1ull) atomicAdd(&h[digit], 1u);
}

// Sums inside a wave without a trip through LDS: DPP row shifts add up the 16 lanes of a row, the
// four row totals travel through scalar registers.
// Inclusive prefix sum over the lanes of a wave (lane l: x of lanes 0..l).
__device__ __forceinline__ uint32_t wave_prefix_incl(uint32_t x, int lane) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, true);   // row_shr:1
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, true);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, true);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, true);
  const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)x, 15), r1 = (uint32_t)__builtin_amdgcn_readlane((int)x, 31),
                 r2 = (uint32_t)__builtin_amdgcn_readlane((int)x, 47);
  const int row = lane >> 4;
  return x + (row > 0 ? r0 : 0u) + (row > 1 ? r1 : 0u) + (row > 2 ? r2 : 0u);
}
// Inclusive suffix sum (lane l: x of lanes l..63).
__device__ __forceinline__ uint32_t wave_suffix_incl(uint32_t x, int lane) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x101, 0xf, 0xf, true);   // row_shl:1
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x102, 0xf, 0xf, true);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x104, 0xf, 0xf, true);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x108, 0xf, 0xf, true);
  const uint32_t r1 = (uint32_t)__builtin_amdgcn_readlane((int)x, 16), r2 = (uint32_t)__builtin_amdgcn_readlane((int)x, 32),
                 r3 = (uint32_t)__builtin_amdgcn_readlane((int)x, 48);
  const int row = lane >> 4;
  return x + (row < 1 ? r1 : 0u) + (row < 2 ? r2 : 0u) + (row < 3 ? r3 : 0u);
}
// Smallest / largest of the 64 lanes, the same in every lane.
__device__ __forceinline__ uint32_t wave_max(uint32_t x) {
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x111, 0xf, 0xf, false));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x112, 0xf, 0xf, false));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x114, 0xf, 0xf, false));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x118, 0xf, 0xf, false));
  return max(max((uint32_t)__builtin_amdgcn_readlane((int)x, 15), (uint32_t)__builtin_amdgcn_readlane((int)x, 31)),
             max((uint32_t)__builtin_amdgcn_readlane((int)x, 47), (uint32_t)__builtin_amdgcn_readlane((int)x, 63)));
}
__device__ __forceinline__ uint32_t wave_min(uint32_t x) { return ~wave_max(~x); }
// Sum of x over lanes 0..15 (one DPP row), the same in every lane.
__device__ __forceinline__ uint32_t row0_total(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, true);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, true);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, true);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, true);
  return (uint32_t)__builtin_amdgcn_readlane((int)x, 15);
}

// Threads 0..255 bring the number of candidates per digit; sel[0] = the digit that holds the
// need-th largest candidate, sel[1] = how many keys of that digit are still needed.
__device__ __forceinline__ void choose_digit(uint32_t tot, uint32_t need, int tid, int wave, int lane,
                                             uint32_t *wtot, uint32_t *sel) {
  uint32_t above = 0;
  if (tid < 256) {
    const uint32_t incl = wave_suffix_incl(tot, lane);   // lanes >= lane
    if (lane == 0) wtot[wave] = incl;
    above = incl - tot;
  }
  __syncthreads();
  if (tid < 256) {
    for (int w = wave + 1; w < 4; w++) above += wtot[w];
    if (above < need && need <= above + tot) {   // exactly one digit satisfies this
      sel[0] = (uint32_t)tid;
      sel[1] = need - above;
    }
  }
  __syncthreads();
}

constexpr int kDirectMax = 256;    // candidates that are ranked against each other instead of by a further digit
constexpr int kDigitBits = 11, kDigits = 1 << kDigitBits;

// Rows of N <= 1024 * KPT scores, several workgroups per image in one launch.  Every one of them selects for itself, all
// keys of its image in registers (after the first reader they come from the L2), and places the outputs [k*c/chunks, k*(c+1)/chunks)
// of its chunk c: ranges of outputs, not of inputs, because kept tokens cluster.  The selection is a chain of barriers and
// one CU's instruction issue, which several CUs that do the same do not lengthen; the placement, which one CU took 2.4 us for at
// 16384 scores, is shared.  Two images of 16384 scores, the copy of 60 % of 2 KB rows included: 29.8 -> 24.7 us a call (one
// workgroup per image, digits of 8 bits -> this).  Copying the rows in this launch too was slower wherever the copy is
// large (8 x 16384: 63 -> 70 us): 16 waves per CU keep fewer bytes on their way than the copy kernel's 32.  Scores that are NaN have no place in the order; any bit pattern but the padding's gets a
// key, so that counts and indices stay in range whatever the scores hold.
//
// Wave w owns the 64*KPT consecutive indices from w*64*KPT; in its group i (256 indices) lane l holds the four indices
// 256*i + 4*l .. + 3.  So a wave loads 1 KB of consecutive scores per instruction, index order is (wave, group, lane,
// element), and the kept indices of a group go to consecutive output positions in lane order.
template <int KPT>
__global__ __launch_bounds__(kSelThreads) void topk_select_reg_kernel(const float *scores, int N, int k,
                                                                      const int32_t *coords_in,
                                                                      int32_t *kept,
                                                                      int32_t *coords_out) {
  static_assert(KPT % 4 == 0, "keys are held in groups of four");
  const int b = blockIdx.y, chunk = blockIdx.x, chunks = gridDim.x;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const float *sc = scores + (size_t)b * N;
  __shared__ __attribute__((aligned(16))) uint32_t hist[kDigits * 4];
  __shared__ __attribute__((aligned(16))) uint32_t cand[kDirectMax];
  __shared__ uint32_t ranks[kDirectMax];
  __shared__ uint32_t wsum[kSelWaves], sel[3], ncand, wlo[kSelWaves], whi[kSelWaves];
  __shared__ uint32_t wgt[kSelWaves], weq[kSelWaves];

  // Padding slots hold key 0, real ones at least 1.
  uint32_t key[KPT];
  const int j0 = wave * (64 * KPT) + 4 * lane;       // index of key[4*i + e]: j0 + 256*i + e
  const bool vec = (reinterpret_cast<uintptr_t>(sc) & 15) == 0;
#pragma unroll
  for (int i = 0; i < KPT / 4; i++) {
    const int j = j0 + 256 * i;
    if (vec && j + 4 <= N) {
      const f32x4 v = *reinterpret_cast<const f32x4 *>(sc + j);
#pragma unroll
      for (int e = 0; e < 4; e++) key[4 * i + e] = max(order_key(v[e]), 1u);
    } else {
#pragma unroll
      for (int e = 0; e < 4; e++) key[4 * i + e] = j + e < N ? max(order_key(sc[j + e]), 1u) : 0u;
    }
  }
  // The range of the keys: scores are softmax weights of one row, a few octaves out of the 256 that a float's
  // leading bits span, and digits counted from the smallest key tell them apart at once.
  uint32_t lo = 0xffffffffu, hi = 0u;
#pragma unroll
  for (int i = 0; i < KPT; i++) {
    lo = min(lo, key[i] - 1u);                       // (padding wraps around to the largest)
    hi = max(hi, key[i]);
  }
  lo = wave_min(lo);
  hi = wave_max(hi);
  if (lane == 0) { wlo[wave] = lo; whi[wave] = hi; }
  if (tid < 3) sel[tid] = 0;
  if (tid == 0) ncand = 0;
  if (tid < kDirectMax) { cand[tid] = 0u; ranks[tid] = 0u; }       // (a key 0 is below every real key)
  uint4 *hist4 = reinterpret_cast<uint4 *>(hist);
  hist4[tid] = make_uint4(0u, 0u, 0u, 0u);
  hist4[tid + kSelThreads] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  lo = wave_min(wlo[lane & (kSelWaves - 1)]) + 1u;
  hi = wave_max(whi[lane & (kSelWaves - 1)]);

  // k-th largest key by digits of key - lo, most significant first (radix select): a pass histograms the digit of
  // the keys in [lo, lo + span], and the digit that holds the left-th largest of them becomes the next range.  The
  // histogram is kept in four copies, digit d of copy c at word 4*d + c, and lane l adds to copy l % 4: the copies of a digit are
  // one 16-byte read, and equal scores serialise over 16 lanes and not 64.  Once the candidates are few enough (after
  // one pass, as a rule: a digit of 11 bits takes a smooth score row's 16384 keys apart to a few dozen), they are
  // ranked against each other directly.  Digits of 8 bits leave 200 to 500 of them, whose ranking took 6 us of 11.
  // (key - lo <= span holds for no key below lo: lo + span <= hi does not wrap around, the difference does.)
  // In the end `left` is the number of keys equal to tau that are kept.
  // Where no score is negative, the range ends 16 octaves below the largest one at first: a few scores next to zero would
  // spread the digits over up to 250.  If fewer than k lie in it, no digit is chosen, and what lies below is next.
  // Rows with many equal scores (the empty part of a slide) leave them all in one digit, however narrow.  Two neighbouring
  // lanes with the same key give them away; that key is tried as tau once.
  // Two rows of 16384 (digits of the whole range to the end -> this; in brackets 8-bit digits, one workgroup): one octave of
  // smooth scores 9.6 -> 9.7 us (11.3), one of them next to zero 11.1 -> 10.4 (11.3), 40 % of them equal 15.7 -> 11.2 (11.5),
  // zeros and ones 17.5 -> 11.4 (11.7), all equal 10.6 -> 6.7 (11.6); normally distributed, with signs, 11.0 -> 11.8 (9.9).
  const uint32_t least = lo;
  if (lo >= 0x7fffffffu) lo = max(lo, hi - ((16u << 23) - 1u));
  uint32_t span = hi - lo, left = (uint32_t)k;
  int shift = max(32 - kDigitBits - __clz((int)span), 0);         // (span 0: clz 32)
  uint32_t tau = lo;
  bool tried = false;
  while (span != 0u) {
#pragma unroll
    for (int i = 0; i < KPT; i++) {
      const uint32_t u = key[i] - lo;
      if (u <= span) atomicAdd(&hist[((u >> shift) << 2) + (lane & 3)], 1u);
    }
    __syncthreads();
    {
      // thread t has digits 2t and 2t + 1; of a wave's keys above, its own lanes' and then the later waves'
      const uint4 h0 = hist4[2 * tid], h1 = hist4[2 * tid + 1];
      const uint32_t n0 = (h0.x + h0.y) + (h0.z + h0.w), n1 = (h1.x + h1.y) + (h1.z + h1.w);
      const uint32_t incl = wave_suffix_incl(n0 + n1, lane);
      if (lane == 0) wsum[wave] = incl;
      __syncthreads();
      const uint32_t later = row0_total(lane > wave ? wsum[lane & (kSelWaves - 1)] : 0u);
      const uint32_t above1 = later + incl - (n0 + n1), above0 = above1 + n1;   // keys above digit 2t + 1, above digit 2t
      if (above1 < left && left <= above1 + n1) { sel[0] = 2 * tid + 1; sel[1] = left - above1; sel[2] = n1; }
      if (above0 < left && left <= above0 + n0) { sel[0] = 2 * tid; sel[1] = left - above0; sel[2] = n0; }
      __syncthreads();
    }
    const uint32_t nc = sel[2];
    if (__builtin_expect(nc == 0u, 0)) {                          // tau lies below the first range
      left -= row0_total(wsum[lane & (kSelWaves - 1)]);
      span = lo - 1u - least;
      lo = least;
    } else {
      const uint32_t before = sel[0] << shift;
      lo += before;
      left = sel[1];
      span = min(span - before, (1u << shift) - 1u);
    }
    tau = lo;
    if (__builtin_expect(span == 0u, 0)) break;
    if (__builtin_expect(nc - 1u < (uint32_t)kDirectMax, 1)) {
      // ---- the candidates into a list, in any order
#pragma unroll
      for (int i = 0; i < KPT; i++)
        if (key[i] - lo <= span) cand[min(atomicAdd(&ncand, 1u), (uint32_t)kDirectMax - 1u)] = key[i];
      __syncthreads();
      // 16, 8 or 4 threads count the candidates above one candidate (low half) and not below it (high half), each in its
      // part of the list
      const int bits = nc <= 64u ? 6 : nc <= 128u ? 7 : 8, slot = tid & ((1 << bits) - 1);
      const uint4 *cand4 = reinterpret_cast<const uint4 *>(cand);
      const uint32_t mine = cand[slot], n4 = (nc + 3u) >> 2, per = (n4 + (kSelThreads >> bits) - 1u) >> (10 - bits);
      const uint32_t c0 = (uint32_t)(wave >> (bits - 6)) * per, c1 = min(c0 + per, n4);
      uint32_t gt = 0, ge = 0;
#pragma unroll 4
      for (uint32_t c = c0; c < c1; c++) {
        const uint4 o = cand4[c];
        gt += (o.x > mine) + (o.y > mine) + (o.z > mine) + (o.w > mine);
        ge += (o.x >= mine) + (o.y >= mine) + (o.z >= mine) + (o.w >= mine);
      }
      if (ge) atomicAdd(&ranks[slot], gt | (ge << 16));
      __syncthreads();
      // tau is the candidate with fewer than `left` above it and at least `left` not below it (equal ones all say the same)
      if (tid < kDirectMax) {
        const uint32_t c = cand[tid], n = ranks[tid];
        if (c != 0u && (n & 0xffffu) < left && left <= (n >> 16)) { sel[0] = c; sel[1] = left - (n & 0xffffu); }
      }
      __syncthreads();
      tau = sel[0];
      left = sel[1];
      break;
    }
    if (!tried) {
      tried = true;
      uint32_t twice = 0;                    // a candidate that two neighbouring lanes have
#pragma unroll
      for (int i = 0; i < KPT; i += KPT / 2) {
        const uint64_t same = __ballot(key[i] - lo <= span && key[i] == (uint32_t)__builtin_amdgcn_update_dpp(0, (int)key[i], 0x111, 0xf, 0xf, false));
        if (same) twice = (uint32_t)__builtin_amdgcn_readlane((int)key[i], __builtin_ctzll(same));
      }
      if (lane == 0) wlo[wave] = twice;
      __syncthreads();
      const uint32_t t = wave_max(wlo[lane & (kSelWaves - 1)]);
      if (t != 0u) {
        uint32_t gt = 0, eq = 0;
#pragma unroll
        for (int i = 0; i < KPT; i++) {
          gt += (uint32_t)__popcll(__ballot(key[i] > t));
          eq += (uint32_t)__popcll(__ballot(key[i] == t));
        }
        if (lane == 0) { wgt[wave] = gt; weq[wave] = eq; }
        __syncthreads();
        gt = row0_total(wgt[lane & (kSelWaves - 1)]);
        eq = row0_total(weq[lane & (kSelWaves - 1)]);
        if (gt < (uint32_t)k && (uint32_t)k <= gt + eq) {
          tau = t;
          left = (uint32_t)k - gt;
          __syncthreads();                   // (wgt and weq have been read: they are written again)
          break;
        }
      }
    }
    shift = max(32 - kDigitBits - __clz((int)span), 0);
    __syncthreads();                         // (sel and this pass's histogram have been read)
    if (tid < 3) sel[tid] = 0;
    hist4[tid] = make_uint4(0u, 0u, 0u, 0u);
    hist4[tid + kSelThreads] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
  }

  // every score above tau is kept; of those equal to it, the first `need` in index order
  const uint32_t need = left;
  // keys above tau and equal to it, by group: counted on the scalar unit from the compare masks
  uint32_t group_gt[KPT / 4], group_eq[KPT / 4];
  {
    uint32_t wave_gt = 0, wave_eq = 0;
#pragma unroll
    for (int i = 0; i < KPT / 4; i++) {
      group_gt[i] = group_eq[i] = 0;
#pragma unroll
      for (int e = 0; e < 4; e++) {
        group_gt[i] += (uint32_t)__popcll(__ballot(key[4 * i + e] > tau));
        group_eq[i] += (uint32_t)__popcll(__ballot(key[4 * i + e] == tau));
      }
      wave_gt += group_gt[i];
      wave_eq += group_eq[i];
    }
    if (lane == 0) { wgt[wave] = wave_gt; weq[wave] = wave_eq; }
  }
  __syncthreads();
  const uint32_t og = lane < wave ? wgt[lane & (kSelWaves - 1)] : 0u, oe = lane < wave ? weq[lane & (kSelWaves - 1)] : 0u;
  uint32_t run_gt = row0_total(og), run_eq = row0_total(oe);   // in the waves before this one (wave < 16 lanes of row 0)
  // this workgroup's outputs
  const uint32_t p0 = (uint32_t)((unsigned long long)k * chunk / chunks), p1 = (uint32_t)((unsigned long long)k * (chunk + 1) / chunks);
  asm volatile("" : "+v"(tau));   // (compare again below: kept from the counts, the masks of all groups would spill)
  int32_t *kb = kept + (size_t)b * k;
#pragma unroll
  for (int i = 0; i < KPT / 4; i++) {
    const uint32_t first = run_gt + min(run_eq, need);
    const uint32_t last = run_gt + group_gt[i] + min(run_eq + group_eq[i], need);
    if (first < p1 && last > p0) {                               // (uniform in the wave)
      uint32_t c = 0;
#pragma unroll
      for (int e = 0; e < 4; e++) c += (uint32_t)(key[4 * i + e] > tau) + ((uint32_t)(key[4 * i + e] == tau) << 16);
      const uint32_t incl = wave_prefix_incl(c, lane);           // at most 256 per half
      uint32_t ngt = run_gt + ((incl - c) & 0xffffu), neq = run_eq + ((incl - c) >> 16);
      int32_t xy[4] = {0, 0, 0, 0};
      if (coords_in)
#pragma unroll
        for (int e = 0; e < 4; e++) xy[e] = coords_in[(size_t)b * N + min(j0 + 256 * i + e, N - 1)];
#pragma unroll
      for (int e = 0; e < 4; e++) {
        const bool gt = key[4 * i + e] > tau, eq = key[4 * i + e] == tau;
        const uint32_t pos = ngt + min(neq, need);
        if ((gt || (eq && neq < need)) && pos >= p0 && pos < p1) {
          const int j = j0 + 256 * i + e;
          kb[pos] = j;
          if (coords_in) coords_out[(size_t)b * k + pos] = xy[e];
        }
        ngt += gt;
        neq += eq;
      }
    }
    run_gt += group_gt[i];
    run_eq += group_eq[i];
  }
}

// ---- several workgroups per image (score rows too long for one CU to select from quickly)
//
// Four digit passes of 8 bits over the order-preserving keys, most significant first, and a
// placement pass, each one launch over (chunks, images).  A pass histograms the digit of the keys
// that match the prefix chosen so far, per chunk, into `part`; the next launch begins by adding the
// chunks' histograms (every workgroup does so for itself: a few hundred loads) and choosing the
// digit that holds the k-th largest key.  No atomics on global memory, no waiting between
// workgroups: the launches order the passes.
struct SelState { uint32_t prefix, need; };

// The state after digit `upto` (0..3) has been chosen, from the state before and that digit's
// histograms; workgroup 0 of the image records it for the next launch.  The histograms were
// written by other workgroups (other L2s): every load is a long trip, so all threads take part
// (thread t: digit t % 256, every fourth chunk) and keep eight loads in flight.
// quarter[4..7], if asked for (before >= 0): the same sums over the chunks below `before` only.
__device__ __forceinline__ SelState advance_state(int upto, int b, int B, int k, int nchunk, const uint32_t *part,
                                                  SelState *state, bool record, int before, int tid, int wave,
                                                  int lane, uint32_t *wtot, uint32_t *sel, uint32_t (*quarter)[256]) {
  SelState st = {0u, (uint32_t)k};
  if (upto > 0) st = state[(size_t)(upto - 1) * B + b];
  {
    const uint32_t *h = part + ((size_t)upto * B + b) * (size_t)nchunk * 256 + (tid & 255);
    uint32_t acc = 0, acc_before = 0;
#pragma unroll 8
    for (int c = tid >> 8; c < nchunk; c += 4) {
      const uint32_t n = h[(size_t)c * 256];
      acc += n;
      acc_before += c < before ? n : 0u;
    }
    quarter[tid >> 8][tid & 255] = acc;
    if (before >= 0) quarter[4 + (tid >> 8)][tid & 255] = acc_before;
  }
  __syncthreads();
  const uint32_t tot = tid < 256 ? quarter[0][tid] + quarter[1][tid] + quarter[2][tid] + quarter[3][tid] : 0u;
  choose_digit(tot, st.need, tid, wave, lane, wtot, sel);
  st.prefix |= sel[0] << (24 - 8 * upto);
  st.need = sel[1];
  if (record && tid == 0) state[(size_t)upto * B + b] = st;
  return st;
}

// grid (nchunk, B): digit `pass` (0 = bits 31..24) of the keys of chunk blockIdx.x.  The last pass
// also counts the chunk's keys above the 24-bit prefix (they are kept whatever the last digit is).
__global__ __launch_bounds__(kSelThreads) void topk_digit_pass_kernel(const float *scores, int N, int k, int pass,
                                                                     int kpt, uint32_t *part, SelState *state,
                                                                     uint32_t *above) {
  const int b = blockIdx.y, B = gridDim.y, c = blockIdx.x, nchunk = gridDim.x;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const float *sc = scores + (size_t)b * N;
  __shared__ uint32_t hist[kSelWaves][256];
  __shared__ uint32_t wtot[4], sel[2], wabove[kSelWaves];
  SelState st = {0u, (uint32_t)k};
  if (pass > 0)     // (the first rows of hist serve as its exchange buffer)
    st = advance_state(pass - 1, b, B, k, nchunk, part, state, c == 0, -1, tid, wave, lane, wtot, sel, hist);
  for (int i = tid; i < kSelWaves * 256; i += kSelThreads) (&hist[0][0])[i] = 0;
  __syncthreads();
  const uint32_t mask = pass ? 0xffffffffu << (32 - 8 * pass) : 0u;
  const int shift = 24 - 8 * pass;
  const int base = c * kpt * kSelThreads;
  uint32_t nabove = 0;     // wave-uniform
  for (int i = 0; i < kpt; i++) {
    const int j = base + i * kSelThreads + tid;
    bool cand = false, over = false;
    uint32_t digit = 0;
    if (j < N) {
      const uint32_t key = order_key(sc[j]);
      cand = (key & mask) == st.prefix;
      over = (key & mask) > st.prefix;
      digit = (key >> shift) & 255u;
    }
    wave_histogram_add(hist[wave], cand, digit, lane);
    if (pass == 3) nabove += (uint32_t)__popcll(__ballot(over));
  }
  if (pass == 3 && lane == 0) wabove[wave] = nabove;
  __syncthreads();
  if (tid < 256) {
    uint32_t tot = 0;
#pragma unroll
    for (int w = 0; w < kSelWaves; w++) tot += hist[w][tid];
    part[(((size_t)pass * B + b) * nchunk + c) * 256 + tid] = tot;
  }
  if (pass == 3 && tid == 0) {
    uint32_t t = 0;
    for (int w = 0; w < kSelWaves; w++) t += wabove[w];
    above[(size_t)b * nchunk + c] = t;
  }
}

// grid (nchunk, B): the kept keys of chunk blockIdx.x go to their places (ascending index order;
// of the keys equal to the k-th largest, the first `need` in index order are kept).  What the
// chunks before this one keep comes from their histograms of the last digit and their counts of
// keys above the prefix: no key of another chunk is read.
__global__ __launch_bounds__(kSelThreads) void topk_place_kernel(const float *scores, int N, int k, int kpt,
                                                                const uint32_t *part, SelState *state,
                                                                const uint32_t *above, const int32_t *coords_in,
                                                                int32_t *kept, int32_t *coords_out) {
  const int b = blockIdx.y, B = gridDim.y, c = blockIdx.x, nchunk = gridDim.x;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const float *sc = scores + (size_t)b * N;
  __shared__ uint32_t quarter[8][256];
  __shared__ uint32_t wtot[4], sel[2];
  __shared__ uint32_t wgt[kSelWaves], weq[kSelWaves];
  const uint32_t above_mine = tid < c ? above[(size_t)b * nchunk + tid] : 0u;     // at most 128 chunks
  const SelState st = advance_state(3, b, B, k, nchunk, part, state, false, c, tid, wave, lane, wtot, sel, quarter);
  const uint32_t tau = st.prefix, need = st.need, digit = tau & 255u;
  uint32_t cgt = above_mine, ceq = 0;
  if (tid < 256) {
    const uint32_t n = quarter[4][tid] + quarter[5][tid] + quarter[6][tid] + quarter[7][tid];
    cgt += (uint32_t)tid > digit ? n : 0u;
    ceq = (uint32_t)tid == digit ? n : 0u;
  }
  if (wave < 4) {
#pragma unroll
    for (int sft = 1; sft < 64; sft <<= 1) {
      cgt += (uint32_t)__shfl_xor((int)cgt, sft);
      ceq += (uint32_t)__shfl_xor((int)ceq, sft);
    }
    if (lane == 0) { wgt[wave] = cgt; weq[wave] = ceq; }
  }
  __syncthreads();
  uint32_t gt_before = wgt[0] + wgt[1] + wgt[2] + wgt[3], eq_before = weq[0] + weq[1] + weq[2] + weq[3];
  __syncthreads();
  const int base = c * kpt * kSelThreads;
  int32_t *kb = kept + (size_t)b * k;
  const unsigned long long lt = (1ull << lane) - 1ull;
  for (int i = 0; i < kpt; i++) {          // index order inside the chunk: (i, wave, lane)
    const int j = base + i * kSelThreads + tid;
    const uint32_t key = j < N ? order_key(sc[j]) : 0u;
    const bool gt = j < N && key > tau, eq = j < N && key == tau;
    const unsigned long long bgt = __ballot(gt), beq = __ballot(eq);
    if (lane == 0) { wgt[wave] = (uint32_t)__popcll(bgt); weq[wave] = (uint32_t)__popcll(beq); }
    __syncthreads();
    uint32_t my_gt = gt_before + (uint32_t)__popcll(bgt & lt), my_eq = eq_before + (uint32_t)__popcll(beq & lt);
    uint32_t all_gt = 0, all_eq = 0;
#pragma unroll
    for (int w = 0; w < kSelWaves; w++) {
      my_gt += w < wave ? wgt[w] : 0u;
      my_eq += w < wave ? weq[w] : 0u;
      all_gt += wgt[w];
      all_eq += weq[w];
    }
    if (gt || (eq && my_eq < need)) {
      const uint32_t pos = my_gt + min(my_eq, need);
      if (pos < (uint32_t)k) {   // always, when the scores hold no NaN
        kb[pos] = j;
        if (coords_in) coords_out[(size_t)b * k + pos] = coords_in[(size_t)b * N + j];
      }
    }
    gt_before += all_gt;
    eq_before += all_eq;
    __syncthreads();
  }
}

// grid (ceil((G+k)/4), B), 256 threads: one wave per output row; the G global rows come first.
__global__ __launch_bounds__(256) void gather_rows_kernel(const uint4 *x, const int32_t *kept,
                                                          uint4 *y, int N, int k, int G, int vec_per_row) {
  const int b = blockIdx.y;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= G + k) return;
  const int src = row < G ? row : G + kept[(size_t)b * k + row - G];
  const uint4 *xs = x + ((size_t)b * (G + N) + src) * vec_per_row;
  uint4 *yd = y + ((size_t)b * (G + k) + row) * vec_per_row;
  // (streamed once: non-temporal accesses leave the caches to the kernels around this one)
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 *src4 = reinterpret_cast<const u32x4 *>(xs);
  u32x4 *dst4 = reinterpret_cast<u32x4 *>(yd);
  for (int i = lane; i < vec_per_row; i += 64) __builtin_nontemporal_store(__builtin_nontemporal_load(src4 + i), dst4 + i);
}

}  // namespace

// Keys per thread of the several-workgroup selection: at most 128 chunks per image.
static int multi_kpt(int N) { return (int)(((long long)N + 128LL * kSelThreads - 1) / (128LL * kSelThreads)); }
static int multi_chunks(int N) { return (N + multi_kpt(N) * kSelThreads - 1) / (multi_kpt(N) * kSelThreads); }

// Keys per thread of the one-workgroup selection at most.  (With 64 keys a row of 65536 scores takes one
// compute unit 43 us; the five launches of the several-workgroup selection take 26 us plus their gaps.)
constexpr int kRegMaxKeys = 32;

size_t topk_select_workspace_bytes(int B, int N) {
  if (N <= kRegMaxKeys * kSelThreads) return 0;                    // one launch, state in registers and LDS
  return (size_t)4 * B * multi_chunks(N) * 256 * sizeof(uint32_t) + (size_t)4 * B * sizeof(SelState) +
         (size_t)B * multi_chunks(N) * sizeof(uint32_t);
}

ns_status launch_topk_select(int B, int N, int k, const float *scores, const int32_t *coords_in,
                             int32_t *kept, int32_t *coords_out, void *ws, hipStream_t s) {
  if (N <= kRegMaxKeys * kSelThreads) {
    // up to 16 workgroups per image, as long as every one has a CU, for at least 64 outputs each; one where an output lies
    // over the scores, which are then all read before the first index is written
    auto over_scores = [&](const int32_t *out) {
      const uintptr_t o = reinterpret_cast<uintptr_t>(out), i = reinterpret_cast<uintptr_t>(scores);
      return out && o < i + (size_t)4 * B * N && i < o + (size_t)4 * B * k;
    };
    const bool apart = !over_scores(kept) && !over_scores(coords_out);
    const dim3 grid(apart ? std::max(1, std::min({16, device_cu_count() / B, k / 64})) : 1, B), block(kSelThreads);
    const auto kern = N <= 4 * kSelThreads    ? topk_select_reg_kernel<4>
                      : N <= 8 * kSelThreads  ? topk_select_reg_kernel<8>
                      : N <= 16 * kSelThreads ? topk_select_reg_kernel<16>
                                              : topk_select_reg_kernel<32>;
    hipLaunchKernelGGL(kern, grid, block, 0, s, scores, N, k, coords_in, kept, coords_out);
    return check_launch("topk_select_reg_kernel");
  }
  const int kpt = multi_kpt(N), nchunk = multi_chunks(N);
  uint32_t *part = static_cast<uint32_t *>(ws);
  SelState *state = reinterpret_cast<SelState *>(part + (size_t)4 * B * nchunk * 256);
  uint32_t *above = reinterpret_cast<uint32_t *>(state + (size_t)4 * B);
  for (int pass = 0; pass < 4; pass++)
    hipLaunchKernelGGL(topk_digit_pass_kernel, dim3(nchunk, B), dim3(kSelThreads), 0, s, scores, N, k, pass, kpt,
                       part, state, above);
  hipLaunchKernelGGL(topk_place_kernel, dim3(nchunk, B), dim3(kSelThreads), 0, s, scores, N, k, kpt, part, state,
                     above, coords_in, kept, coords_out);
  return check_launch("topk_place_kernel");
}

ns_status launch_gather_rows(int B, int N, int k, int G, size_t row_bytes, const void *x,
                             const int32_t *kept, void *y, hipStream_t s) {
  dim3 grid((G + k + 3) / 4, B);
  hipLaunchKernelGGL(gather_rows_kernel, grid, dim3(256), 0, s, static_cast<const uint4 *>(x), kept,
                     static_cast<uint4 *>(y), N, k, G, (int)(row_bytes / 16));
  return check_launch("gather_rows_kernel");
}

}  // namespace ns
