// Top-K attention over a whole sequence (paper Sec. 2.1: computing the full weights of a query and keeping the
// highest is the ideal sparsity; Sec. 2.2, first strategy, and App. "Implementation Details": the backbone is
// fine-tuned with attention whose weights outside the top K are masked out).  Causal, per (sequence, head):
//
//   w[i][j] = q_i . k_j  (j <= i);   kept(i) = the top_k largest w[i][.], equal weights to the lower j
//   out_i   = sum_{j in kept(i)} softmax_j(w[i][j] / sqrt(d)) v_j
//
// A query's K-th largest weight needs all its weights, but not all of them at once.  A workgroup takes NQ = 32 or 64
// consecutive queries of one (sequence, head) and goes over the keys they can see several times; every time the weights are
// made anew on the matrix cores (32x32x16 bf16), which is cheaper than keeping them (64 queries x 8192 keys are 2 MB):
//
//   1 range     mean and deviation of the weights over an evenly spaced sample of the keys give a range in which the K-th
//               largest is expected.
//   2 count     a histogram per query in LDS over that range (256 bins, two to a word, [word][query]: every query has a bank of its
//               own); the bin that holds the K-th largest weight and its rank in it.  Counted again for the queries whose K-th largest
//               is outside the range, or in a bin with more than 16 weights that do not all stay: up to twice over another range,
//               then over bins that are equal in the order-preserving integer images of the weights, between the two weights it is
//               known to lie between (8 of at most 32 bits a count; at once where the bin stands alone, as one of equal weights
//               does).  So a workgroup counts at most 3 + 4 times whatever the weights' sizes and distribution, and the result
//               never depends on the sample, only the time does.
//   3 ties      only where more than 16 weights are equal to the K-th largest: one pass in which the last position that stays is
//               found from the bit masks of each step.
//   4 product   P = exp2((w - max) / sqrt(d) . log2 e) of the weights above the bin (the same instructions on the same
//               operands give the weights the very bits they had in 2), as two bf16 terms, and O^T += V^T . P^T.  The second term
//               is rounded to nearest, so that the two are within 2^-16 of P and as often above it as below, at the cost of cutting
//               it off (which leaves up to 2^-15, always below): of 8 rows of 1024 tokens at d = 128 (1 M outputs, 96 kept of Gaussian
//               weights) 4295 are not the exact result's rounding, with the term cut off 6395, with the weights of every K-th largest's
//               bin in fp32 besides 6390.  (Both terms rounded: 2295, but 64 rows of 1000 at d = 64 take 1 to 4 % longer.)
//               A lane's weights sit where the second product wants its operand; V comes out of LDS transposed (ds_read_b64_tr_b16).  The few weights inside the bin are set aside with their positions, unless the whole
//               bin stays: then they are above it like the others.  Setting one aside is a detour of the wave's other 63 lanes: with
//               128 bins, and bins that stay whole set aside as well, 3.2 weights a query made that a fifth of 512 rows of 1024 tokens;
//               now it is one (660 -> 610 us; 8192 tokens 5690 -> 5520, 40 rows of 1000 tokens at d = 64 55.1 -> 48.8).
//   5 the rest  the weights set aside are ranked directly (equal ones by position), those that stay add their rows of V in fp32;
//               the waves' partial sums are added through LDS in a fixed order, rounded once.
//
// A wave holds 32 queries and takes one 32-key block of each step of KB blocks (wave = key block x query block), so a step's K
// (and V) rows are read once from the L2 per workgroup, coalesced, and each LDS operand serves 32 queries.  The products of
// a step run next to the arithmetic on the weights of the step before.  64 queries go with KB = 2, four waves and 79 KB of LDS, so
// that two workgroups share a compute unit: one works where the other waits at a barrier, for its first tiles, or for the bins and the
// rows of V of the weights set aside (a third of the time at 1024 tokens).  One workgroup of eight waves and KB = 4 per unit took 850
// us for 512 rows of 1024 tokens and 6670 us for 128 rows of 8192.
//
// Measured (us per call, K = 96): 512 rows of 1024 tokens, d = 128: 1900 -> 610; 128 rows of 8192 tokens, d = 128:
// 80900 -> 5520; 4 rows of 128 tokens, d = 64: 21.3 -> 10.5.  At first, 16 queries per workgroup kept their fp32 weights in LDS (in
// memory beyond 2048 tokens, read again by every pass of a radix select), with K and a transposed copy of V loaded straight
// into the operand layout: 16 look-ups in the L1 per 256 bytes, K and V read from the L2 once per 16 queries.
// Those are Gaussian weights, which mostly need one count.  256 rows of 1024 tokens (128 bins a word each / now): Gaussian 339 / 312, 60 %
// of the keys zeroed 456 / 433, whole-numbered q and k 592 / 598 (ranges alone would take 17 counts to close in on a zero), all keys equal 560 /
// 541.  Two bins a word cost a count over a range one operation a weight (21.4 -> 22.4 thousand cycles a workgroup, the one per cent of the
// whole numbers).  What gave the equal keys their time back (593 before): counts over images number their bins from below (30.6 -> 28.8
// thousand cycles), the pass of the ties has its next tile on the way (21.6 -> 20.7), and in the product one end of the bin tells which of
// the equal weights stay wherever a block of keys is all before the last of them or all behind it (40.8 -> 31.1; each weight's position was
// compared at every step).  Keys that wander from position to position (a random walk), 16 rows of 4096: 268 / 275, 256 of 1024: 362 / 332.
// What bounds it now, at 8192 tokens (counters): a SIMD issues vector instructions in 51 % of its cycles and has matrix work in 33 %, which
// two waves a SIMD (what 253 registers leave room for) hardly overlap; a wave waits for LDS or a barrier in 22 %.  LDS is busy in 34 %.  A
// quarter fewer vector instructions a step gave 1 %.  The wave in a step's products goes first (s_setprio): 609 -> 598 us at 1024 tokens, 451 ->
// 429 for 64 rows of 3000; not at d = 64 nor with 32 queries, where it makes no difference or costs 1 %.
// Tried and not kept: thresholds from a sample and candidate lists in LDS instead of histograms (6.5 vector instructions per
// weight and a selection of 20000 cycles per workgroup; 1080 us / 8800 us); a pass of its own for the weights of the bin (965 us /
// 7700 us); the K operand of the next step fetched a step ahead (132 registers too many); the bins' ends searched for in every
// workgroup, so that the product compares instead of multiplying (the same, 10.6 -> 11.0 us for the smallest); the product's loop
// unrolled by two like the counts' (78 registers spilled); 128 queries and eight waves a workgroup, one per unit, which reads K and V half
// as often (759 us / 5730 us); all sixteen weights of a step looked at ahead of its products, for one detour a step (661 us / 5900 us); a
// narrower range, 0.75 of the deviation (598 us / 5500 us, but where 60 % of the keys are zero its counts miss: 491 for 455).
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "adore.h"
#include "device_utils.h"

namespace adore {

namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kRows = 128;           // a histogram's words: two bins each, the even one's and the odd one's weights together in the lower
constexpr int kBins = 2 * kRows;     // half, the odd one's in the upper (at most 32768 keys).  Bin 0: below the range, the last one: above it
constexpr int kFew = 16;             // weights of a bin that are ranked directly
constexpr int kSample = 128;         // keys of the sample: mean and deviation to a tenth of the deviation, for a range of two
// A weight's bin is read off the bits of y = a w + b: with bin 0 at kBin0 = 2^23, where floats are the integers, and as many units a
// bin as half a row of the histogram has bytes, the bits of y hold the row's place (one multiply-add, a clamp and an and-or, no conversion).
constexpr float kBin0 = 8388608.f;
constexpr int kRangeCounts = 3;      // most counts over ranges of weights; then at most ceil(32 / 8) over images

// Order-preserving image of a weight (larger float <=> larger integer, never 0 for a number) and back.
__device__ inline uint32_t weight_image(float x) {
  const uint32_t b = __float_as_uint(x);
  return b ^ (uint32_t(int32_t(b) >> 31) | 0x80000000u);
}
__device__ inline float image_weight(uint32_t u) { return __uint_as_float(u & 0x80000000u ? u ^ 0x80000000u : ~u); }

// z with P(N(0,1) > z) = p, to about 3e-3 (Abramowitz and Stegun, Handbook of Mathematical Functions, 26.2.22)
__device__ inline float normal_quantile(float p) {
  const float q = fminf(p, 1.f - p);
  const float t = __builtin_amdgcn_sqrtf(-1.3862944f * __builtin_amdgcn_logf(fmaxf(q, 1e-7f)));   // sqrt(-2 ln q); logf is base 2
  const float z = t - (2.30753f + 0.27061f * t) * __builtin_amdgcn_rcpf(1.f + t * (0.99229f + 0.04481f * t));
  return p <= 0.5f ? z : -z;
}

// Bits of the lanes whose x is at least y (none where one is NaN).
__device__ __forceinline__ uint64_t lanes_ge(float x, float y) { return __builtin_amdgcn_fcmpf(x, y, 3); }   // 3: ordered, >=
// ... whose x is in [0, y) for a y whose bits are `end`.
__device__ __forceinline__ uint64_t lanes_below(float x, uint32_t end) {
  return __builtin_amdgcn_uicmp(__float_as_uint(x), end, 36);   // 36: unsigned, <
}

// Both rounded to bf16 (to nearest, ties to even), a in the lower half.
__device__ __forceinline__ uint32_t two_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

constexpr uint32_t kLowest = 0x007fffffu, kHighest = 0xff800000u;   // images of the infinities
// Right shift after which the distances 0 .. span fit the bins.
__device__ inline int image_shift(uint32_t span) { return max(0, 24 - __clz(int(span))); }

struct TopkArgs {
  const bf16_t *Q, *K, *V;   // [rows][S][d]
  bf16_t *O;
  int S, rows, topk;
  float scale_log2;          // log2(e) / sqrt(d)
};

// Shared memory: two K tiles (one in use, one being written), then the histograms or two V tiles; the merge buffer overlays all of
// it.  The weights set aside and the small arrays sit behind.
template <int DH, int NQB, int KB>
struct TopkLds {
  static constexpr int NQ = 32 * NQB;
  static constexpr int kTile = 32 * KB * DH * 2;
  static constexpr int kHist = NQ * kRows * 4;
  static constexpr int kBig = 2 * kTile + (kHist > 2 * kTile ? kHist : 2 * kTile);
  static constexpr int kMerge = KB * NQB * (DH / 32) * 16 * 64 * 4;
  static constexpr int kFewAt = kBig > kMerge ? kBig : kMerge;
  static constexpr int kMisc = kFewAt + NQ * kFew * 8;
  static constexpr int kBytes = kMisc + NQ * (16 + 3 * KB) * 4 + 32;
};

template <int DH, int NQB, int KB>
__global__ __launch_bounds__(64 * NQB * KB, NQB) void topk_attend_kernel(const TopkArgs a) {
  using Lds = TopkLds<DH, NQB, KB>;
  constexpr int NT = 64 * NQB * KB, NQ = 32 * NQB;
  constexpr int kStep = 32 * KB;               // keys per step
  constexpr int TPQ = NT / NQ, RPT = kRows / TPQ;   // threads per query and rows per thread where the histograms are read
  constexpr int CPR = DH / 8;                  // 16-byte chunks per row
  constexpr int NLD = kStep * CPR / NT;        // chunks of a tile per thread
  constexpr int KT = DH / 16, DB = DH / 32;
  constexpr bool kFirst = DH == 128 && NQB == 2;   // a wave in its products issues before the other one of its SIMD
  constexpr uint32_t kRow = NQ * 4;            // bytes of a histogram's row
  constexpr float kBinWidth = float(kRow / 2);
  extern __shared__ __align__(16) unsigned char smem[];
  uint32_t *s_hist = reinterpret_cast<uint32_t *>(smem + 2 * Lds::kTile);   // [kRows][NQ]
  float2 *s_few = reinterpret_cast<float2 *>(smem + Lds::kFewAt);       // [NQ][kFew] weight, bits of its position, of the weights set aside
  float *s_a = reinterpret_cast<float *>(smem + Lds::kMisc);   // [NQ] bin of w = a w + b, while its range is counted (else 0)
  float *s_b = s_a + NQ;
  float *s_lo = s_b + NQ;                                      // [NQ] the range
  float *s_hi = s_lo + NQ;
  float *s_ga = s_hi + NQ;                                     // [NQ] a, b and the bin that holds the K-th largest weight; where images
  float *s_gb = s_ga + NQ;                                     // were counted (s_flag[3]) its lower end and the weight above it
  float *s_bin = s_gb + NQ;
  uint32_t *s_first = reinterpret_cast<uint32_t *>(s_bin + NQ);   // [NQ] images between which it is known to be; both 0 once it is found
  uint32_t *s_last = s_first + NQ;
  uint32_t *s_over = s_last + NQ;                              // [NQ] weights above s_last
  uint32_t *s_min = s_over + NQ;                               // [NQ] smallest and largest image among the weights just counted
  uint32_t *s_most = s_min + NQ;
  int *s_need = reinterpret_cast<int *>(s_most + NQ);          // [NQ] its rank in that bin: how many of its weights stay
  int *s_tie = s_need + NQ;                                    // [NQ] crowded bin (-2 until it is known): its weights, all equal, stay up to this position
  uint32_t *s_max = reinterpret_cast<uint32_t *>(s_tie + NQ);  // [NQ] image of the largest weight
  int *s_n = reinterpret_cast<int *>(s_max + NQ);              // [NQ] weights set aside
  float *s_l = reinterpret_cast<float *>(s_n + NQ);            // [KB][NQ]
  uint32_t *s_part = reinterpret_cast<uint32_t *>(s_l + KB * NQ);   // [2 KB][NQ]
  int *s_flag = reinterpret_cast<int *>(s_part + 2 * KB * NQ);      // [0] count images again, [1] a crowded bin of equal weights, [2] count ranges again, [3] some queries need images counted, [4] huge weights

  // Workgroup -> (row, query block): all blocks of a row on one XCD (consecutive workgroups go to the 8 XCDs in turn), so
  // that its K and V come from memory once; within a row the blocks with the most keys first.  Rows that do not make up a
  // group of eight go to all XCDs and come first, the longest blocks of all of them before the next: a launch ends with
  // short blocks (behind the others before: 10 rows of 6152 tokens, d = 64, 294 -> 215 us; 12 of 2048, d = 128, 105 -> 83; 61 of
  // 2048, 290 -> 264).
  const int nq = (a.S + NQ - 1) / NQ;
  const int odd = a.rows & 7, L = int(blockIdx.x) - odd * nq;
  int row_, qi;
  if (L < 0) {
    qi = int(blockIdx.x) / odd;
    row_ = (a.rows & ~7) + int(blockIdx.x) - qi * odd;
  } else {
    const int slot = L >> 3;
    row_ = slot / nq * 8 + (L & 7);
    qi = slot - slot / nq * nq;
  }
  const int q0 = (nq - 1 - qi) * NQ;
  const int nkeys = min(a.S, q0 + NQ);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qg = wave % NQB, kg = wave / NQB;
  const int c = lane & 31, h = lane >> 5;
  const int ql = qg * 32 + c;                  // the lane's query within the workgroup
  const int qpos = q0 + ql;
  const int qfirst = q0 + qg * 32;
  const size_t base = size_t(row_) * a.S * DH;
  const bf16_t *Kb = a.K + base, *Vb = a.V + base;

  // 16-byte chunk `ch` of tile row r, permuted so that neither 8 rows x 1 chunk (the K operand) nor 4 rows x 2 neighbouring
  // chunks (V, transposed) meet in a bank
  auto chunk_at = [](int r, int ch) { 
    const int x = (r & 3) << 1 | ((r >> 2) & 1);
    return DH == 128 ? r * 256 + ((ch ^ (x | (r & 8))) << 4) : r * 128 + ((ch ^ x) << 4);
  };
  const int ld_row = tid / CPR;
  const uint32_t ld_col = uint32_t(tid % CPR) * 16u;
  // Keys beyond the last one read the last one; only a step that has some works out an address per row.
  const uint32_t ld_at = uint32_t(ld_row) * (DH * 2) + ld_col;
  auto load_tile = [&](const bf16_t *src, int step, u32x4 (&r)[NLD]) {
    auto at = (const __attribute__((address_space(1))) char *)src + size_t(step) * (kStep * DH * 2);
    asm("" : "+s"(at));   // a scalar base and one offset per thread, not an address per thread and row kept from step to step
    if ((step + 1) * kStep <= a.S) {
#pragma unroll
      for (int i = 0; i < NLD; ++i) r[i] = *(const __attribute__((address_space(1))) u32x4 *)(at + i * (NT / CPR * DH * 2) + ld_at);
    } else {
      const int last = a.S - 1 - step * kStep;
#pragma unroll
      for (int i = 0; i < NLD; ++i)
        r[i] = *(const __attribute__((address_space(1))) u32x4 *)(at + (uint32_t(min(ld_row + i * (NT / CPR), last)) * (DH * 2) + ld_col));
    }
  };
  auto load_sample = [&](int step, uint32_t stride_fp, u32x4 (&r)[NLD]) {   // key = (index * stride_fp) >> 12
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const uint32_t key = (uint32_t(step * kStep + ld_row + i * (NT / CPR)) * stride_fp) >> 12;
      r[i] = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(Kb) + (key * (DH * 2) + ld_col));
    }
  };
  auto store_tile = [&](int dst, const u32x4 (&r)[NLD]) {   // dst: where the tile starts in shared memory
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      *reinterpret_cast<u32x4 *>(smem + dst + chunk_at(ld_row + i * (NT / CPR), tid % CPR)) = r[i];
    }
  };
  // The query operand, through LDS like the keys: straight from memory its 16-byte pieces of 32 rows cost the L1 a look-up per
  // lane (4096 of them per workgroup, 3 us before the first product).
  if (tid < 5) s_flag[tid] = 0;
  bf16x8 qf[KT];
  {
    constexpr int NQL = NQ * CPR / NT;
    u32x4 r[NQL];
#pragma unroll
    for (int i = 0; i < NQL; ++i)
      r[i] = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(a.Q + base) +
                                              (uint32_t(min(q0 + ld_row + i * (NT / CPR), a.S - 1)) * (DH * 2) + ld_col));
#pragma unroll
    for (int i = 0; i < NQL; ++i) *reinterpret_cast<u32x4 *>(smem + chunk_at(ld_row + i * (NT / CPR), tid % CPR)) = r[i];
    __syncthreads();
#pragma unroll
    for (int t = 0; t < KT; ++t) qf[t] = *reinterpret_cast<const bf16x8 *>(smem + chunk_at(ql, 2 * t + h));
  }
  // Weights of the lane's query against its wave's 32 keys of the K tile at `tile`: [i] is key kg * 32 + 8 (i / 4) + 4 h + i % 4.
  // meanwhile(g), g = 0 .. 3: other work, a share of it behind every two matrix instructions, in that order (a wave issues in
  // order: left to itself the compiler puts all of one kind first, and matrix and vector units take turns).
  auto weights = [&](int tile, auto &&meanwhile) {
    bf16x8 kv[KT];
#pragma unroll
    for (int t = 0; t < KT; ++t) kv[t] = *reinterpret_cast<const bf16x8 *>(smem + tile + chunk_at(kg * 32 + c, 2 * t + h));
    __builtin_amdgcn_sched_barrier(0);   // all reads on their way before the first product waits for one
    f32x16 s = {0.f};
#pragma unroll
    for (int g = 0; g < 4; ++g) {
#pragma unroll
      for (int t = g * (KT / 4); t < (g + 1) * (KT / 4); ++t) {
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kv[t], qf[t], s, 0, 0, 0);
        asm volatile("" : "+v"(s));    // issued here, not where the result is first needed
      }
      meanwhile(g);
      __builtin_amdgcn_sched_barrier(0);
    }
    return s;
  };
  auto nothing = [](int) {};
  // keys from kb on that the query cannot see become NaN, which no comparison lets through
  auto hide = [&](f32x16 &s, int kb) {
    const int seen = qpos - 4 * h - kb;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      constexpr int kGreater = 38;               // signed
      const uint64_t hidden = __builtin_amdgcn_sicmp(8 * (i >> 2) + (i & 3), seen, kGreater);
      s[i] = __builtin_amdgcn_inverse_ballot_w64(hidden) ? __builtin_nanf("") : s[i];
    }
  };

  // ---- one pass over the keys (SAMPLE: over a sample of those before q0, which all queries see): consume(w0, .. w3, g, first
  // key) takes the weights of keys 8 g + 4 h .. + 3 of the wave's block ----
  auto sweep = [&](auto sample_, int steps, uint32_t stride_fp, auto &&consume) {
    constexpr bool SAMPLE = decltype(sample_)::value;
    u32x4 kr[NLD];
    auto load = [&](int st) {
      if constexpr (SAMPLE)
        load_sample(st, stride_fp, kr);
      else
        load_tile(Kb, st, kr);
    };
    load(0);
    __syncthreads();                   // the tiles of the pass before are done with
    store_tile(0, kr);
    if (steps > 1) load(1);
    __syncthreads();
    if (steps > 1) store_tile(Lds::kTile, kr);
    if (steps > 2) load(2);
    f32x16 s = weights(0, nothing);
    int kb = kg * 32;
    if (!SAMPLE && kb + 31 > qfirst) hide(s, kb);
    // tile 0 or 1: the one of step st, known when compiled, so that the tiles' places in LDS are too and the weights change hands
    // without moves
    auto one = [&](auto tile_, int st, const f32x16 &w, f32x16 &next) {
      constexpr int kThis = decltype(tile_)::value * Lds::kTile, kOther = Lds::kTile - kThis;
      __syncthreads();                 // tile st is there, and nobody reads tile st - 1 any more
      if (st + 1 < steps) store_tile(kOther, kr);
      if (st + 2 < steps) load(st + 2);
      if constexpr (kFirst) __builtin_amdgcn_s_setprio(1);
      next = weights(kThis, [&](int g) { consume(w[4 * g], w[4 * g + 1], w[4 * g + 2], w[4 * g + 3], g, kb); });
      if constexpr (kFirst) __builtin_amdgcn_s_setprio(0);
      kb += kStep;
      if (!SAMPLE && kb + 31 > qfirst) hide(next, kb);
    };
    int st = 1;
    for (; st + 1 < steps; st += 2) {
      f32x16 t;
      one(std::integral_constant<int, 1>(), st, s, t);
      one(std::integral_constant<int, 0>(), st + 1, t, s);
    }
    if (st < steps) {
      f32x16 t;
      one(std::integral_constant<int, 1>(), st, s, t);
      s = t;
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) consume(s[4 * g], s[4 * g + 1], s[4 * g + 2], s[4 * g + 3], g, kb);
  };
  const int steps = (nkeys + kStep - 1) / kStep;

  // Query q counts over lo .. hi next, or over images where that makes no grid: an empty, huge or tiny range, or bins below
  // four units in the last place of its ends.
  auto set_range = [&](int q, float lo, float hi) {
    const float sa = float(kBins - 2) / (hi - lo);
    const bool grid = hi > lo && sa < 1e30f && fmaxf(fabsf(lo), fabsf(hi)) * sa < 0x1p22f;
    s_lo[q] = lo;
    s_hi[q] = hi;
    s_a[q] = grid ? kBinWidth * sa : 0.f;
    s_b[q] = grid ? fmaf(-lo, kBinWidth * sa, kBin0 + kBinWidth) : 0.f;
    s_flag[grid ? 2 : 3] = 1;
  };

  // ---- 1: the range ----
  {
    float sum = 0.f, sq = 0.f;
    const bool sampled = q0 >= kSample;
    auto moments = [&](float w0, float w1, float w2, float w3, int, int) {
      const float x0 = w0 == w0 ? w0 : 0.f, x1 = w1 == w1 ? w1 : 0.f, x2 = w2 == w2 ? w2 : 0.f, x3 = w3 == w3 ? w3 : 0.f;
      sum += (x0 + x1) + (x2 + x3);
      sq += fmaf(x0, x0, x1 * x1) + fmaf(x2, x2, x3 * x3);
    };
    if (sampled)
      sweep(std::true_type(), kSample / kStep, (uint32_t(q0) << 12) / kSample, moments);
    else
      sweep(std::false_type(), steps, 0u, moments);
    sum += __shfl_xor(sum, 32, 64);
    sq += __shfl_xor(sq, 32, 64);
    float *part = reinterpret_cast<float *>(s_part);
    if (h == 0) {
      part[kg * NQ + ql] = sum;
      part[(KB + kg) * NQ + ql] = sq;
    }
    __syncthreads();
    if (tid < NQ) {
      float t0 = 0.f, t1 = 0.f;
#pragma unroll
      for (int g = 0; g < KB; ++g) {
        t0 += part[g * NQ + tid];
        t1 += part[(KB + g) * NQ + tid];
      }
      const int n = q0 + tid + 1;
      const float inv = 1.f / float(sampled ? kSample : min(n, a.S));
      const float mean = t0 * inv, dev = __builtin_amdgcn_sqrtf(fmaxf(t1 * inv - mean * mean, 0.f));
      const float mid = fmaf(dev, normal_quantile(fminf(float(a.topk) / float(n), 1.f)), mean);
      const float half = fmaxf(dev, 1e-6f * fabsf(mid));
      const bool open = n <= a.S && n > a.topk;   // else: all stay, or no such query
      s_a[tid] = s_b[tid] = 0.f;
      if (open) set_range(tid, mid - half, mid + half);
      s_first[tid] = open ? kLowest : 0u;
      s_last[tid] = open ? kHighest : 0u;
      s_over[tid] = 0u;
      s_ga[tid] = 0.f;                            // unless a bin is found: 0 w + 1 bin - 0 >= 1 bin, everything is above it
      s_gb[tid] = kBinWidth;
      s_bin[tid] = 0.f;
      s_need[tid] = 0;
      s_tie[tid] = -1;
      s_max[tid] = 0u;
      s_n[tid] = 0;
    }
  }

  // ---- 2: the bin of the K-th largest weight ----
  // Images of the smallest weights whose a w + b reaches `bin` and the next one (rounding is monotone): searched for within four
  // units in the last place of the points the line gives, both at once.
  auto ends_of = [&](float sa, float sb, float bin, uint32_t (&from)[2]) {
    const float inv = __builtin_amdgcn_rcpf(sa);
    uint32_t below[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float y = bin + float(i) * kBinWidth, d = y - sb - 0.5f, q = d * inv;   // (a w + b is rounded to a unit)
      const uint32_t at = weight_image(fmaf(fmaf(-q, sa, d), inv, q));
      below[i] = at - 4u;
      from[i] = at + 4u;
      if (!(fmaf(image_weight(below[i]), sa, sb) < y)) below[i] = kLowest;
      if (!(fmaf(image_weight(from[i]), sa, sb) >= y)) from[i] = kHighest;
    }
    while (max(from[0] - below[0], from[1] - below[1]) > 1u) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const uint32_t mid = below[i] + ((from[i] - below[i]) >> 1);   // (`below` itself once the search is over)
        const bool reached = fmaf(image_weight(mid), sa, sb) >= bin + float(i) * kBinWidth;
        from[i] = reached ? mid : from[i];
        below[i] = reached ? below[i] : mid;
      }
    }
  };
#pragma unroll 1
  for (int tries = 0, ranges = 1; tries < kRangeCounts + 4; ++tries) {
    if (tid == 0) s_flag[0] = 0;
    if (tid == 1) s_flag[2] = 0;
    for (int i = tid; i < NQ * kRows / 4; i += NT) reinterpret_cast<u32x4 *>(s_hist)[i] = u32x4{0u, 0u, 0u, 0u};
    if (tid < NQ) {
      s_min[tid] = ~0u;
      s_most[tid] = 0u;
    }
    __syncthreads();
    if (ranges) {
      const float sa = s_a[ql], sb = s_b[ql];
      float top = -INFINITY;
      using LdsCount = __attribute__((address_space(3))) uint32_t;
      const uint32_t column = uint32_t(uintptr_t((LdsCount *)smem)) + uint32_t(ql) * 4u;   // (shared memory starts at 0: nothing in it is static)
      sweep(std::false_type(), steps, 0u, [&](float w0, float w1, float w2, float w3, int, int) {
        const float w[4] = {w0, w1, w2, w3};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float y = __builtin_amdgcn_fmed3f(fmaf(w[i], sa, sb), kBin0, kBin0 + float(kBins - 1) * kBinWidth);
          uint32_t at = (__float_as_uint(y) & (uint32_t(kRows - 1) * kRow)) | column;   // row y's bin is in, of [kRows][NQ]
          asm("" : "+v"(at));                    // (one operation; left to itself the or joins the address's sum)
          const uint32_t one = (__float_as_uint(y) & (kRow / 2)) * (65536u / (kRow / 2)) | 1u;   // in both halves where the bin is odd
          __hip_atomic_fetch_add((LdsCount *)uintptr_t(at + 2 * Lds::kTile), one, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        top = fmaxf(fmaxf(fmaxf(fmaxf(top, w0), w1), w2), w3);   // (numbers go before NaN)
        asm volatile("" : "+v"(top));
      });
      __hip_atomic_fetch_max(&s_max[ql], weight_image(top), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (fabsf(top) * a.scale_log2 > 0x1p27f && top != -INFINITY) s_flag[4] = 1;   // (-infinity: no key of these was visible)
    } else {
      const uint32_t first = s_first[ql], span = s_last[ql] - first;
      const int shift = image_shift(span);
      uint32_t least = ~0u, most = 0u;
      sweep(std::false_type(), steps, 0u, [&](float w0, float w1, float w2, float w3, int, int) {
        const float w[4] = {w0, w1, w2, w3};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t u = weight_image(w[i] + 0.f), up = u - first;   // (-0 counts as 0)
          if (up <= span) {                      // not for the NaN of a hidden key, whose image is beyond both infinities'
            __hip_atomic_fetch_add(&s_hist[(up >> (shift + 1)) * NQ + ql], ((up >> shift) & 1u) << 16 | 1u, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
            least = min(least, u);
            most = max(most, u);
          }
        }
      });
      __hip_atomic_fetch_min(&s_min[ql], least, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      __hip_atomic_fetch_max(&s_most[ql], most, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __syncthreads();
    // TPQ threads per query, RPT rows each
    const int q = tid % NQ, grp = tid / NQ;
    const float sa = s_a[q];
    uint32_t word[RPT], mine = 0u;
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
      word[j] = s_hist[(grp * RPT + j) * NQ + q];
      mine += word[j] & 0xffffu;
    }
    s_part[grp * NQ + q] = mine;
    const bool open = ranges ? sa != 0.f : s_last[q] != 0u;
    uint32_t above = ranges ? 0u : s_over[q];
    __syncthreads();
#pragma unroll
    for (int g = 1; g < TPQ; ++g) above += g > grp ? s_part[g * NQ + q] : 0u;
    const uint32_t want = uint32_t(a.topk);
    if (open && above < want && above + mine >= want) {   // this thread's bins hold it
      int bin = 0;
      uint32_t here = 0u, up = 0u, down = 0u, over = 0u;   // the row's word, the next one's, the one's before, the weights above the row
      bool found = false;
#pragma unroll
      for (int j = RPT - 1; j >= 0; --j) {
        const uint32_t both = word[j] & 0xffffu;
        if (!found && above + both >= want) {
          found = true;
          bin = 2 * (grp * RPT + j);
          here = word[j];
          up = j + 1 < RPT ? word[j + 1] : 0u;
          down = j > 0 ? word[j - 1] : 0u;
          over = above;
        }
        above += both;
      }
      const uint32_t odd = here >> 16, even = (here & 0xffffu) - odd;
      const bool upper = over + odd >= want;     // in the odd bin
      if (upper) ++bin;
      else over += odd;
      const uint32_t in = upper ? odd : even, need = want - over;
      const uint32_t beside = upper ? even + (up & 0xffffu) - (up >> 16) : odd + (down >> 16);
      const bool all = need == in;               // the whole bin stays: nothing of it has to be ranked, however many they are
      const bool few = in <= uint32_t(kFew);
      if (ranges) {
        const float sb = s_b[q];
        s_a[q] = 0.f;
        s_b[q] = 0.f;
        if ((few || all) && bin > 0 && bin < kBins - 1) {
          s_ga[q] = sa;
          s_gb[q] = sb;
          s_bin[q] = kBin0 + kBinWidth * float(bin);
          s_need[q] = all ? 0 : int(need);
          s_first[q] = s_last[q] = 0u;
        } else {
          uint32_t end[2];
          ends_of(sa, sb, kBin0 + kBinWidth * float(bin), end);
          if (bin > 0) s_first[q] = max(s_first[q], end[0]);
          if (bin < kBins - 1 && end[1] <= s_last[q]) {
            s_last[q] = end[1] - 1u;
            s_over[q] = want - need;
          }
          const float lo = s_lo[q], hi = s_hi[q], width = (hi - lo) * (1.f / float(kBins - 2));
          const float at = fmaf(float(bin - 1), width, lo);
          const bool lonely = bin > 0 && bin < kBins - 1 && 8u * beside < in;
          if (lonely || tries + 1 == kRangeCounts)
            s_flag[3] = 1;
          else if (bin == 0)                     // below the range
            set_range(q, lo - 8.f * float(kBins - 2) * width, lo + width);
          else if (bin == kBins - 1)             // above it
            set_range(q, hi - width, hi + 8.f * float(kBins - 2) * width);
          else                                   // a quarter of a bin to spare on either side, for rounding
            set_range(q, at - 0.25f * width, at + 1.25f * width);
        }
      } else {
        uint32_t first = s_first[q], last = s_last[q];
        const int shift = image_shift(last - first);
        const uint32_t size = (1u << shift) - 1u;
        first += uint32_t(bin) << shift;
        if (last - first > size) last = first + size;
        if (few || all || shift == 0 || s_min[q] == s_most[q]) {   // few weights, or all of them stay, or are equal
          s_ga[q] = image_weight(first);
          s_gb[q] = image_weight(all ? first : last + 1u);   // (NaN behind infinity: nothing is above)
          s_bin[q] = -1.f;
          s_need[q] = all ? 0 : int(need);
          first = last = 0u;
          if (!few && !all) {
            s_tie[q] = -2;
            s_flag[1] = 1;
          }
        } else {
          s_flag[0] = 1;
        }
        s_first[q] = first;
        s_last[q] = last;
        s_over[q] = want - need;
      }
    }
    __syncthreads();
    const bool more = ranges ? (s_flag[2] | s_flag[3]) != 0 : s_flag[0] != 0;
    ranges = ranges ? s_flag[2] : 0;
    __syncthreads();
    if (!more) break;
  }
  // Bins of images are told by their ends (weights >= s_gb are above, those >= s_ga and not above inside); in a workgroup with such
  // queries the others' are as well.  The same variant takes workgroups with weights so large that w / sqrt(d) . log2 e, rounded for
  // the largest one, is off by several units: elsewhere that is a common factor of a query's weights, there they would overflow or
  // vanish.
  const bool by_images = __builtin_amdgcn_readfirstlane(s_flag[3] | s_flag[4]) != 0;
  if (by_images) {
    if (tid < NQ && s_bin[tid] >= 0.f) {
      const float bin = s_bin[tid];
      uint32_t end[2] = {kHighest, kLowest};     // no bin was looked for: all weights are above it
      if (bin > 0.f) ends_of(s_ga[tid], s_gb[tid], bin, end);
      s_ga[tid] = image_weight(end[0]);
      s_gb[tid] = image_weight(bin > 0.f && s_need[tid] == 0 ? end[0] : end[1]);
    }
    __syncthreads();
  }

  // ---- 3: the position up to which the weights of a bin stay that holds many equal ones ----
  const float from = s_ga[ql], above = s_gb[ql], bin = s_bin[ql];   // the ends of the bin, or a, b and the bin
  const float staying = s_need[ql] == 0 ? 0.f : kBinWidth;           // (all of the bin stays, none of it has to be ranked)
  auto inside = [&](float w) { return bool((w >= from) & !(w >= above)); };   // (false for the NaN of a hidden key)
  const bool crowded = s_flag[1] != 0;
  if (crowded) {
    u32x4 kr[NLD];
    load_tile(Kb, 0, kr);
    for (int st = 0; st < steps; ++st) {
      __syncthreads();
      store_tile(0, kr);
      if (st + 1 < steps) load_tile(Kb, st + 1, kr);
      __syncthreads();
      const int kb = st * kStep + kg * 32;
      uint32_t mask = 0u;
      f32x16 s = weights(0, nothing);
      if (kb + 31 > qfirst) hide(s, kb);
#pragma unroll
      for (int i = 0; i < 16; ++i) mask |= inside(s[i]) ? 1u << i : 0u;
      s_part[(kg * 2 + h) * NQ + ql] = mask;
      __syncthreads();
      if (tid < NQ && s_tie[tid] == -2) {
        int need = s_need[tid];
#pragma unroll
        for (int b = 0; b < KB; ++b) {
          const uint32_t m0 = s_part[2 * b * NQ + tid], m1 = s_part[(2 * b + 1) * NQ + tid];
          uint32_t pm = 0u;   // the block's 32 keys in order
#pragma unroll
          for (int j = 0; j < 4; ++j) pm |= ((m0 >> (4 * j)) & 15u) << (8 * j) | ((m1 >> (4 * j)) & 15u) << (8 * j + 4);
          const int here = __builtin_popcount(pm);
          if (need > 0 && need <= here) {
            for (int i = 1; i < need; ++i) pm &= pm - 1u;
            s_tie[tid] = st * kStep + b * 32 + __builtin_ctz(pm);
            need = 0;
          } else if (need > 0) {
            need -= here;
          }
        }
        if (need > 0) s_need[tid] = need;
      }
    }
    __syncthreads();
  }

  // ---- 4: O^T += V^T . P^T ----
  f32x16 o[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) o[db] = f32x16{0.f};
  float lsum = 0.f;
  auto product = [&](auto by_images_) {
    constexpr bool IMAGES = decltype(by_images_)::value;
    const float top = image_weight(s_max[ql]), negmax = -top * a.scale_log2;
    auto exponent = [&](float x) { return IMAGES ? (x - top) * a.scale_log2 : fmaf(x, a.scale_log2, negmax); };
    const int tie = s_tie[ql];
    const int grp = lane >> 4, vrow = 4 * (grp >> 1) + ((lane & 15) >> 2), vcol = (grp & 1) * 16 + (lane & 3) * 4;
    int vat[DB][2];                            // where the lane reads V^T in a tile: block of 32 head dimensions, half of 16 keys
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int e4 = 0; e4 < 2; ++e4)
        vat[db][e4] = chunk_at(kg * 32 + 8 * e4 + vrow, (db * 32 + vcol) >> 3) + (vcol & 4) * 2;
    // K is one step ahead of V: a step's products Q K^T run next to the exponentials of the step before
    constexpr int kV = 2 * Lds::kTile;
    u32x4 kr[NLD], vr[NLD];
    load_tile(Kb, 0, kr);
    __syncthreads();
    store_tile(0, kr);
    if (steps > 1) load_tile(Kb, 1, kr);
    load_tile(Vb, 0, vr);
    __syncthreads();
    if (steps > 1) store_tile(Lds::kTile, kr);
    store_tile(kV, vr);
    if (steps > 2) load_tile(Kb, 2, kr);
    if (steps > 1) load_tile(Vb, 1, vr);
    f32x16 s = weights(0, nothing);
    int kb = kg * 32;
    if (kb + 31 > qfirst) hide(s, kb);
    // The weights w of step st - 1 into the result, and those of step st into next (unless LAST: no such step).
    auto one = [&](auto last_, int st, const f32x16 &w, f32x16 &next) {
      constexpr bool LAST = decltype(last_)::value;
      const int tile = (st & 1) * Lds::kTile, other = Lds::kTile - tile;
      __syncthreads();                         // tiles st of K and st - 1 of V are there
      if constexpr (!LAST) {
        if (st + 1 < steps) store_tile(other, kr);
        store_tile(kV + tile, vr);
        if (st + 2 < steps) load_tile(Kb, st + 2, kr);
        if (st + 1 < steps) load_tile(Vb, st + 1, vr);
      }
      // P of two of the lane's weights, as two bf16 terms: the upper 16 bits, and what is left (exact, >= 0) rounded
      auto exponentials = [&](float x0, float x1, uint64_t stays0, uint64_t stays1, uint32_t &ph, uint32_t &pl) {
        const float p0 = __builtin_amdgcn_inverse_ballot_w64(stays0) ? __builtin_amdgcn_exp2f(exponent(x0)) : 0.f;
        const float p1 = __builtin_amdgcn_inverse_ballot_w64(stays1) ? __builtin_amdgcn_exp2f(exponent(x1)) : 0.f;
        lsum += p0 + p1;
        asm volatile("" : "+v"(lsum));        // added here: sixteen of them are not kept for the end of the step
        const uint32_t h0 = __float_as_uint(p0), h1 = __float_as_uint(p1);
        ph = __builtin_amdgcn_perm(h1, h0, 0x07060302u);   // (h0 >> 16) | (h1 & 0xffff0000)
        pl = two_bf16(p0 - __uint_as_float(h0 & 0xffff0000u), p1 - __uint_as_float(h1 & 0xffff0000u));
        asm volatile("" : "+v"(ph), "+v"(pl));   // done here, between the matrix instructions
      };
      // V^T operand: head dimensions db * 32 + c; element e of lane half h is key 16 ks + 8 (e / 4) + 4 h + e % 4
      const int vt = kV + other;
      union Operand {
        s16x4 q[2];
        bf16x8 v;
      };
      Operand vo[DB];
      auto read_v = [&](int ks, int db) {
#pragma unroll
        for (int e4 = 0; e4 < 2; ++e4) {
          const int at = vat[db][e4] + vt + ks * (16 * DH * 2);
          vo[db].q[e4] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(smem + at));
        }
      };
      auto add_product = [&](int db, const u32x4 &ph, const u32x4 &pl) {
        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vo[db].v, *reinterpret_cast<const bf16x8 *>(&ph), o[db], 0, 0, 0);
        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vo[db].v, *reinterpret_cast<const bf16x8 *>(&pl), o[db], 0, 0, 0);
        asm volatile("" : "+v"(o[db]));
      };
      // Of equal weights those up to `tie` stay: in a block that is all before it or all behind it one end of the bin tells them.
      float low = from, high = above;
      if (IMAGES && crowded) {
        const bool before = kb + 31 <= tie, behind = tie >= 0 && kb > tie;
        high = before ? from : above;
        low = before || behind ? high : from;
      }
      uint32_t ph[8], pl[8];
      auto share = [&](int g) {
        // the lanes whose weight stays, and those whose weight is inside the bin (neither for the NaN of a hidden key)
        uint64_t stays[4], in[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float x = w[4 * g + i];
          if constexpr (IMAGES) {
            stays[i] = lanes_ge(x, high);
            in[i] = lanes_ge(x, low) & ~stays[i];
          } else {
            // >= kBinWidth above the bin, in [0, kBinWidth) inside it, else below (exact: rounding is monotone, and the difference is
            // exact inside the bin)
            const float d = fmaf(x, from, above) - bin;
            stays[i] = lanes_ge(d, staying);
            in[i] = lanes_below(d, __float_as_uint(staying));
          }
        }
        if ((in[0] | in[1] | in[2] | in[3]) != 0) {
          if (IMAGES && crowded) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              stays[i] |= in[i] & __builtin_amdgcn_ballot_w64(kb + 8 * g + 4 * h + i <= tie);
              in[i] &= __builtin_amdgcn_ballot_w64(tie < 0);
            }
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if (__builtin_amdgcn_inverse_ballot_w64(in[i])) {
              const int at = __hip_atomic_fetch_add(&s_n[ql], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
              if (at < kFew) s_few[ql * kFew + at] = float2{w[4 * g + i], __int_as_float(kb + 8 * g + 4 * h + i)};
            }
          }
        }
        exponentials(w[4 * g], w[4 * g + 1], stays[0], stays[1], ph[2 * g], pl[2 * g]);
        exponentials(w[4 * g + 2], w[4 * g + 3], stays[2], stays[3], ph[2 * g + 1], pl[2 * g + 1]);
        if (g >= 4 - DB) read_v(0, g - 4 + DB);
      };
      if constexpr (LAST) {
#pragma unroll
        for (int g = 0; g < 4; ++g) share(g);
      } else {
        if constexpr (kFirst) __builtin_amdgcn_s_setprio(1);
        next = weights(tile, share);
        if constexpr (kFirst) __builtin_amdgcn_s_setprio(0);
      }
#pragma unroll
      for (int g = 0; g < DB; ++g) {
        add_product(g, u32x4{ph[0], ph[1], ph[2], ph[3]}, u32x4{pl[0], pl[1], pl[2], pl[3]});
        read_v(1, g);
        // each read of the second half under the products of the first: 663 -> 659 us for 512 rows of 1024; not with 32 queries, where a
        // wave has its SIMD to itself and the compiler's order is the better one (2 rows of 3000 112 -> 105, 4 of 1000 46.2 -> 44.0)
        if constexpr (NQB == 2) __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int g = 0; g < DB; ++g) add_product(g, u32x4{ph[4], ph[5], ph[6], ph[7]}, u32x4{pl[4], pl[5], pl[6], pl[7]});
      kb += kStep;
      if (!LAST && kb + 31 > qfirst) hide(next, kb);
    };
    int st = 1;
    for (; st < steps; ++st) {
      const f32x16 w = s;
      one(std::false_type(), st, w, s);
    }
    one(std::true_type(), st, s, s);
  };
  if (by_images)
    product(std::true_type());
  else
    product(std::false_type());

  // ---- 5: the weights set aside, and the four key groups' partial sums in order ----
  lsum += __shfl_xor(lsum, 32, 64);
  if (h == 0) s_l[kg * NQ + ql] = lsum;
  __syncthreads();
  f32x4 *s_mrg = reinterpret_cast<f32x4 *>(smem);   // [wave][DB][4][64], lanes permuted so that the reads below spread over the banks
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      s_mrg[((wave * DB + db) * 4 + j) * 64 + (lane ^ ((db * 4 + j) & 7))] = f32x4{o[db][4 * j], o[db][4 * j + 1], o[db][4 * j + 2], o[db][4 * j + 3]};
  // TPQ threads per query: each ranks its share of the weights and notes the ones that stay; then each adds its share of their rows
  // of V, 16-byte chunks sub, sub + TPQ, .., in fp32.
  constexpr int WPT = kFew / TPQ, CPT = CPR / TPQ;   // weights and chunks per thread
  const int q = tid / TPQ, sub = tid % TPQ, held = min(s_n[q], kFew), need = s_need[q];
  float extra[8 * CPT] = {0.f}, extra_l = 0.f;
  if (held > 0) {
    float2 mine[WPT];
    int before[WPT] = {0};
#pragma unroll
    for (int e = 0; e < WPT; ++e) mine[e] = s_few[q * kFew + sub + TPQ * e];
    for (int j = 0; j < held; ++j) {
      const float2 v = s_few[q * kFew + j];
#pragma unroll
      for (int e = 0; e < WPT; ++e) before[e] += v.x > mine[e].x || (v.x == mine[e].x && __float_as_int(v.y) < __float_as_int(mine[e].y)) ? 1 : 0;
    }
    // in the order of their rank, so that the sum does not hang on the order they were set aside in
    wave_lds_fence();
#pragma unroll
    for (int e = 0; e < WPT; ++e)
      if (sub + TPQ * e < held) s_few[q * kFew + before[e]] = mine[e];
    wave_lds_fence();
    const float top = image_weight(s_max[q]), less = by_images ? top : 0.f, negmax = by_images ? 0.f : -top * a.scale_log2;
    const int stay = min(need, held);
    for (int j0 = 0; j0 < stay; j0 += 4) {     // four rows on their way at once
      u32x4 row[4][CPT];
      float p[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float2 v = s_few[q * kFew + min(j0 + j, stay - 1)];
        p[j] = j0 + j < stay ? __builtin_amdgcn_exp2f(fmaf(v.x - less, a.scale_log2, negmax)) : 0.f;   // (as in the product)
        const bf16_t *src = Vb + size_t(__float_as_int(v.y)) * DH + sub * 8;
#pragma unroll
        for (int e = 0; e < CPT; ++e) row[j][e] = *reinterpret_cast<const u32x4 *>(src + 8 * TPQ * e);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        extra_l += p[j];
#pragma unroll
        for (int e = 0; e < CPT; ++e)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            extra[8 * e + 2 * i] = fmaf(p[j], __uint_as_float(row[j][e][i] << 16), extra[8 * e + 2 * i]);
            extra[8 * e + 2 * i + 1] = fmaf(p[j], __uint_as_float(row[j][e][i] & 0xffff0000u), extra[8 * e + 2 * i + 1]);
          }
      }
    }
  }
  __syncthreads();
  // The same thread finishes its chunks of the query's row: chunk ch, head dimensions 8 ch + d, sits at block ch / 4, element
  // 4 (ch % 4) + d % 4 of the lane half d / 4.
  float l = extra_l;
#pragma unroll
  for (int g = 0; g < KB; ++g) l += s_l[g * NQ + q];
  const float inv = l > 0.f ? 1.f / l : 0.f;
  if (q0 + q < a.S) {
#pragma unroll
    for (int e = 0; e < CPT; ++e) {
      const int ch = TPQ * e + sub, db = ch / 4, j = ch % 4;
      uint32_t r[8];
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        f32x4 sum = f32x4{extra[8 * e + 4 * half], extra[8 * e + 4 * half + 1], extra[8 * e + 4 * half + 2], extra[8 * e + 4 * half + 3]};
#pragma unroll
        for (int g = 0; g < KB; ++g) {
          const f32x4 v = s_mrg[(((g * NQB + q / 32) * DB + db) * 4 + j) * 64 + ((half * 32 + (q & 31)) ^ ((db * 4 + j) & 7))];
#pragma unroll
          for (int i = 0; i < 4; ++i) sum[i] += v[i];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) r[4 * half + i] = f32_to_bf16_rne(sum[i] * inv);
      }
      *reinterpret_cast<u32x4 *>(a.O + base + size_t(q0 + q) * DH + 8 * ch) =
          u32x4{r[0] | (r[1] << 16), r[2] | (r[3] << 16), r[4] | (r[5] << 16), r[6] | (r[7] << 16)};
    }
  }
}

template <int DH, int NQB, int KB>
hipError_t launch(TopkArgs a, hipStream_t st) {
  constexpr int lds = TopkLds<DH, NQB, KB>::kBytes, threads = 64 * NQB * KB;
  static_assert(lds <= 160 * 1024, "shared memory of a compute unit");
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&topk_attend_kernel<DH, NQB, KB>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  // A launch holds fewer than 2^32 threads: whole groups of eight rows (one per XCD) at a time where there are more
  // (from 8193 tokens on, at 65535 rows).
  const int blocks = (a.S + 32 * NQB - 1) / (32 * NQB), rows = a.rows;
  const int most = int(0xffffffffu / (unsigned(threads) * unsigned(blocks)) / 8u * 8u);
  for (int r0 = 0; r0 < rows; r0 += most) {
    a.rows = rows - r0 < most ? rows - r0 : most;
    hipLaunchKernelGGL((topk_attend_kernel<DH, NQB, KB>), dim3(unsigned(a.rows) * unsigned(blocks)), dim3(threads), lds, st, a);
    const size_t done = size_t(a.rows) * a.S * DH;
    a.Q += done;
    a.K += done;
    a.V += done;
    a.O += done;
  }
  return hipGetLastError();
}

constexpr int kMaxStaticSeq = 2048;  // longest sequence adore_topk_attention_static takes
constexpr int kMaxSeq = 32768;       // longest sequence taken at all

// The launch of both entry points.  64 queries per workgroup read K and V half as often, and two such workgroups share a compute unit;
// 32 where that leaves units without one.  At d = 128 a workgroup of 32 has a unit to itself, so that more than 256 of them take a
// second round (us, 32 / 64 queries: 8 rows of 1024 tokens, 128 workgroups of 64, 47 / 48; 8 of 2048, 256 of them, 107 / 111; 4 of 4096, 256,
// 258 / 139; 20 of 1024, 320, 104 / 60; 33 of 777, 429, 104 / 45); at d = 64 two of them fit (16 of 512, 128, 19.8 / 24.7; 24 of 1024, 384, 44.3 /
// 46.2; 40 of 500, 320, 30.1 / 28.3).
int enqueue_topk(const void *q, const void *k, const void *v, void *out, int rows, int seq, int head_dim, int top_k,
                 hipStream_t st) {
  TopkArgs a;
  a.Q = static_cast<const bf16_t *>(q);
  a.K = static_cast<const bf16_t *>(k);
  a.V = static_cast<const bf16_t *>(v);
  a.O = static_cast<bf16_t *>(out);
  a.S = seq;
  a.rows = rows;
  a.topk = top_k;
  a.scale_log2 = 1.4426950408889634f / sqrtf(float(head_dim));
  hipError_t e;
  if (rows * ((seq + 63) / 64) < (head_dim == 128 ? 256 : 512))
    e = head_dim == 128 ? launch<128, 1, 4>(a, st) : launch<64, 1, 4>(a, st);
  else
    e = head_dim == 128 ? launch<128, 2, 2>(a, st) : launch<64, 2, 2>(a, st);
  return e == hipSuccess ? ADORE_OK : ADORE_E_HIP;
}

// What the ABI promises to ask a caller for: room for a transposed copy of V and, for long sequences, for the weights of 512
// workgroups of 16 queries.  Nothing uses it any more; the amounts stay, so that callers who keep track of them see no change.
size_t padded_keys(int S) { return size_t(S + 31) / 32 * 32; }
size_t vt_bytes(int rows, int S, int d) { return (size_t(rows) * d * padded_keys(S) * 2 + 255) / 256 * 256; }

}  // namespace

}  // namespace adore

extern "C" {

size_t adore_topk_attention_workspace_bytes(int32_t rows, int32_t seq, int32_t head_dim) {
  if (rows <= 0 || seq <= 0 || head_dim <= 0) return 0;
  if (seq > adore::kMaxSeq || rows > 65535 || head_dim > 1024) return 0;   // nothing the entry point would take
  const size_t blocks = size_t(rows) * ((seq + 15) / 16);
  const size_t weights = seq > adore::kMaxStaticSeq ? (blocks < 512 ? blocks : 512) * 16 * (adore::padded_keys(seq) + 4) * 4 : 0;
  return adore::vt_bytes(rows, seq, head_dim) + (weights + 255) / 256 * 256;
}

int adore_topk_attention(const void *q, const void *k, const void *v, void *out, void *workspace,
                         size_t workspace_bytes, int32_t rows, int32_t seq, int32_t head_dim, int32_t top_k,
                         void *hip_stream) {
  using namespace adore;
  if (!q || !k || !v || !out || !workspace || rows <= 0 || seq <= 0 || head_dim <= 0 || top_k < 1) return ADORE_E_INVALID;
  if ((head_dim != 64 && head_dim != 128) || seq > kMaxSeq || rows > 65535) return ADORE_E_UNSUPPORTED;
  if (workspace_bytes < adore_topk_attention_workspace_bytes(rows, seq, head_dim) ||
      (reinterpret_cast<uintptr_t>(workspace) & 255) != 0)
    return ADORE_E_WORKSPACE;
  return enqueue_topk(q, k, v, out, rows, seq, head_dim, top_k, static_cast<hipStream_t>(hip_stream));
}

int adore_topk_attention_static(const void *q, const void *k, const void *v, void *out, int32_t rows, int32_t seq,
                                int32_t head_dim, int32_t top_k, void *hip_stream) {
  using namespace adore;
  if (!q || !k || !v || !out || rows <= 0 || seq <= 0 || head_dim <= 0 || top_k < 1) return ADORE_E_INVALID;
  if ((head_dim != 64 && head_dim != 128) || rows > 65535) return ADORE_E_UNSUPPORTED;
  if (seq > kMaxStaticSeq || vt_bytes(rows, seq, head_dim) > size_t(ADORE_TOPK_STATIC_SCRATCH_BYTES)) return ADORE_E_WORKSPACE;
  return enqueue_topk(q, k, v, out, rows, seq, head_dim, top_k, static_cast<hipStream_t>(hip_stream));
}

}  // extern "C"
