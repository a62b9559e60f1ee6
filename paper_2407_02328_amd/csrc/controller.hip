// Stage 2: the controller module (paper Sec. 2.2, Eq. 2; App. "Implementation
// Details": GRU input size D -> d', position layer 1 -> d', interaction layer
// d' -> d' with tanh, output layer d' -> 1 with sigmoid).
//
//   z_i     = GRU(x_i, z_{i-1})
//   sigma_i = sigmoid(out_w . tanh(W_1 (p_i + z_i) + b_1) + out_b),  p_i = pos_w * (i * pos_scale) + pos_b
//
// Two kernels.  ctrl_input computes the input pre-activations W_ih x for a
// batch of tokens: the only part that reads D-wide data, and free of any
// dependence between tokens, so a whole prompt chunk goes in one launch.  In
// bf16 it is a [tokens x D] x [D x 3d'] contraction on the matrix cores
// (16x16x32 tiles: 16 tokens x 16 gate rows), cut along D into `ksplit` slices
// so that a decode step (16 tokens) still spreads over many compute units; the
// slices are added up in a fixed order by the cell kernel.  ctrl_cell does the
// recurrent part token by token: W_hh z, the gates, the MLP and the score.
// All sums are fp32 in a fixed order, so results are reproducible run to run.
#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "ctrl_device.h"

namespace adore {

namespace {

// grid (3d'/16, ceil(ntok/16), ksplit), 256 threads
__global__ __launch_bounds__(256) void ctrl_input_mfma_kernel(const bf16_t *__restrict__ W_ih,
                                                              const bf16_t *__restrict__ x,
                                                              float *__restrict__ part, int D, int G3, int ntok,
                                                              int per_seq, int seq_rows, int kslice) {
  __builtin_amdgcn_s_setprio(3);   // short, latency-bound work that shares compute units with the GEMM: its waves go first
  __shared__ float red[kInputTileLds];
  ctrl_input_mfma_tile(W_ih, x, part, D, G3, ntok, per_seq, seq_rows, kslice, blockIdx.x, blockIdx.y, blockIdx.z, red);
}

template <typename T>
__global__ __launch_bounds__(256) void ctrl_input_kernel(const T *__restrict__ W_ih, const T *__restrict__ x,
                                                         float *__restrict__ gi, int D, int G3, int ntok,
                                                         int per_seq, int seq_rows) {
  __shared__ float red[4 * JT * NB];
  ctrl_input_plain_tile<T>(W_ih, x, gi, D, G3, ntok, per_seq, seq_rows, blockIdx.x, blockIdx.y, red);
}

// ---- input projection of a prompt chunk, bf16, matrix cores ---------------------------
// Thousands of tokens at once: a workgroup owns 64 tokens x 64 gate rows (4 x 4 tiles of the shape above)
// and the whole of D; its 4 waves cut D and keep all 16 tiles each, so a wave multiplies 16 tiles with
// 4 + 4 operand loads per step (the 16-token tile above re-reads W_ih once per 16 tokens and x once per
// 16 gate rows: at 8192 tokens that was 800 us).  The waves' sums are added in a fixed order.
// grid (ceil(3d'/64), ceil(ntok/64)), 256 threads.  gi[tok][j] (one D-slice).
__global__ __launch_bounds__(256) void ctrl_input_prompt_kernel(const bf16_t *__restrict__ W_ih,
                                                                const bf16_t *__restrict__ x,
                                                                float *__restrict__ gi, int D, int G3, int ntok,
                                                                int per_seq, int seq_rows) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int j0 = blockIdx.x * 64, t0 = blockIdx.y * 64;
  const int kw = D / 4;                            // k-range of one wave, a multiple of 32
  // a step of 32 k is one contiguous 64-byte run of every row, lane group g = lane/16 taking its g-th quarter
  // (with thousands of rows in flight, rows walked in four places at once would not stay in the L1)
  const int kbeg = wave * kw + (lane >> 4) * 8;
  const u32x4 *pa[4], *pb[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int tok = t0 + 16 * i + (lane & 15);
    if (tok >= ntok) tok = ntok - 1;               // padded rows read a valid token; dropped at the store
    const size_t xrow = size_t(tok / per_seq) * seq_rows + tok % per_seq;
    pa[i] = reinterpret_cast<const u32x4 *>(x + xrow * D + kbeg);
    int j = j0 + 16 * i + (lane & 15);
    if (j >= G3) j = G3 - 1;
    pb[i] = reinterpret_cast<const u32x4 *>(W_ih + size_t(j) * D + kbeg);
  }
  f32x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) acc[i][jj] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int steps = kw / 32;
#define PROMPT_STEP(VA, VB)                                                                                   \
  _Pragma("unroll") for (int i = 0; i < 4; ++i)                                                               \
    _Pragma("unroll") for (int jj = 0; jj < 4; ++jj)                                                          \
      acc[i][jj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8 *>(&VA[i]),         \
                                                           *reinterpret_cast<const bf16x8 *>(&VB[jj]), acc[i][jj], 0, 0, 0);
  int s = 0;
  for (; s + 2 <= steps; s += 2) {          // two steps' loads in flight
    u32x4 va[2][4], vb[2][4];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) { va[u][i] = pa[i][(s + u) * 4]; vb[u][i] = pb[i][(s + u) * 4]; }
    PROMPT_STEP(va[0], vb[0])
    PROMPT_STEP(va[1], vb[1])
  }
  for (; s < steps; ++s) {
    u32x4 va[4], vb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) { va[i] = pa[i][s * 4]; vb[i] = pb[i][s * 4]; }
    PROMPT_STEP(va, vb)
  }
#undef PROMPT_STEP
  // waves 3, 2, 1 hand their tiles to wave 0 through LDS, one after the other
  __shared__ float red[16][4][64];   // [tile][v][lane]: conflict-free, lane-private
  for (int w = 3; w >= 1; --w) {
    if (wave == w) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
#pragma unroll
          for (int v = 0; v < 4; ++v) red[i * 4 + jj][v][lane] = acc[i][jj][v];
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[i][jj][v] += red[i * 4 + jj][v][lane];
    }
    __syncthreads();
  }
  if (wave == 0) {   // accumulator element v of lane L: token 4*(L/16) + v, gate row L%16 of its tile
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int tok = t0 + 16 * i + 4 * (lane >> 4) + v, j = j0 + 16 * jj + (lane & 15);
          if (tok < ntok && j < G3) gi[size_t(tok) * G3 + j] = acc[i][jj][v];
        }
  }
}

// One token per sequence (a decode step).  One workgroup of 12 waves per sequence.  A step's cost is not its
// arithmetic (100 k multiply-adds) but its trips to memory, each of which takes microseconds next to the
// attention's traffic: so everything the step reads is requested at the top, before anything is waited for: the
// state, the D-slices of the input pre-activations, W_hh (32 rows per wave), W_1 (32 rows each for 4 of the
// waves), the small vectors.  After that the kernel only computes, with three barriers.
template <typename T>
__global__ __launch_bounds__(768) void ctrl_cell128_kernel(const CellArgs a) {
  __builtin_amdgcn_s_setprio(3);   // short, latency-bound work next to the attention: its waves go first
  constexpr int DP = 128;
  __shared__ float gi_s[3 * DP];   // W_ih x + b_ih
  __shared__ float gh[3 * DP];     // W_hh h + b_hh
  __shared__ float t_in[DP];       // p_i + z_i
  __shared__ float u1[DP];         // W_1 (p + z) + b_1
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const T *W_hh = static_cast<const T *>(a.W_hh);
  const size_t tok = size_t(b);    // nsteps == 1
  // ---- requests ----
  const float2 hx = *reinterpret_cast<const float2 *>(a.z + size_t(b) * DP + 2 * lane);   // z_{i-1}, in every wave
  decltype(load_raw2(W_hh)) rhh[32];
  rows_request<T, 32>(W_hh, wave * 32, lane, rhh);
  float2 rw1[32];                  // (batches of 32 rows, as where a prompt chunk is scored: the same sums in the same order)
  if (wave < 4) rows_request<float, 32>(a.W1, wave * 32, lane, rw1);
  float g = 0.f, hold = 0.f, pw = 0.f, pb = 0.f, ow0 = 0.f, ow1 = 0.f, ob = 0.f, ov = 0.f;
  if (tid < 3 * DP) g = gi_sum(a, tok, tid) + a.b_ih[tid];
  if (tid < DP) {
    hold = a.z[size_t(b) * DP + tid];
    pw = a.pos_w[tid];
    pb = a.pos_b[tid];
  }
  if (wave == 0) {
    ow0 = a.out_w[lane];
    ow1 = a.out_w[lane + 64];
    ob = a.out_b[0];
    if (a.override_) ov = a.override_[size_t(b) * a.override_stride];
  }
  __builtin_amdgcn_sched_barrier(0);   // all of the above is under way before the first use
  // ---- recurrent pre-activations, the gates, the new state ----
  rows_finish<decltype(load_raw2(W_hh)), 32>(rhh, wave * 32, hx.x, hx.y, a.b_hh, gh, lane);
  if (tid < 3 * DP) gi_s[tid] = g;
  __syncthreads();
  if (tid < DP) {
    const float r = sigmoidf_(gi_s[tid] + gh[tid]);
    const float u = sigmoidf_(gi_s[DP + tid] + gh[DP + tid]);
    const float cand = tanhf(gi_s[2 * DP + tid] + r * gh[2 * DP + tid]);
    const float hnew = (1.0f - u) * cand + u * hold;
    const float delta = a.cvec ? 0.f : float(a.pos0) * a.pos_scale;   // rescore mode: distance to itself
    a.z[size_t(b) * DP + tid] = hnew;
    t_in[tid] = fmaf(pw, delta, pb) + hnew;
  }
  __syncthreads();
  // ---- interaction layer, output layer, sigmoid ----
  if (wave < 4) rows_finish<float2, 32>(rw1, wave * 32, t_in[2 * lane], t_in[2 * lane + 1], a.b1, u1, lane);
  __syncthreads();
  if (a.cvec && tid < DP) a.cvec[(size_t(b) * a.N_max + a.pos0) * DP + tid] = u1[tid];
  if (wave == 0) {
    float s = fmaf(ow0, tanhf(u1[lane]), ow1 * tanhf(u1[lane + 64]));
    s = wave_sum(s);
    if (lane == 0) a.score[size_t(b) * a.N_max + a.pos0] = a.override_ ? ov : sigmoidf_(s + ob);
  }
}

// ---- a prompt chunk, d' = 128: the recurrence alone, then the layers above it for all tokens at once ----
// Only z_i = GRU(x_i, z_{i-1}) ties a token to the one before it; the position, interaction and output layers
// do not.  The scan therefore does nothing but the recurrence, one workgroup of 4 waves per sequence.  With fp32
// weights W_hh stays in registers as fp32 for the whole chunk: wave w keeps columns 32w .. 32w+31 of all 384 rows (lane l: rows
// l, l+64, .., l+320), so a token costs a wave 8 16-byte reads of the state from LDS (same address in every
// lane) and 192 multiply-adds per lane on each of the four SIMDs; the four partial sums of a row meet in LDS,
// 128 threads apply the gates.  Two barriers and no memory round trip per token.  The gates use the hardware's exp2 and reciprocal
// (about 2e-7 absolute); z_i goes to zseq[b * nsteps + i][128] for the kernel below.
__device__ inline float scan_sigmoid(float a) {
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504f * a));
}
__device__ inline float scan_tanh(float a) {
  return 1.0f - 2.0f * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(2.88539008f * a));
}

template <typename T>
__global__ __launch_bounds__(256) void ctrl_scan128_kernel(const CellArgs a, float *__restrict__ zseq) {
  constexpr int DP = 128, KW = 32, RPL = 6;               // columns per wave, rows per lane
  constexpr int TB = 16, GPT = TB * (3 * DP / 4) / 256;   // tokens per block of input pre-activations; float4 per thread
  __shared__ __attribute__((aligned(16))) float h[DP];   // z_{i-1}, then z_i
  __shared__ float part[4][3 * DP];                        // the waves' partial sums of W_hh h
  __shared__ float4 gbuf[2][TB * (3 * DP / 4)];            // input pre-activations of two blocks of tokens
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float w[RPL][KW];
  {
    constexpr int EPL = Vec16<T>::EPL;
#pragma unroll
    for (int m = 0; m < RPL; ++m) {
      const T *row = static_cast<const T *>(a.W_hh) + size_t(lane + 64 * m) * DP + wave * KW;
#pragma unroll
      for (int c = 0; c < KW; c += EPL) {
        float f[EPL];
        Vec16<T>::load(row + c, f);
#pragma unroll
        for (int e = 0; e < EPL; ++e) w[m][c + e] = f[e];
      }
    }
  }
  float b_r = 0.f, b_u = 0.f, b_in = 0.f, b_hn = 0.f, hcur = 0.f;
  if (tid < DP) {
    hcur = a.z[size_t(b) * DP + tid];
    h[tid] = hcur;
    b_r = a.b_ih[tid] + a.b_hh[tid];
    b_u = a.b_ih[DP + tid] + a.b_hh[DP + tid];
    b_in = a.b_ih[2 * DP + tid];
    b_hn = a.b_hh[2 * DP + tid];
  }
  // The input pre-activations reach the gates through LDS, TB tokens at a time: the rows of block j+1 are
  // fetched (all threads, 16 bytes each, the D-slices added up) while block j is worked through, so the
  // recurrence never waits for memory.
  const int nblk = (a.nsteps + TB - 1) / TB;
  const float4 *gsrc = reinterpret_cast<const float4 *>(a.gi) + size_t(b) * a.nsteps * (3 * DP / 4);
  const size_t slice4 = size_t(a.ntok) * (3 * DP / 4);   // distance between two D-slices
  float4 stage[GPT];
  auto fetch = [&](int blk) {
    const int rows = a.nsteps - blk * TB < TB ? a.nsteps - blk * TB : TB;
#pragma unroll
    for (int q = 0; q < GPT; ++q) {
      const int idx = tid + 256 * q;
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (idx < rows * (3 * DP / 4)) {
        const float4 *p = gsrc + size_t(blk) * TB * (3 * DP / 4) + idx;
        v = p[0];
        for (int k = 1; k < a.ksplit; ++k) {
          const float4 t = p[size_t(k) * slice4];
          v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w;
        }
      }
      stage[q] = v;
    }
  };
  auto park = [&](int buf) {
#pragma unroll
    for (int q = 0; q < GPT; ++q) gbuf[buf][tid + 256 * q] = stage[q];
  };
  if (nblk > 0) {
    fetch(0);
    park(0);
  }
  __syncthreads();
  for (int blk = 0; blk < nblk; ++blk) {
    if (blk + 1 < nblk) fetch(blk + 1);
    const float *g = reinterpret_cast<const float *>(gbuf[blk & 1]);
    const int rows = a.nsteps - blk * TB < TB ? a.nsteps - blk * TB : TB;
    for (int ii = 0; ii < rows; ++ii) {
      const size_t tok = size_t(b) * a.nsteps + blk * TB + ii;
      float acc[RPL];
#pragma unroll
      for (int m = 0; m < RPL; ++m) acc[m] = 0.f;
#pragma unroll
      for (int k = 0; k < KW; k += 4) {
        const float4 hv = *reinterpret_cast<const float4 *>(&h[wave * KW + k]);
#pragma unroll
        for (int m = 0; m < RPL; ++m) {
          acc[m] = fmaf(w[m][k], hv.x, acc[m]);
          acc[m] = fmaf(w[m][k + 1], hv.y, acc[m]);
          acc[m] = fmaf(w[m][k + 2], hv.z, acc[m]);
          acc[m] = fmaf(w[m][k + 3], hv.w, acc[m]);
        }
      }
#pragma unroll
      for (int m = 0; m < RPL; ++m) part[wave][lane + 64 * m] = acc[m];
      __syncthreads();
      if (tid < DP) {
        const float s_r = (part[0][tid] + part[1][tid]) + (part[2][tid] + part[3][tid]);
        const float s_u = (part[0][DP + tid] + part[1][DP + tid]) + (part[2][DP + tid] + part[3][DP + tid]);
        const float s_n = (part[0][2 * DP + tid] + part[1][2 * DP + tid]) + (part[2][2 * DP + tid] + part[3][2 * DP + tid]);
        const float *gt = g + ii * 3 * DP;
        const float r = scan_sigmoid(gt[tid] + b_r + s_r);
        const float u = scan_sigmoid(gt[DP + tid] + b_u + s_u);
        const float cand = scan_tanh(gt[2 * DP + tid] + b_in + r * (s_n + b_hn));
        hcur = (1.0f - u) * cand + u * hcur;
        h[tid] = hcur;
        zseq[tok * DP + tid] = hcur;
      }
      __syncthreads();
    }
    if (blk + 1 < nblk) park((blk + 1) & 1);   // read next after at least one more barrier
  }
  if (tid < DP) a.z[size_t(b) * DP + tid] = hcur;
}

// The same recurrence with bf16 weights, on the matrix cores: W_hh z with z as three bf16 terms (8 + 8 + 8 significant
// bits: the split is exact, so is every product, and the sums are fp32).  One workgroup of 4 waves per sequence; wave w owns
// the units 32w .. 32w+31 of all three gates: six 16-row tiles of W_hh in registers as 16x16x32 operands (96 registers).  The
// columns of the other operand are the three terms (column c holds term c % 4, the fourth is zero), so a token costs a wave
// 24 matrix instructions; four neighbouring lanes then hold the terms of one sum, two DPP additions put it together, and the
// gates follow in the same wave: one barrier per token, for the exchange of z through LDS.
// What bounds it is the serial chain of a token on one compute unit: 384 cycles of matrix instructions, then the sums, the
// gates' three exponentials and reciprocals, and the trip of z through LDS.  0.365 us per token (187 us per chunk of 512; 386 us
// with 192 fp32 multiply-adds per lane and token, two barriers: ctrl_scan128_kernel, which fp32 weights still take).  Error of z
// against 64 bits over prompts of 8 to 2048 tokens: 1.0e-7 to 2.1e-7 relative, as before.
template <int CTRL>
__device__ inline float quad_add(float v) {   // v + the value of the lane that CTRL (a quad_perm) names
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}

// SPLIT: the pre-activations come in several D-slices (a short prompt of few sequences); they are added up and staged
// through LDS, 16 tokens at a time.  Otherwise a lane reads its own three values, kAhead tokens before their use: a wait for a
// block of staged loads cost 2 to 3 us per 16 tokens, as much as the arithmetic.
//
// PIECES, MEET: most recurrences forget where they started, and then a chunk need not be one chain.  PIECES takes it in m.pieces
// pieces, one workgroup each: the first starts from the state before the chunk, every other one from zero kWarmUp tokens before its
// own (grid [sequences][pieces]).  What that costs is what is left, behind the kWarmUp tokens, of the state they should have started
// from.  It is not looked for in the states themselves, where it would have to stand out from their rounding (two runs of one chain
// that differ in the last place of one state stay 2e-7 apart, and units that hardly forget can lose less than that at every joint):
// the derivative of the state carries a vector of +-1 from the first token of the warm-up to the last, in the fourth column of the
// matrix operand.  A piece stands if no unit keeps more than kForget = 2^-24 of it, half a unit in the last place; any other one
// ends there.
// MEET, one workgroup per sequence, also compares the state with which each piece began with the one in which the piece before it
// ended: with no more than kMeet between them in any unit they are one chain, but for rounding.  Where a piece began elsewhere the
// tokens are worked through again from the true state until it meets the one that is there, which costs what the chain costs.  A
// piece that ended early says so, and so does one that is through where the next has said nothing yet: the later of the two goes on,
// through the tokens of the piece that ended early, from the state the one before it left (none waits for another).  So the result
// never hangs on how fast the recurrence forgets, only the time does; a sequence half of whose chunk was not done in pieces takes its
// later chunks as one chain at once.  Error against 64 bits (2-norm, prompts of 200 to 1024
// tokens, update gates as drawn and opened by 0.3, 0.5, 0.65): z 1.06e-7 to 1.54e-7 as one chain, 1.08e-7 to 1.48e-7 in pieces;
// from gates opened by 0.8 on, or with a few units that hardly forget, no piece stands and both are the same bits.
// 16 sequences, a chunk of 512 tokens: 187 -> 57 us (52 the pieces, 50 without the vector, 5 the meeting); where no piece stands 196.
// Inits, one chain / pieces: 16 prompts of 1024 610 / 375 us, 1 of 512 241 / 105, 64 of 2048 1110 / 840; of remembered prompts, one
// chain / pieces whose tokens are left to MEET / as it is: 610 / 681 / 633, 241 / 276 / 247, 1110 / 1220 / 1190.
enum { WHOLE = 0, PIECES = 1, MEET = 2 };
constexpr int kWarmUp = 64, kMinPiece = 32, kMaxPieces = 14;
constexpr float kMeet = 0x1p-21f, kForget = 0x1p-24f;
struct ScanPieces {
  int pieces, len;             // tokens of every piece but the first, which has what is left, and the last, which has nsteps % 8 more
  float *guess;                // [B][pieces][128] the state a piece began with, unless it ended early
  int *alone;                  // [B] this sequence does not forget; 0 before the prompt's first chunk
  int *said;                   // [B][kMaxPieces] what is known at the joint in front of a piece (bits below); 0 before every chunk
};
enum { LEFT = 1, EARLY = 2, STANDS = 4 };   // the one before it is through, its state in memory; it ended before its first token; it goes on itself

template <bool SPLIT, int PART>
__global__ __launch_bounds__(256, 2) void ctrl_scan128_mfma_kernel(const CellArgs a, float *__restrict__ zseq, const ScanPieces m) {
  __builtin_amdgcn_s_setprio(3);   // a serial chain that may share its compute unit with the scoring of the chunk before
  constexpr int DP = 128, kAhead = 8;
  constexpr int TB = 16, GPT = TB * (3 * DP / 4) / 256;    // SPLIT: tokens per block; float4 per thread
  constexpr int SPS = DP + 32;                             // distance between two terms: 16 lanes' reads hit 64 different banks
  __shared__ __attribute__((aligned(16))) uint16_t sp[2][4 * SPS];   // z as bf16 terms, of two tokens in turn
  __shared__ float4 gbuf[SPLIT ? 2 : 1][SPLIT ? TB * (3 * DP / 4) : 1];   // input pre-activations of two blocks of tokens
  __shared__ int s_meet[4];                             // what the waves found
  __shared__ int s_joint;                               // PIECES: what is known at a joint
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane & 15, g = lane >> 4;
  // this lane's unit: register c / 4 of the rows 4g .. 4g+3 of the half c % 2 (lanes with c & 2 repeat it)
  const int unit = wave * 32 + (c & 1) * 16 + 4 * g + (c >> 2);
  const int len0 = PART == WHOLE ? a.nsteps : (a.nsteps & ~7) - (m.pieces - 1) * m.len;   // tokens of the first piece
  float *zrow = zseq + size_t(b) * a.nsteps * 128 + unit;
  int begin = 0, end = a.nsteps, keep = 0;                 // tokens to go through; those from `keep` on are its own
  uint32_t apart = 0, slow = 0;                            // MEET: pieces (bits) that did not begin where the one before ended; that ended early
  if constexpr (PART == PIECES) {
    const int j = blockIdx.y;
    const bool alone = m.alone[b] != 0;
    if (j > 0 && alone) return;
    keep = j == 0 ? 0 : len0 + (j - 1) * m.len;
    begin = j == 0 ? 0 : keep - kWarmUp;
    end = alone || j == m.pieces - 1 ? a.nsteps : len0 + j * m.len;
  }
  if constexpr (PART == MEET) {
    const bool alone = m.alone[b] != 0;   // its first piece was the whole chunk
    if (!alone) {
      float was[kMaxPieces], is[kMaxPieces];
      int said[kMaxPieces];
#pragma unroll
      for (int j = 1; j < kMaxPieces; ++j) {
        const int jj = min(j, m.pieces - 1);
        said[j] = m.said[b * kMaxPieces + jj];
        was[j] = m.guess[(size_t(b) * m.pieces + jj) * 128 + unit];
        is[j] = zrow[size_t(len0 + (jj - 1) * m.len - 1) * 128];
      }
      static_assert(kMaxPieces <= 16, "two masks in a word");
#pragma unroll
      for (int j = 1; j < kMaxPieces; ++j) {
        if (j < m.pieces) apart |= said[j] & EARLY ? 0x10000u << j : !(fabsf(was[j] - is[j]) <= kMeet) ? 1u << j : 0u;
      }
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) apart |= __shfl_xor(apart, off, 64);
      if (lane == 0) s_meet[wave] = int(apart);
      __syncthreads();
      apart = uint32_t(s_meet[0] | s_meet[1] | s_meet[2] | s_meet[3]);
      __syncthreads();
      if (tid < kMaxPieces) m.said[b * kMaxPieces + tid] = 0;
    }
    apart = __builtin_amdgcn_readfirstlane(apart);
    slow = apart >> 16;
    apart &= 0xffffu;
    if (apart == 0) {            // as a rule: all of them stand
      if ((c & 2) == 0) a.z[size_t(b) * 128 + unit] = zrow[size_t(a.nsteps - 1) * 128];
      if (tid == 0 && !alone) m.alone[b] = 2 * __builtin_popcount(slow) * m.len > a.nsteps;
      return;
    }
  }
  bf16x8 w[6][4];                                          // [gate * 2 + half of the wave's units][k-step]
#pragma unroll
  for (int t = 0; t < 6; ++t)
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int row = (t >> 1) * DP + wave * 32 + (t & 1) * 16 + c;
      w[t][s] = *reinterpret_cast<const bf16x8 *>(static_cast<const bf16_t *>(a.W_hh) + size_t(row) * DP + s * 32 + g * 8);
    }
  const bool odd = ((c >> 2) & 1) != 0, upper = (c >> 3) != 0, half1 = (c & 1) != 0, twin = (c & 2) != 0;
  const float b_r = a.b_ih[unit] + a.b_hh[unit];
  const float b_u = a.b_ih[DP + unit] + a.b_hh[DP + unit];
  const float b_in = a.b_ih[2 * DP + unit], b_hn = a.b_hh[2 * DP + unit];
  float hcur = PART == PIECES && blockIdx.y > 0 ? 0.f : a.z[size_t(b) * DP + unit];
  auto put_state = [&](uint16_t *dst) {   // the first term rounded down to 8 bits, the second the next 8, the third the rest
    const uint32_t hi = __float_as_uint(hcur) & 0xffff0000u;
    const float rest = hcur - __uint_as_float(hi);
    const uint32_t mid = __float_as_uint(rest) & 0xffff0000u;
    const float lo = rest - __uint_as_float(mid);
    dst[(twin ? SPS : 0) + unit] = uint16_t((twin ? mid : hi) >> 16);
    if (!twin) dst[2 * SPS + unit] = uint16_t(__float_as_uint(lo) >> 16);
  };
  int cur = 0;
  float along = PART == PIECES ? (uint32_t(unit) * 0x9e3779b1u >> 31 ? -1.f : 1.f) : 0.f;   // the vector that the derivative carries
  auto put_along = [&](uint16_t *dst) {
    if (twin) dst[3 * SPS + unit] = uint16_t(__float_as_uint(along) >> 16);   // (rounded down: 64 tokens take off an eighth of it)
  };
  // one token, from the state in sp[cur] to the state in sp[cur ^ 1]; the caller's barrier follows.  warm: of a warm-up, with the
  // vector and without the state's way out
  auto token = [&](auto warm_, int i, float g_r, float g_u, float g_n) {
    constexpr bool WARM = decltype(warm_)::value;
    bf16x8 hv[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) hv[s] = *reinterpret_cast<const bf16x8 *>(&sp[cur][(c & 3) * SPS + s * 32 + g * 8]);
    f32x4 acc[6];
#pragma unroll
    for (int t = 0; t < 6; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    // two gates' tiles side by side (no instruction waits for the one before it), the third's under the first gates' sums
#pragma unroll
    for (int s = 0; s < 4; ++s) {
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[t][s], hv[s], acc[t], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int t = 4; t < 6; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[t][s], hv[s], acc[t], 0, 0, 0);
    float sum[3], dsum[3] = {0.f, 0.f, 0.f};
#pragma unroll
    for (int gate = 0; gate < 3; ++gate) {
      float x[2], dx[2] = {0.f, 0.f};
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        const f32x4 v = acc[gate * 2 + hf];
        const float lo2 = odd ? v[1] : v[0], hi2 = odd ? v[3] : v[2];
        const float term = upper ? hi2 : lo2;
        if (WARM) dx[hf] = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(term), 0xFF, 0xf, 0xf, true));   // lane 3 of a quad
        x[hf] = quad_add<0x4E>(quad_add<0xB1>(term));   // lanes 0+1, 2+3 of a quad, then both
      }
      sum[gate] = half1 ? x[1] : x[0];
      if (WARM) {                // (where a piece stands, the vector is below the state's last place long before its own tokens)
        dsum[gate] = half1 ? dx[1] : dx[0];
        sum[gate] -= dsum[gate];
      }
    }
    const float r = scan_sigmoid(g_r + b_r + sum[0]);
    const float u = scan_sigmoid(g_u + b_u + sum[1]);
    const float cand = scan_tanh(g_n + b_in + r * (sum[2] + b_hn));
    if (WARM) {
      const float dr = r * (1.f - r) * dsum[0], du = u * (1.f - u) * dsum[1];
      const float dcand = (1.f - cand * cand) * (dr * (sum[2] + b_hn) + r * dsum[2]);
      along = u * along + (du * (hcur - cand) + (1.f - u) * dcand);
    }
    hcur = (1.0f - u) * cand + u * hcur;
    cur ^= 1;
    put_state(sp[cur]);
    if (WARM) put_along(sp[cur]);
    else if (!twin) zrow[size_t(i) * DP] = hcur;
  };
  constexpr std::false_type own = {};
  constexpr std::true_type warm_up = {};
  // Behind the warm-up: whether the piece goes on.
  auto forgot = [&]() {
    const uint64_t kept = __ballot(!(fabsf(along) <= kForget));
    if (lane == 0) s_meet[wave] = kept != 0;
    for (int i = tid; i < SPS; i += 256) sp[0][3 * SPS + i] = sp[1][3 * SPS + i] = 0;
    __syncthreads();
    const bool ok = (s_meet[0] | s_meet[1] | s_meet[2] | s_meet[3]) == 0;
    if (ok && !twin) m.guess[(size_t(b) * m.pieces + blockIdx.y) * DP + unit] = hcur;
    if (tid == 0) {
      const int known = __hip_atomic_fetch_or(m.said + b * kMaxPieces + blockIdx.y, ok ? STANDS : EARLY, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (!ok) s_joint = known & LEFT;   // (a word of its own: other waves may still be reading s_meet)
    }
    if (ok) return true;
    __syncthreads();
    if (s_joint == 0) return false;
    hcur = __hip_atomic_load(zrow + size_t(keep - 1) * DP, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    put_state(sp[cur]);
    __syncthreads();
    return true;
  };
  // At the end of a piece: whether to go on through those behind it; then `end` has moved.
  int done = PART == PIECES ? int(blockIdx.y) + 1 : 0;      // the first piece behind `end`
  auto goes_on = [&]() {
    if (PART != PIECES || end == a.nsteps) return false;
    int *said = m.said + b * kMaxPieces;
    if (wave == 0) {
      const int known = lane < m.pieces ? __hip_atomic_load(said + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
      const int more = __builtin_ctzll(~(__ballot(known & EARLY) >> done));
      if (lane == done) s_joint = more > 0 ? more : known & STANDS ? 0 : -1;
    }
    __syncthreads();
    int more = s_joint;
    if (more < 0) {              // nothing is known of the next one
      if (!twin) __hip_atomic_store(zrow + size_t(end - 1) * DP, hcur, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if (tid == 0) s_joint = __hip_atomic_fetch_or(said + done, LEFT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & EARLY ? 1 : 0;
      __syncthreads();
      more = s_joint;
    }
    __syncthreads();
    more = __builtin_amdgcn_readfirstlane(more);
    done += more;
    end = done == m.pieces ? a.nsteps : end + more * m.len;
    return more > 0;
  };
  const bool warms = PART == PIECES && keep > 0;           // uniform over the workgroup
  if (warms) put_along(sp[0]);
  else
    for (int i = tid; i < SPS; i += 256) sp[0][3 * SPS + i] = sp[1][3 * SPS + i] = 0;
  const float *gsrc = a.gi + size_t(b) * a.nsteps * (3 * DP) + unit;
  if constexpr (PART == MEET) {
    // from the first piece apart on, the tokens again, eight at a time, until the state met the one that is there or the one with which
    // the next piece began (never inside a piece that ended early, where there is none); then the next piece apart
    int again = __builtin_popcount(slow) * m.len;
    bool on = false;             // hcur is the true state behind token i - 1 (otherwise the one that is there stands)
    float pre[kAhead][3];
    auto ahead = [&](float (&v)[3], int i) {
      const float *p = gsrc + size_t(min(i, a.nsteps - 1)) * (3 * DP);
      v[0] = p[0]; v[1] = p[DP]; v[2] = p[2 * DP];
      if constexpr (SPLIT) {
        for (int k = 1; k < a.ksplit; ++k) {
          const float *q = p + size_t(k) * a.ntok * (3 * DP);
          v[0] += q[0]; v[1] += q[DP]; v[2] += q[2 * DP];
        }
      }
    };
    for (int i = 0; i < a.nsteps;) {             // uniform over the workgroup
      if (!on) {
        const int next = i < len0 ? 1 : (i - len0) / m.len + 2;   // the first piece that begins behind i
        const uint32_t rest = next < m.pieces ? apart >> next << next : 0u;
        if (rest == 0) break;
        i = len0 + (__builtin_ctz(rest) - 1) * m.len;
        hcur = zrow[size_t(i - 1) * DP];
        put_state(sp[cur]);
#pragma unroll
        for (int u = 0; u < kAhead; ++u) ahead(pre[u], i + u);
        __syncthreads();
        on = true;
      }
      const int count = min(kAhead, a.nsteps - i), to = i + count;
      // (pieces begin at multiples of eight)
      const int piece = to < len0 ? 0 : min((to - len0) / m.len + 1, m.pieces - 1);
      const bool joint = piece > 0 && to == len0 + (piece - 1) * m.len, may = to < a.nsteps && ((slow >> piece) & 1u) == 0;
      const float there = joint ? m.guess[(size_t(b) * m.pieces + piece) * DP + unit] : zrow[size_t(to - 1) * DP];
      if (count == kAhead) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
          token(own, i + u, pre[u][0], pre[u][1], pre[u][2]);
          ahead(pre[u], i + u + kAhead);
          __syncthreads();
        }
      } else {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
          if (u < count) {
            token(own, i + u, pre[u][0], pre[u][1], pre[u][2]);
            __syncthreads();
          }
        }
      }
      // (looked for at every token, with its own exchange: 0.55 us a token instead of 0.37)
      const uint64_t off = __ballot(!(fabsf(hcur - there) <= kMeet));
      if (lane == 0) s_meet[wave] = off != 0;
      __syncthreads();
      if (may && (s_meet[0] | s_meet[1] | s_meet[2] | s_meet[3]) == 0) on = false;
      __syncthreads();
      if (((slow >> (i < len0 ? 0 : min((i - len0) / m.len + 1, m.pieces - 1))) & 1u) == 0) again += count;
      i = to;
    }
    if (!on) hcur = zrow[size_t(a.nsteps - 1) * DP];
    if (tid == 0) m.alone[b] = again * 2 > a.nsteps;
  } else {
  put_state(sp[0]);
  if constexpr (SPLIT) {
    const float4 *gsrc4 = reinterpret_cast<const float4 *>(a.gi) + size_t(b) * a.nsteps * (3 * DP / 4);
    const size_t slice4 = size_t(a.ntok) * (3 * DP / 4);   // distance between two D-slices
    float4 stage[GPT];
    auto fetch = [&](int blk) {
      const int rows = min(end - begin - blk * TB, TB);
#pragma unroll
      for (int q = 0; q < GPT; ++q) {
        const int idx = tid + 256 * q;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (idx < rows * (3 * DP / 4)) {
          const float4 *p = gsrc4 + size_t(begin + blk * TB) * (3 * DP / 4) + idx;
          v = p[0];
          for (int k = 1; k < a.ksplit; ++k) {
            const float4 t = p[size_t(k) * slice4];
            v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w;
          }
        }
        stage[q] = v;
      }
    };
    auto park = [&](int buf) {
#pragma unroll
      for (int q = 0; q < GPT; ++q) gbuf[buf][tid + 256 * q] = stage[q];
    };
    auto block = [&](auto warm_, int blk, int nblk) {
      if (blk + 1 < nblk) fetch(blk + 1);
      const float *gt = reinterpret_cast<const float *>(gbuf[blk & 1]) + unit;
      const int rows = min(end - begin - blk * TB, TB);
      for (int ii = 0; ii < rows; ++ii, gt += 3 * DP) {
        token(warm_, begin + blk * TB + ii, gt[0], gt[DP], gt[2 * DP]);
        // the next block's rows: their buffer was last read a block ago, and they are read behind the barrier
        if (ii == rows - 1 && blk + 1 < nblk) park((blk + 1) & 1);
        __syncthreads();
      }
    };
    static_assert(kWarmUp % TB == 0 && kWarmUp % kAhead == 0, "a warm-up of whole blocks");
    do {
      const int nblk = (end - begin + TB - 1) / TB;
      int blk = 0;
      fetch(0);
      park(0);
      __syncthreads();
      if constexpr (PART == PIECES) {
        if (warms && begin < keep) {
          for (; blk < kWarmUp / TB; ++blk) block(warm_up, blk, nblk);
          if (!forgot()) return;
        }
      }
      for (; blk < nblk; ++blk) block(own, blk, nblk);
      begin = end;
    } while (goes_on());
  } else {
    float pre[kAhead][3];
    auto ahead = [&](float (&v)[3], int i) {
      const float *p = gsrc + size_t(min(i, a.nsteps - 1)) * (3 * DP);
      v[0] = p[0]; v[1] = p[DP]; v[2] = p[2 * DP];
    };
#pragma unroll
    for (int j = 0; j < kAhead; ++j) ahead(pre[j], begin + j);
    __syncthreads();
    int i0 = begin;
    auto eight = [&](auto warm_) {
#pragma unroll
      for (int j = 0; j < kAhead; ++j) {
        token(warm_, i0 + j, pre[j][0], pre[j][1], pre[j][2]);
        ahead(pre[j], i0 + j + kAhead);
        __syncthreads();
      }
      i0 += kAhead;
    };
    if constexpr (PART == PIECES) {
      if (warms) {
        for (int n = 0; n < kWarmUp / kAhead; ++n) eight(warm_up);
        if (!forgot()) return;
      }
    }
    do {
      while (i0 + kAhead <= end) eight(own);
    } while (goes_on());                    // (pieces end at multiples of eight, but for the last)
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      if (i0 + j < end) {                 // uniform over the workgroup
        token(own, i0 + j, pre[j][0], pre[j][1], pre[j][2]);
        __syncthreads();
      }
    }
  }
  }
  if (PART == PIECES) return;
  if (!twin) a.z[size_t(b) * DP + unit] = hcur;
}

// sigma_i = sigmoid(out_w . tanh(W_1 (p_i + z_i) + b_1) + out_b) for the tokens of a chunk, from the z_i the scan
// left.  grid (ceil(nsteps / 16), B), 4 waves, 4 tokens per wave; the arithmetic is the cell kernel's (rows_request,
// rows_finish, same order), so a token scored here and one scored by a step agree bit for bit given the same z_i.
// A wave multiplies each batch of 32 rows of W_1 by its four tokens: read once per token, the 64 KB of W_1 were what bound it
// (8192 tokens: 48 -> 23 us).
__global__ __launch_bounds__(256) void ctrl_mlp128_kernel(const CellArgs a, const float *__restrict__ zseq) {
  constexpr int DP = 128, TPW = 4;
  __shared__ float u1[4][TPW][DP];
  const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i0 = blockIdx.x * 16 + wave * TPW;
  float x0[TPW], x1[TPW];
#pragma unroll
  for (int q = 0; q < TPW; ++q) {
    const int i = i0 + q < a.nsteps ? i0 + q : 0;       // lanes past the end redo token 0 and store nothing
    const size_t tok = size_t(b) * a.nsteps + i;
    const float delta = a.cvec ? 0.f : float(a.pos0 + i) * a.pos_scale;   // rescore mode: distance to itself
    x0[q] = fmaf(a.pos_w[2 * lane], delta, a.pos_b[2 * lane]) + zseq[tok * DP + 2 * lane];
    x1[q] = fmaf(a.pos_w[2 * lane + 1], delta, a.pos_b[2 * lane + 1]) + zseq[tok * DP + 2 * lane + 1];
  }
#pragma unroll 1
  for (int part = 0; part < 4; ++part) {
    float2 raw[32];
    rows_request<float, 32>(a.W1, part * 32, lane, raw);
#pragma unroll
    for (int q = 0; q < TPW; ++q) rows_finish<float2, 32>(raw, part * 32, x0[q], x1[q], a.b1, u1[wave][q], lane);
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < TPW; ++q) {
    const int i = i0 + q;
    if (i >= a.nsteps) break;                           // uniform over the wave
    if (a.cvec) {
      float *c = a.cvec + (size_t(b) * a.N_max + a.pos0 + i) * DP;
      c[lane] = u1[wave][q][lane];
      c[lane + 64] = u1[wave][q][lane + 64];
    }
    float s = fmaf(a.out_w[lane], tanhf(u1[wave][q][lane]), a.out_w[lane + 64] * tanhf(u1[wave][q][lane + 64]));
    s = wave_sum(s);
    if (lane == 0) {
      float sig = sigmoidf_(s + a.out_b[0]);
      if (a.override_) sig = a.override_[size_t(b) * a.override_stride + i];
      a.score[size_t(b) * a.N_max + a.pos0 + i] = sig;
    }
  }
}

// ---- cell, any d' -------------------------------------------------------------------
// One workgroup per sequence; loops over `nsteps` consecutive tokens starting at position pos0.
template <typename T>
__global__ __launch_bounds__(512) void ctrl_cell_kernel(const CellArgs a) {
  __builtin_amdgcn_s_setprio(3);   // short, latency-bound work that shares compute units with the GEMM: its waves go first
  extern __shared__ float smem[];
  const int dp = a.dp;
  float *h = smem;            // [dp]   z_{i-1}, then z_i
  float *gh = h + dp;         // [3dp]  W_hh h
  float *t_in = gh + 3 * dp;  // [dp]   p_i + z_i
  float *hn = t_in + dp;      // [dp]   z_i before it replaces h
  float *red = hn + dp;       // [8]    per-wave partial sums of the output layer
  const int b = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nwaves = blockDim.x >> 6;
  const T *W_hh = static_cast<const T *>(a.W_hh);

  for (int j = tid; j < dp; j += blockDim.x) h[j] = a.z[size_t(b) * dp + j];
  __syncthreads();

  for (int i = 0; i < a.nsteps; ++i) {
    const size_t tok = size_t(b) * a.nsteps + i;
    // recurrent pre-activations: one wave per row, lanes along the row
    for (int row = wave; row < 3 * dp; row += nwaves) {
      float s = 0.f;
      for (int t = lane; t < dp; t += 64) s = fmaf(to_float(W_hh[size_t(row) * dp + t]), h[t], s);
      s = wave_sum(s);
      if (lane == 0) gh[row] = s + a.b_hh[row];
    }
    __syncthreads();
    const float delta = a.cvec ? 0.f : float(a.pos0 + i) * a.pos_scale;   // rescore mode: distance to itself
    for (int j = tid; j < dp; j += blockDim.x) {
      const float r = sigmoidf_(gi_sum(a, tok, j) + a.b_ih[j] + gh[j]);
      const float u = sigmoidf_(gi_sum(a, tok, dp + j) + a.b_ih[dp + j] + gh[dp + j]);
      const float cand = tanhf(gi_sum(a, tok, 2 * dp + j) + a.b_ih[2 * dp + j] + r * gh[2 * dp + j]);
      const float hnew = (1.0f - u) * cand + u * h[j];
      hn[j] = hnew;
      t_in[j] = fmaf(a.pos_w[j], delta, a.pos_b[j]) + hnew;
    }
    __syncthreads();
    for (int j = tid; j < dp; j += blockDim.x) h[j] = hn[j];
    // interaction layer: one wave per row; output layer folded in
    float part = 0.f;
    for (int row = wave; row < dp; row += nwaves) {
      float s = 0.f;
      for (int t = lane; t < dp; t += 64) s = fmaf(a.W1[size_t(row) * dp + t], t_in[t], s);
      s = wave_sum(s);
      if (a.cvec && lane == 0) a.cvec[(size_t(b) * a.N_max + a.pos0 + i) * dp + row] = s + a.b1[row];
      part = fmaf(a.out_w[row], tanhf(s + a.b1[row]), part);
    }
    if (lane == 0) red[wave] = part;
    __syncthreads();
    if (tid == 0) {
      float s = 0.f;
      for (int wv = 0; wv < nwaves; ++wv) s += red[wv];
      float sig = sigmoidf_(s + a.out_b[0]);
      if (a.override_) sig = a.override_[size_t(b) * a.override_stride + i];
      a.score[size_t(b) * a.N_max + a.pos0 + i] = sig;
    }
    __syncthreads();
  }
  for (int j = tid; j < dp; j += blockDim.x) a.z[size_t(b) * dp + j] = h[j];
}

// ---- rescore mode -----------------------------------------------------------------
// W_1 (pos_w * delta + pos_b + z_i) + b_1  =  c_i + delta * a   with  c_i = W_1 (z_i + pos_b) + b_1  kept per
// token by the cell kernels and  a = W_1 pos_w:  scoring a token again costs d' tanh and one dot product.
__global__ __launch_bounds__(256) void ctrl_avec_kernel(const float *__restrict__ W1,
                                                        const float *__restrict__ pos_w,
                                                        float *__restrict__ avec, int dp) {
  for (int row = threadIdx.x; row < dp; row += blockDim.x) {
    float s = 0.f;
    for (int k = 0; k < dp; ++k) s = fmaf(W1[size_t(row) * dp + k], pos_w[k], s);
    avec[row] = s;
  }
}

// sigma_i(n) = sigmoid(out_w . tanh(c_i + (n - i) * pos_scale * a) + out_b) for i = 0..upto.  16 lanes per
// token, 16 tokens per workgroup; grid = (tokens / 16, B).  In a step upto = n - 1: the current token's score (distance
// 0) is the cell kernel's, which runs next to this one.
__global__ __launch_bounds__(256) void rescore_kernel(const float *__restrict__ cvec,
                                                      const float *__restrict__ avec,
                                                      const float *__restrict__ out_w,
                                                      const float *__restrict__ out_b,
                                                      float *__restrict__ score, int n, int upto, int N_max,
                                                      int dp, float pos_scale) {
  __builtin_amdgcn_s_setprio(3);   // short, latency-bound work that shares compute units with the GEMM: its waves go first
  const int b = blockIdx.y;
  const int i = blockIdx.x * 16 + (threadIdx.x >> 4);
  const int lig = threadIdx.x & 15;
  const int ic = i <= upto ? i : upto;           // lanes past the end redo the last token and store nothing
  const float delta = float(n - ic) * pos_scale;
  const float *c = cvec + (size_t(b) * N_max + ic) * dp;
  float s = 0.f;
  for (int e = lig * 4; e < dp; e += 64) {
    const float4 cv = *reinterpret_cast<const float4 *>(c + e);
    const float4 av = *reinterpret_cast<const float4 *>(avec + e);
    const float4 wv = *reinterpret_cast<const float4 *>(out_w + e);
    s = fmaf(wv.x, tanhf(fmaf(delta, av.x, cv.x)), s);
    s = fmaf(wv.y, tanhf(fmaf(delta, av.y, cv.y)), s);
    s = fmaf(wv.z, tanhf(fmaf(delta, av.z, cv.z)), s);
    s = fmaf(wv.w, tanhf(fmaf(delta, av.w, cv.w)), s);
  }
  s = group_sum<16>(s);
  if (lig == 0 && i <= upto) score[size_t(b) * N_max + i] = sigmoidf_(s + out_b[0]);
}

// Number of D-slices of the bf16 input projection: enough workgroups to cover the chip when
// there are few tokens, and slices short enough that a wave walks at most four 32-wide steps of its quarter (the
// operand loads of a step touch 64 cache lines and wait for each other: at 128 tokens, two slices of 2048 took
// 225 us); one slice when there are many tokens.  A slice is a multiple of 128 (4 waves x 32).
// rows: what the copy of the pre-activations holds (ntok per slice).
int ctrl_input_ksplit(const adore_config &c, int ntok, size_t rows) {
  const int tiles = ((3 * c.ctrl_hidden + 15) / 16) * ((ntok + 15) / 16);
  int ks = 1;
  if (ntok > kCtrlSplitTokens) return 1;
  while (ks < kMaxCtrlSplit && (tiles * ks < 256 || c.hidden / ks > 512) && c.hidden % (ks * 2 * 128) == 0 &&
         size_t(ks) * 2 * ntok <= rows)
    ks *= 2;
  return ks;
}

// fp32: a tile of 16 tokens x 16 rows walks all of D in one workgroup, whose time is the row's (4.3, 5.7, 7.9, 11.7, 18.5 us
// at D = 256, 512, 1024, 2048, 4096) until there are more tiles than compute units; the plain kernel's grows with the outputs.
// Plain / tiles at d' = 128: D = 256, 16 tokens 5.7 / 5.7 us; 512, 32: 6.7 / 5.6; 1024, 32: 6.5 / 7.8, 96: 8.5 / 8.5, 256: 14.4 / 11.2;
// 2048, 64: 9.2 / 11.6, 128: 12.2 / 12.5, 256: 19.4 / 18.6; 4096, 16: 10.3 / 18.3, 128: 20.1 / 20.3, 256: 33.7 / 33.6.  d' = 64 and 512 turn
// at the same number of outputs.
bool input_on_tiles(const adore_config &c, int ntok) { return ntok >= 16 && (long long)ntok * 3 * c.ctrl_hidden >= 24LL * c.hidden; }

}  // namespace

// buf: which copy of the pre-activations is written (a prompt's chunks take them in turn), rows: how many it has room for.
hipError_t launch_ctrl_input(adore_ctx *ctx, hipStream_t st, const void *x, int ntok, int per_seq,
                             int seq_rows, int buf, size_t rows, int *ksplit_out) {
  const adore_config &c = ctx->cfg;
  const int G3 = 3 * c.ctrl_hidden;
  float *gi = ctx->gi[buf];
  ScopedTimer t(ctx, ADORE_KERNEL_CTRL_INPUT, st);
  *ksplit_out = 1;
  const bool tiled = c.dtype == ADORE_BF16 ? ntok > kCtrlSplitTokens : input_on_tiles(c, ntok);
  if (tiled &&
      launch_plain_projection(ctx, t, st, x, ctx->w.gru_w_ih, gi, ntok, per_seq, seq_rows, G3, c.hidden)) {
    // a prompt chunk on the rebuild's 128x128 tile (3d' a multiple of 128, D of 64)
  } else if (c.dtype == ADORE_BF16 && c.hidden % 128 == 0 && ntok > kCtrlSplitTokens) {
    dim3 grid((G3 + 63) / 64, (ntok + 63) / 64);
    ADORE_LAUNCH(t, ctrl_input_prompt_kernel, grid, dim3(256), 0, st,
                       static_cast<const bf16_t *>(ctx->w.gru_w_ih), static_cast<const bf16_t *>(x), gi,
                       c.hidden, G3, ntok, per_seq, seq_rows);
  } else if (c.dtype == ADORE_BF16 && c.hidden % 128 == 0) {
    const int ks = ctrl_input_ksplit(c, ntok, rows);
    if (size_t(ks) * ntok > rows) return hipErrorInvalidValue;
    *ksplit_out = ks;
    dim3 grid((G3 + 15) / 16, (ntok + 15) / 16, ks);
    ADORE_LAUNCH(t, ctrl_input_mfma_kernel, grid, dim3(256), 0, st,
                       static_cast<const bf16_t *>(ctx->w.gru_w_ih), static_cast<const bf16_t *>(x), gi,
                       c.hidden, G3, ntok, per_seq, seq_rows, c.hidden / ks);
  } else if (c.dtype == ADORE_BF16) {
    dim3 grid((G3 + JT - 1) / JT, (ntok + NB - 1) / NB);
    ADORE_LAUNCH(t, (ctrl_input_kernel<bf16_t>), grid, dim3(256), 0, st,
                       static_cast<const bf16_t *>(ctx->w.gru_w_ih), static_cast<const bf16_t *>(x), gi,
                       c.hidden, G3, ntok, per_seq, seq_rows);
  } else {
    dim3 grid((G3 + JT - 1) / JT, (ntok + NB - 1) / NB);
    ADORE_LAUNCH(t, (ctrl_input_kernel<float>), grid, dim3(256), 0, st,
                       static_cast<const float *>(ctx->w.gru_w_ih), static_cast<const float *>(x), gi,
                       c.hidden, G3, ntok, per_seq, seq_rows);
  }
  return hipGetLastError();
}

namespace {

CellArgs cell_args(adore_ctx *ctx, int nsteps, int pos0, const float *score_override, int override_stride, int buf, int ksplit) {
  const adore_config &c = ctx->cfg;
  CellArgs a;
  a.W_hh = ctx->w.gru_w_hh;
  a.b_ih = ctx->w.gru_b_ih; a.b_hh = ctx->w.gru_b_hh;
  a.pos_w = ctx->w.pos_w; a.pos_b = ctx->w.pos_b;
  a.W1 = ctx->w.mlp_w1; a.b1 = ctx->w.mlp_b1;
  a.out_w = ctx->w.out_w; a.out_b = ctx->w.out_b;
  a.gi = ctx->gi[buf]; a.z = ctx->z; a.score = ctx->score;
  a.cvec = c.score_mode == ADORE_SCORE_RESCORE ? ctx->cvec : nullptr;
  a.override_ = score_override; a.override_stride = override_stride;
  a.dp = c.ctrl_hidden; a.nsteps = nsteps; a.pos0 = pos0; a.N_max = c.max_positions;
  a.ksplit = ksplit; a.ntok = c.batch * nsteps;
  a.pos_scale = c.pos_scale;
  return a;
}

}  // namespace

// A chunk of several tokens at d' = 128 is two launches, of which only the first has to wait for the chunk before it.
bool ctrl_chunk_in_two(const adore_config &c, int nsteps) { return c.ctrl_hidden == 128 && nsteps > 1; }

// What a prompt starts from: states of zero, and nothing known of any sequence or piece (see ScanPieces).
__global__ void ctrl_start_kernel(float *z, int n_z, int *words, int n_words) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_z) z[i] = 0.f;
  if (i < n_words) words[i] = 0;
}

// In how many pieces a chunk's recurrence is worked through (bf16): as many as keep two workgroups a compute unit, of at least
// kMinPiece tokens; 1: as one chain (two launches cost 5 us more than one, 14 tokens).
int scan_pieces(const adore_config &c, int nsteps) {
  const int most = std::min(kMaxPieces, (c.heads * kMaxSplits * (c.head_dim + 2) - kMaxPieces - 1) / 128);   // (what the attention's partials have room for)
  const char *whole = getenv("ADORE_NO_PIECES");       // comparison runs
  if (whole && atoi(whole) != 0) return 1;
  const int n = std::min({most, 512 / c.batch, (nsteps - kWarmUp) / kMinPiece});
  return n >= 2 && nsteps - kWarmUp - (nsteps - kWarmUp) / n > 32 ? n : 1;
}

hipError_t launch_ctrl_start(adore_ctx *ctx) {
  const int B = ctx->cfg.batch, n_z = B * ctx->cfg.ctrl_hidden, n_words = B * (kMaxPieces + 1);
  hipLaunchKernelGGL(ctrl_start_kernel, dim3((std::max(n_z, n_words) + 255) / 256), dim3(256), 0, ctx->stream, ctx->z, n_z,
                     reinterpret_cast<int *>(ctx->att_part), n_words);
  return hipGetLastError();
}

hipError_t launch_ctrl_scan(adore_ctx *ctx, hipStream_t st, int nsteps, int buf, int ksplit) {
  const adore_config &c = ctx->cfg;
  const CellArgs a = cell_args(ctx, nsteps, 0, nullptr, 0, buf, ksplit);
  ScopedTimer t(ctx, ADORE_KERNEL_CTRL_CELL, st);
  float *zseq = ctx->zseq[buf];
  ScanPieces m = {};
  if (c.dtype != ADORE_BF16) {
    ADORE_LAUNCH(t, (ctrl_scan128_kernel<float>), dim3(c.batch), dim3(256), 0, st, a, zseq);
    return hipGetLastError();
  }
  m.pieces = scan_pieces(c, nsteps);
  if (m.pieces == 1) {
    if (ksplit > 1)
      ADORE_LAUNCH(t, (ctrl_scan128_mfma_kernel<true, WHOLE>), dim3(c.batch), dim3(256), 0, st, a, zseq, m);
    else
      ADORE_LAUNCH(t, (ctrl_scan128_mfma_kernel<false, WHOLE>), dim3(c.batch), dim3(256), 0, st, a, zseq, m);
    return hipGetLastError();
  }
  m.len = (nsteps - kWarmUp) / m.pieces & ~7;
  m.alone = reinterpret_cast<int *>(ctx->att_part);   // no attention runs before the init is through
  m.said = m.alone + c.batch;
  m.guess = ctx->att_part + size_t(c.batch) * (kMaxPieces + 1);
  if (ksplit > 1)
    ADORE_LAUNCH(t, (ctrl_scan128_mfma_kernel<true, PIECES>), dim3(c.batch, m.pieces), dim3(256), 0, st, a, zseq, m);
  else
    ADORE_LAUNCH(t, (ctrl_scan128_mfma_kernel<false, PIECES>), dim3(c.batch, m.pieces), dim3(256), 0, st, a, zseq, m);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  ScopedTimer tm(ctx, ADORE_KERNEL_CTRL_CELL, st);
  if (ksplit > 1)
    ADORE_LAUNCH(tm, (ctrl_scan128_mfma_kernel<true, MEET>), dim3(c.batch), dim3(256), 0, st, a, zseq, m);
  else
    ADORE_LAUNCH(tm, (ctrl_scan128_mfma_kernel<false, MEET>), dim3(c.batch), dim3(256), 0, st, a, zseq, m);
  return hipGetLastError();
}

hipError_t launch_ctrl_score(adore_ctx *ctx, hipStream_t st, int nsteps, int pos0, const float *score_override,
                             int override_stride, int buf) {
  const adore_config &c = ctx->cfg;
  const CellArgs a = cell_args(ctx, nsteps, pos0, score_override, override_stride, buf, 1);
  ScopedTimer t(ctx, ADORE_KERNEL_CTRL_CELL, st);
  ADORE_LAUNCH(t, ctrl_mlp128_kernel, dim3((nsteps + 15) / 16, c.batch), dim3(256), 0, st, a,
               static_cast<const float *>(ctx->zseq[buf]));
  return hipGetLastError();
}

hipError_t launch_ctrl_cell(adore_ctx *ctx, hipStream_t st, int nsteps, int pos0,
                            const float *score_override, int override_stride, int buf, int ksplit) {
  const adore_config &c = ctx->cfg;
  const CellArgs a = cell_args(ctx, nsteps, pos0, score_override, override_stride, buf, ksplit);
  ScopedTimer t(ctx, ADORE_KERNEL_CTRL_CELL, st);
  if (c.ctrl_hidden == 128 && nsteps == 1) {
    if (c.dtype == ADORE_BF16) {
      ADORE_LAUNCH(t, (ctrl_cell128_kernel<bf16_t>), dim3(c.batch), dim3(768), 0, st, a);
    } else {
      ADORE_LAUNCH(t, (ctrl_cell128_kernel<float>), dim3(c.batch), dim3(768), 0, st, a);
    }
  } else {
    const size_t smem = size_t(6 * c.ctrl_hidden + 8) * sizeof(float);
    if (c.dtype == ADORE_BF16) {
      ADORE_LAUNCH(t, (ctrl_cell_kernel<bf16_t>), dim3(c.batch), dim3(512), smem, st, a);
    } else {
      ADORE_LAUNCH(t, (ctrl_cell_kernel<float>), dim3(c.batch), dim3(512), smem, st, a);
    }
  }
  return hipGetLastError();
}

// Whether the controller of a step can ride in the step's other launches, and its two parts.
bool step_ctrl_supported(const adore_config &c) {
  return c.ctrl_hidden == 128 && (c.dtype == ADORE_F32 ? !input_on_tiles(c, c.batch) : c.batch <= kCtrlSplitTokens);
}

void fill_step_ctrl(adore_ctx *ctx, const void *x, int pos, const float *score_override, StepCtrl &s, StepTail &t) {
  const adore_config &c = ctx->cfg;
  const int G3 = 3 * c.ctrl_hidden;
  const bool mfma = c.dtype == ADORE_BF16 && c.hidden % 128 == 0;
  // behind the slices of the pre-activations there is room for B more rows
  const int ks = mfma ? ctrl_input_ksplit(c, c.batch, ctx->gi_rows[0] - c.batch) : 1;
  s.kslice = mfma ? c.hidden / ks : 0;
  s.tiles_j = mfma ? (G3 + 15) / 16 : (G3 + JT - 1) / JT;
  s.tiles_t = mfma ? (c.batch + 15) / 16 : (c.batch + NB - 1) / NB;
  s.n_in = s.tiles_j * s.tiles_t * ks;
  s.n = s.n_in + 6 * c.batch;
  s.W_ih = ctx->w.gru_w_ih; s.x = x; s.W_hh = ctx->w.gru_w_hh;
  s.z = ctx->z; s.b_hh = ctx->w.gru_b_hh;
  s.gi = ctx->gi[0]; s.gh = ctx->gi[0] + size_t(ks) * c.batch * G3;
  s.D = c.hidden; s.B = c.batch; s.seq_rows = 1;
  t.cell = cell_args(ctx, 1, pos, score_override, 1, 0, ks);
  t.gh = s.gh;
  t.n_cell = c.batch;
  t.rows = 0;
}

hipError_t launch_ctrl_avec(adore_ctx *ctx, hipStream_t st) {
  hipLaunchKernelGGL(ctrl_avec_kernel, dim3(1), dim3(256), 0, st, ctx->w.mlp_w1, ctx->w.pos_w, ctx->avec,
                     ctx->cfg.ctrl_hidden);
  return hipGetLastError();
}

hipError_t launch_rescore(adore_ctx *ctx, hipStream_t st, int n, int upto) {
  const adore_config &c = ctx->cfg;
  if (upto < 0) return hipSuccess;
  ScopedTimer t(ctx, ADORE_KERNEL_RESCORE, st);
  ADORE_LAUNCH(t, rescore_kernel, dim3((upto + 16) / 16, c.batch), dim3(256), 0, st, ctx->cvec, ctx->avec,
               ctx->w.out_w, ctx->w.out_b, ctx->score, n, upto, c.max_positions, c.ctrl_hidden, c.pos_scale);
  return hipGetLastError();
}

}  // namespace adore
