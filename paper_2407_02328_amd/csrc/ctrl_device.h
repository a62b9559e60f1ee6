// Device code of the controller that more than one launch carries: the input projection of a step's tokens, the recurrent
// product, and the cell with the layers above it (kernels of their own in controller.hip; extra workgroups of the attention's
// and the projection's launches where a step is short, see StepCtrl).
#pragma once

#include "device_utils.h"

namespace adore {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// ---- input projection, bf16, matrix cores -----------------------------------------
// 256 threads own the 16-token x 16-row tile (tt, jt) and the D-slice z; the 4 waves cut the slice again and are summed
// through LDS (red: kInputTileLds floats).
// Inside a wave, lane group g = lane/16 walks the g-th quarter of the wave's k-range in
// 16-byte steps (both operands use the same assignment, so the order of k does not matter).
// part[z][tok][j] = sum over the slice of W_ih[j][k] * x_tok[k].
constexpr int kInputTileLds = 4 * 16 * 17;
__device__ __forceinline__ void ctrl_input_mfma_tile(const bf16_t *__restrict__ W_ih, const bf16_t *__restrict__ x,
                                            float *__restrict__ part, int D, int G3, int ntok, int per_seq, int seq_rows,
                                            int kslice, int jt, int tt, int z, float *lds) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int j0 = jt * 16, t0 = tt * 16;
  const int kw = kslice / 4;                       // k-range of one wave, a multiple of 32
  const int kbeg = z * kslice + wave * kw + (lane >> 4) * (kw / 4);
  int tok = t0 + (lane & 15);
  if (tok >= ntok) tok = ntok - 1;                 // padded rows read a valid token; dropped at the store
  const size_t xrow = size_t(tok / per_seq) * seq_rows + tok % per_seq;
  int j = j0 + (lane & 15);
  if (j >= G3) j = G3 - 1;
  const u32x4 *pa = reinterpret_cast<const u32x4 *>(x + xrow * D + kbeg);
  const u32x4 *pb = reinterpret_cast<const u32x4 *>(W_ih + size_t(j) * D + kbeg);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  const int steps = kw / 32;                       // each MFMA consumes 32 k: 8 per lane group
  for (int s = 0; s < steps; ++s) {
    const u32x4 va = pa[s], vb = pb[s];
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8 *>(&va),
                                                  *reinterpret_cast<const bf16x8 *>(&vb), acc, 0, 0, 0);
  }
  // accumulator element v of lane L: token 4*(L/16) + v, gate row L%16
  float (*red)[16][17] = reinterpret_cast<float (*)[16][17]>(lds);
#pragma unroll
  for (int v = 0; v < 4; ++v) red[wave][4 * (lane >> 4) + v][lane & 15] = acc[v];
  __syncthreads();
  {
    const int m = tid >> 4, nn = tid & 15;
    if (t0 + m < ntok && j0 + nn < G3) {
      const float s = (red[0][m][nn] + red[1][m][nn]) + (red[2][m][nn] + red[3][m][nn]);
      part[(size_t(z) * ntok + t0 + m) * G3 + j0 + nn] = s;
    }
  }
}

// Sums over a wave of a batch of rows at once: at every halving step a lane keeps one half of its partial sums and hands the
// other half to its partner, so N rows cost N-1 exchanges instead of 6N.
// v[i] is this lane's partial sum of row i.  Returns, in every lane, the complete sum of row
// lane / (64 / N).
template <int N, int OFF>
struct ReduceRows {
  __device__ static __forceinline__ float run(float (&v)[N], int lane) {
    float w[N / 2];
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
      const uint32_t lo = __float_as_uint(v[i]), hi = __float_as_uint(v[i + N / 2]);
      if constexpr (OFF == 32) {
        const auto s = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
        w[i] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
      } else if constexpr (OFF == 16) {
        const auto s = __builtin_amdgcn_permlane16_swap(lo, hi, false, false);
        w[i] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
      } else {
        const bool upper = (lane & OFF) != 0;
        const float a = add_lane_xor<OFF>(v[i]), b = add_lane_xor<OFF>(v[i + N / 2]);
        w[i] = upper ? b : a;
      }
    }
    return ReduceRows<N / 2, OFF / 2>::run(w, lane);
  }
};
template <int OFF>
struct ReduceRows<1, OFF> {
  __device__ static __forceinline__ float run(float (&v)[1], int) {
    return group_sum<2 * OFF>(v[0]);
  }
};
template <int N>
__device__ __forceinline__ float reduce_rows(float (&v)[N], int lane) {
  return ReduceRows<N, 32>::run(v, lane);
}

// ---- input projection, any storage type, plain ALUs ---------------------------------
constexpr int JT = 4;  // gate rows per 256 threads
constexpr int NB = 8;  // tokens per 256 threads

// gi[tok][j] = sum_t W_ih[j][t] * x_tok[t]       (bias added in the cell kernel)
// Token tok = b * per_seq + i reads the row x[(b * seq_rows + i) * D].
template <typename T>
__device__ __forceinline__ void ctrl_input_plain_tile(const T *__restrict__ W_ih, const T *__restrict__ x, float *__restrict__ gi, int D,
                                             int G3, int ntok, int per_seq, int seq_rows, int jt, int tt, float *lds) {
  constexpr int EPL = Vec16<T>::EPL;
  const int j0 = jt * JT;
  const int t0 = tt * NB;
  const int tid = threadIdx.x;
  float acc[JT][NB];
#pragma unroll
  for (int jj = 0; jj < JT; ++jj)
#pragma unroll
    for (int tt = 0; tt < NB; ++tt) acc[jj][tt] = 0.f;

  for (int c = tid * EPL; c < D; c += 256 * EPL) {
    float wf[JT][EPL];
#pragma unroll
    for (int jj = 0; jj < JT; ++jj) {
      if (j0 + jj < G3) {
        Vec16<T>::load(W_ih + size_t(j0 + jj) * D + c, wf[jj]);
      } else {
#pragma unroll
        for (int e = 0; e < EPL; ++e) wf[jj][e] = 0.f;
      }
    }
#pragma unroll
    for (int tt = 0; tt < NB; ++tt) {
      if (t0 + tt < ntok) {
        float xf[EPL];
        const int tok = t0 + tt;
        const size_t row = size_t(tok / per_seq) * seq_rows + tok % per_seq;
        Vec16<T>::load(x + row * D + c, xf);
#pragma unroll
        for (int jj = 0; jj < JT; ++jj)
#pragma unroll
          for (int e = 0; e < EPL; ++e) acc[jj][tt] = fmaf(wf[jj][e], xf[e], acc[jj][tt]);
      }
    }
  }
  float (*red)[JT][NB] = reinterpret_cast<float (*)[JT][NB]>(lds);
  const int wave = tid >> 6, lane = tid & 63;
  // (one sum at a time, 192 shuffles, was a quarter of a decode step's launch)
  const float s = reduce_rows<JT * NB>(reinterpret_cast<float (&)[JT * NB]>(acc), lane);
  if ((lane & 1) == 0) red[wave][lane / 2 / NB][lane / 2 % NB] = s;
  __syncthreads();
  if (tid < JT * NB) {
    const int jj = tid / NB, tt = tid % NB;
    if (j0 + jj < G3 && t0 + tt < ntok) {
      gi[size_t(t0 + tt) * G3 + j0 + jj] = (red[0][jj][tt] + red[1][jj][tt]) + (red[2][jj][tt] + red[3][jj][tt]);
    }
  }
}

__device__ __forceinline__ float sigmoidf_(float a) { return 1.0f / (1.0f + expf(-a)); }

struct CellArgs {
  const void *W_hh;            // [3d'][d'] storage type
  const float *b_ih, *b_hh;    // [3d']
  const float *pos_w, *pos_b, *W1, *b1, *out_w, *out_b;
  const float *gi;             // [ksplit][B*nsteps][3d'], token (b, i) at row b*nsteps + i
  float *z;                    // [B][d']
  float *score;                // [B][N_max]
  float *cvec;                 // rescore mode: [B][N_max][d'] interaction-layer pre-activation at distance 0; else null
  const float *override_;      // [B][override_stride] or null
  int override_stride;
  int dp, nsteps, pos0, N_max, ksplit, ntok;
  float pos_scale;
};

// sum of the D-slices of one input pre-activation, in slice order; loads go out eight at a time
__device__ __forceinline__ float gi_sum(const CellArgs &a, size_t tok, int j) {
  const size_t stride = size_t(a.ntok) * 3 * a.dp;
  const float *p = a.gi + tok * 3 * a.dp + j;
  float s = 0.f;
  int k = 0;
  for (; k + 16 <= a.ksplit; k += 16) {   // (sixteen at a time where there are that many: one trip to memory, same order)
    float v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = p[size_t(k + u) * stride];
#pragma unroll
    for (int u = 0; u < 16; ++u) s += v[u];
  }
  for (; k + 8 <= a.ksplit; k += 8) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = p[size_t(k + u) * stride];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += v[u];
  }
  for (; k < a.ksplit; ++k) s += p[size_t(k) * stride];
  return s;
}

// ---- cell, d' = 128 --------------------------------------------------------------------
// A weight row of 128 elements is one coalesced wave load
// (two elements per lane); a wave multiplies a batch of rows by the state it holds in registers and
// reduces the whole batch at once: at every halving step a lane keeps one half of its partial sums
// and hands the other half to its partner, so N rows cost N-1 exchanges instead of 6N.

// two consecutive elements of a weight row, raw, and their conversion
__device__ __forceinline__ uint32_t load_raw2(const bf16_t *p) { return *reinterpret_cast<const uint32_t *>(p); }
__device__ __forceinline__ float2 load_raw2(const float *p) { return *reinterpret_cast<const float2 *>(p); }
__device__ __forceinline__ float dot2(uint32_t u, float x0, float x1) {
  return fmaf(__uint_as_float(u << 16), x0, __uint_as_float(u & 0xffff0000u) * x1);
}
__device__ __forceinline__ float dot2(float2 u, float x0, float x1) { return fmaf(u.x, x0, u.y * x1); }

// out[row0 + r] = bias[row0 + r] + W[row0 + r][:] . x   for r < N, x held as (x0, x1) = x[2*lane], x[2*lane+1], in two
// halves: the N row loads go out where the caller wants them (next to everything else a step reads), the arithmetic follows
// once x is known.
template <typename T, int N>
__device__ __forceinline__ void rows_request(const T *W, int row0, int lane, decltype(load_raw2(W)) (&raw)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) raw[i] = load_raw2(W + size_t(row0 + i) * 128 + 2 * lane);
}
template <typename R, int N>
__device__ __forceinline__ void rows_finish(const R (&raw)[N], int row0, float x0, float x1, const float *bias, float *out, int lane) {
  float v[N];
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = dot2(raw[i], x0, x1);
  const float s = reduce_rows<N>(v, lane);
  constexpr int LPRW = 64 / N;   // lanes holding the same row
  if ((lane & (LPRW - 1)) == 0) {
    const int r = row0 + lane / LPRW;
    out[r] = s + bias[r];
  }
}


// ---- merge of the attention's splits: element e of row bh ---------------------------------------
// part: [rows][nsplit][d + 2] (sums, maximum, sum of weights); ml_out: null, or where the row's maximum and sum go
__device__ __forceinline__ void merge_splits(const float *part, float *out, float *ml_out, int bh, int e, int nsplit, int d) {
  const float *p = part + size_t(bh) * nsplit * (d + 2);
  float M = -INFINITY;
  for (int s = 0; s < nsplit; ++s) M = fmaxf(M, p[s * (d + 2) + d]);
  float sum = 0.f, L = 0.f;
  for (int s = 0; s < nsplit; ++s) {
    const float ms = p[s * (d + 2) + d];
    const float f = (ms == -INFINITY) ? 0.f : exp2f(ms - M);
    sum = fmaf(p[s * (d + 2) + e], f, sum);
    L = fmaf(p[s * (d + 2) + d + 1], f, L);
  }
  out[size_t(bh) * d + e] = sum / L;
  if (ml_out && e == 0) {
    ml_out[size_t(bh) * 2] = M;
    ml_out[size_t(bh) * 2 + 1] = L;
  }
}

// ---- the controller of a short step inside the step's two other launches, d' = 128 ------------
// Nothing in the attention's launch waits for anything in it, and so in the projection's.  What of the controller needs only the
// token's embedding and the state before it rides in the first (StepCtrl), the rest in the second (StepTail), next to the merge of
// the attention's splits: a step on one stream is two launches instead of four or five, and W_hh, which one workgroup per sequence
// streamed through its compute unit (11 us in fp32), is spread over six.  What bounds such a step is latency: two launches of 5 to 8 us,
// each a few dependent trips to memory.  Per step, ordered inputs, before -> now: 1 sequence of 4 heads of 64 31 -> 18 us (fp32 39 -> 20), 8
// of 12 34 -> 21, 16 of 8 heads of 128 37 -> 26, 4 of 32 51 -> 39; with rescoring 3 of 12 47 -> 23 us.  The arithmetic and its order
// are those of the kernels in controller.hip.
struct StepCtrl {
  int n;                       // workgroups of 256 threads: n_in of the input projection, then 6 per sequence of W_hh z
  int n_in, tiles_j, tiles_t;
  int kslice;                  // length of a D-slice on the matrix cores; 0: the plain tiles
  const void *W_ih, *x, *W_hh;
  const float *z, *b_hh;
  float *gi, *gh;              // gh: [B][3d'] W_hh z + b_hh
  int D, B, seq_rows;
};

template <typename T>
__device__ __forceinline__ void step_ctrl_role(const StepCtrl &s, int e, float *lds) {
  constexpr int DP = 128;
  if (e < s.n_in) {
    const int jt = e % s.tiles_j, rest = e / s.tiles_j, tt = rest % s.tiles_t, zz = rest / s.tiles_t;
    if constexpr (sizeof(T) == 2) {
      if (s.kslice > 0) {
        ctrl_input_mfma_tile(static_cast<const bf16_t *>(s.W_ih), static_cast<const bf16_t *>(s.x), s.gi, s.D, 3 * DP, s.B, 1,
                             s.seq_rows, s.kslice, jt, tt, zz, lds);
        return;
      }
    }
    ctrl_input_plain_tile<T>(static_cast<const T *>(s.W_ih), static_cast<const T *>(s.x), s.gi, s.D, 3 * DP, s.B, 1, s.seq_rows,
                             jt, tt, lds);
    return;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int b = (e - s.n_in) / 6, row0 = ((e - s.n_in) % 6 * 4 + wave) * 16;
  const float2 hx = *reinterpret_cast<const float2 *>(s.z + size_t(b) * DP + 2 * lane);
  const T *W_hh = static_cast<const T *>(s.W_hh);
  decltype(load_raw2(W_hh)) raw[16];
  rows_request<T, 16>(W_hh, row0, lane, raw);
  __builtin_amdgcn_sched_barrier(0);
  rows_finish<decltype(load_raw2(W_hh)), 16>(raw, row0, hx.x, hx.y, s.b_hh, s.gh + size_t(b) * 3 * DP, lane);
}

struct StepTail {
  int n, n_cell;               // workgroups: one per sequence of the cell, then those that merge splits
  CellArgs cell;
  const float *gh;
  const float *part;           // [rows][nsplit][d + 2]
  float *out;                  // [rows][d]
  int rows, nsplit, d;
};

constexpr int kStepTailLds = 8 * 128;   // floats
// NT threads (256 or 512); lds: kStepTailLds floats.
template <int NT>
__device__ __forceinline__ void step_tail_role(const StepTail &s, int e, float *lds) {
  constexpr int DP = 128, RPW = DP / (NT / 64);        // rows of W_1 per wave
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (e >= s.n_cell) {
    const int row = (e - s.n_cell) * (NT / s.d) + tid / s.d;
    if (row < s.rows) merge_splits(s.part, s.out, nullptr, row, tid % s.d, s.nsplit, s.d);
    return;
  }
  const CellArgs &a = s.cell;
  float *gi_s = lds, *gh_s = gi_s + 3 * DP, *t_in = gh_s + 3 * DP, *u1 = t_in + DP;
  const int b = e;
  // ---- requests: everything the step reads, before anything is waited for ----
  float2 rw1[RPW];
  rows_request<float, RPW>(a.W1, wave * RPW, lane, rw1);
  float hold = 0.f, pw = 0.f, pb = 0.f, ow0 = 0.f, ow1 = 0.f, ob = 0.f, ov = 0.f;
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
  for (int j = tid; j < 3 * DP; j += NT) {
    const float hh = s.gh[size_t(b) * 3 * DP + j];
    gi_s[j] = gi_sum(a, size_t(b), j) + a.b_ih[j];
    gh_s[j] = hh;
  }
  __syncthreads();
  // ---- the gates, the new state ----
  if (tid < DP) {
    const float r = sigmoidf_(gi_s[tid] + gh_s[tid]);
    const float u = sigmoidf_(gi_s[DP + tid] + gh_s[DP + tid]);
    const float cand = tanhf(gi_s[2 * DP + tid] + r * gh_s[2 * DP + tid]);
    const float hnew = (1.0f - u) * cand + u * hold;
    const float delta = a.cvec ? 0.f : float(a.pos0) * a.pos_scale;   // rescore mode: distance to itself
    a.z[size_t(b) * DP + tid] = hnew;
    t_in[tid] = fmaf(pw, delta, pb) + hnew;
  }
  __syncthreads();
  // ---- interaction layer, output layer, sigmoid ----
  rows_finish<float2, RPW>(rw1, wave * RPW, t_in[2 * lane], t_in[2 * lane + 1], a.b1, u1, lane);
  __syncthreads();
  if (a.cvec && tid < DP) a.cvec[(size_t(b) * a.N_max + a.pos0) * DP + tid] = u1[tid];
  if (wave == 0) {
    float sum = fmaf(ow0, tanhf(u1[lane]), ow1 * tanhf(u1[lane + 64]));
    sum = wave_sum(sum);
    if (lane == 0) a.score[size_t(b) * a.N_max + a.pos0] = a.override_ ? ov : sigmoidf_(sum + ob);
  }
}

}  // namespace adore
