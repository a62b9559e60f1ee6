// Stage 1: insert the current token's k, v and single-query attention over the
// occupied slots of every (sequence, head)  (paper Sec. 2.1: Eq. 1 restricted to
// the retained rows plus the current token).
//
// Memory-bound: every step streams K*d*2 elements of K and V per row once.  A
// row of d elements is 16-byte vectors spread over LPR consecutive lanes, so a
// wave reads 64/LPR whole cache rows (1 KB, contiguous) per load instruction.
// The slots of one (b,h) are cut into `nsplit` chunks, one workgroup each, so
// that small batches still fill the chip; partial (max, sum, acc) triples are
// merged by a second small kernel (a merge inside the first kernel would need a
// device-scope release per workgroup, which on a multi-XCD part writes back the
// whole L2 and costs far more than the extra launch).  When there are enough
// rows, one workgroup of up to 16 waves takes a whole row and no merge kernel
// runs.  Softmax runs online in fp32, base 2.
#include <cstdlib>

#include "ctrl_device.h"
#include "select_device.h"

namespace adore {

namespace {

// The step's two selections as extra workgroups of the attention launch (static score mode: neither selection
// of step n looks at the current token's score, so they depend on nothing this launch computes, and nothing in
// this launch depends on them).  Per sequence: rel_wgs workgroups release heads 1 .. H-1 (one wave per head),
// one more releases head 0 and then chooses the tokens to rebuild from the positions head 0 keeps.
// The chosen positions are entered into the slot maps by the kernel that writes their rows.
struct SchedArgs {
  int kpl, rel_wgs;                 // keys per lane of a row (K / 64 rounded up to 2, 4, 8, 16); 0 workgroups = off
  int prio;                         // wave priority of the role (0 .. 3)
  int hpw;                          // heads a wave releases one after the other (1, or 4 for short rows of many sequences); 0: a
                                    // workgroup per head (few rows)
  const int32_t *slot_src;          // [B*H][K]
  int32_t *slot_dst;                // [B*H][K]
  const float *score;               // [B][N_max]
  int32_t *free_list;               // [B*H][R1]
  int32_t *released_pos, *map_out, *rel_out;
  int H, K, N_max, n, x, R1;
  RebuildSelectArgs sel;
  ChoiceParts parts;                // long sequences: the choice in workgroups of its own, behind the release ones of each sequence
};

struct AttendArgs {
  const void *q, *k_new, *v_new;   // [B*H][d]
  void *Kc, *Vc;                   // [B*H][K][d] of this layer
  const int32_t *slot_pos;         // [B*H][K]
  const int32_t *insert_slot;      // the reserved slot of row bh is insert_slot[bh * ins_stride + ins_off]
  int ins_stride, ins_off;
  int n_sel;                       // the first n_sel workgroups carry the selections (they start first: their chain
                                   // of dependent steps is the longest), the attention's come behind them
  SchedArgs s;
  StepCtrl c;                      // the c.n workgroups behind those carry the controller's first part (c.n = 0: none)
  float *part;                     // [B*H][nsplit][d+2]
  float *out;                      // [B*H][d]
  float *logit_out;                // null, or [B*H][K]: every slot's logit as scaled here (base 2; -inf for a free slot)
  float *ml_out;                   // ... and [B*H][2]: the row's maximum logit and the sum of exp2(logit - maximum),
                                   // from which a row's probabilities follow (the scores of the H2O mode)
  int K, chunk, nsplit;
  float scale_log2;                // log2(e) / sqrt(d)
};

// Dynamic LDS of a workgroup in this role: [scores of the sequence, n + 1 floats][head 0's row, K ints][choice].
// The scores are copied once and the rows are read at the same time, so that afterwards the ranking keys come
// from LDS: under the attention's traffic every dependent trip to memory costs five to seven microseconds.
// hist: 256 words of LDS per wave for the release's radix select (the attention's own merge buffer, which these
// workgroups do not use otherwise).
template <int WAVES, int KPL>
__device__ __forceinline__ void selections_role(const AttendArgs &a, int e, uint64_t *dyn, uint32_t *hist) {
  // Rows short enough to fit four of them into a wave's registers can be released four to a wave: with hundreds of
  // sequences the role's workgroups would otherwise take half of the chip's wave slots from the attention for the
  // time their trips to memory take.
  constexpr int HPW = KPL <= 4 ? 4 : 1;
  const SchedArgs &s = a.s;
  const int per_seq = s.rel_wgs + 1;
  const int b = e / per_seq, part = e - b * per_seq;
  const int tid = threadIdx.x, wave = tid >> 6;
  switch (s.prio) {   // few waves with a long chain of dependent steps
    case 3: __builtin_amdgcn_s_setprio(3); break;
    case 2: __builtin_amdgcn_s_setprio(2); break;
    case 1: __builtin_amdgcn_s_setprio(1); break;
    default: break;
  }
  float *s_score = reinterpret_cast<float *>(dyn);
  const float *sc = s.score + size_t(b) * s.N_max;
  if constexpr (WAVES == 4) {
    if (s.hpw == 0) {              // head 1 + part, the last one head 0 and the choice
      constexpr int WIDE = KPL >= 4 ? KPL / 4 : 1;
      const bool first = part == s.rel_wgs;
      const int row = b * s.H + (first ? 0 : 1 + part);
      const int s_ins = a.insert_slot[size_t(row) * a.ins_stride + a.ins_off];
      int raw[WIDE];
      release_fetch_wide<WIDE>(row, s.slot_src, s.K, raw);
      for (int i = tid; i <= s.n; i += 256) s_score[i] = sc[i];
      __syncthreads();
      int32_t *row_copy = first ? reinterpret_cast<int32_t *>(dyn + (s.n + 2) / 2) : nullptr;
      uint64_t *choice = dyn + (s.n + 2) / 2 + (s.K + 1) / 2;
      if (first) choice_fill_keys(s_score, s.n, choice, tid, 256);
      release_row_wide<WIDE>(row, s_ins, s.slot_dst, s_score, s.free_list, s.released_pos, s.map_out, s.rel_out, s.K, s.n, s.x, s.R1,
                             row_copy, hist, raw);
      if (!first) return;
      __syncthreads();
      choice_from_keys(s.sel, b, row_copy, choice, hist, dyn, (s.n + 2) / 2);   // (the scores are done with)
      return;
    }
  }
  if (part < s.rel_wgs) {          // heads 1 .. H-1
    const int hpw = HPW > 1 ? s.hpw : 1;
    const int h0 = 1 + (part * WAVES + wave) * hpw;
    int raw[HPW][KPL], s_ins[HPW];
#pragma unroll
    for (int i = 0; i < HPW; ++i) {
      if (i < hpw && h0 + i < s.H) {   // whole waves
        const int row = b * s.H + h0 + i;
        s_ins[i] = a.insert_slot[size_t(row) * a.ins_stride + a.ins_off];
        release_fetch<KPL>(row, s.slot_src, s.K, raw[i]);
      }
    }
    for (int i = tid; i <= s.n; i += 64 * WAVES) s_score[i] = sc[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < HPW; ++i) {
      if (i < hpw && h0 + i < s.H)
        release_row<KPL>(b * s.H + h0 + i, s_ins[i], s.slot_src, s.slot_dst, s_score, s.free_list, s.released_pos, s.map_out,
                         s.rel_out, s.K, s.n, s.x, s.R1, nullptr, hist + wave * 256, raw[i]);
    }
    return;
  }
  // head 0, then the choice of the tokens to rebuild from the positions it keeps
  const int row = b * s.H;
  const int s_ins = a.insert_slot[size_t(row) * a.ins_stride + a.ins_off];
  int raw[KPL];
  if (wave == 0) release_fetch<KPL>(row, s.slot_src, s.K, raw);
  for (int i = tid; i <= s.n; i += 64 * WAVES) s_score[i] = sc[i];
  __syncthreads();
  int32_t *row_copy = reinterpret_cast<int32_t *>(dyn + (s.n + 2) / 2);   // head 0's positions after the release
  uint64_t *choice = dyn + (s.n + 2) / 2 + (s.K + 1) / 2;
  if (wave == 0) {
    release_row<KPL>(row, s_ins, s.slot_src, s.slot_dst, s_score, s.free_list, s.released_pos, s.map_out,
                     s.rel_out, s.K, s.n, s.x, s.R1, row_copy, hist, raw);
  } else {
    choice_fill_keys(s_score, s.n, choice, tid - 64, 64 * (WAVES - 1));   // the other waves meanwhile
  }
  __syncthreads();
  choice_from_keys(s.sel, b, row_copy, choice, hist, dyn, (s.n + 2) / 2);   // (the scores are done with)
}

// The same for sequences whose scores do not fit a workgroup's LDS (one launch, parts.n_parts > 0): per sequence rel_wgs workgroups
// release heads 1 .. H-1, one head 0, and n_parts more share the choice (choice_part).  The scores of the rows held are gathered from memory.
template <int WAVES, int KPL>
__device__ __forceinline__ void selections_in_parts_role(const AttendArgs &a, int e, uint64_t *dyn, uint32_t *hist) {
  static_assert(WAVES == 4, "256 threads");
  const SchedArgs &s = a.s;
  const int per_seq = s.rel_wgs + 1 + s.parts.n_parts;
  const int b = e / per_seq, part = e - b * per_seq;
  const int wave = threadIdx.x >> 6;
  __builtin_amdgcn_s_setprio(3);
  if (part > s.rel_wgs) {
    choice_part(s.sel, s.parts, b, part - s.rel_wgs - 1, s.slot_src + size_t(b) * s.H * s.K, dyn);
    choice_arrive(s.sel, s.parts, b, dyn, hist);
    return;
  }
  if (s.hpw == 0) {                // a workgroup per head
    constexpr int WIDE = KPL >= 4 ? KPL / 4 : 1;
    const int row = b * s.H + (part < s.rel_wgs ? 1 + part : 0);
    const int s_ins = a.insert_slot[size_t(row) * a.ins_stride + a.ins_off];
    int raw[WIDE];
    release_fetch_wide<WIDE>(row, s.slot_src, s.K, raw);
    release_row_wide<WIDE>(row, s_ins, s.slot_dst, s.score + size_t(b) * s.N_max, s.free_list, s.released_pos, s.map_out, s.rel_out, s.K,
                           s.n, s.x, s.R1, nullptr, hist, raw);
  }
  // heads 1 .. H-1, a wave each; the last of these workgroups head 0
  const int h = s.hpw == 0 ? s.H : part < s.rel_wgs ? 1 + part * WAVES + wave : wave == 0 ? 0 : s.H;
  if (h < s.H) {                 // whole waves
    const int row = b * s.H + h;
    release_row<KPL>(row, a.insert_slot[size_t(row) * a.ins_stride + a.ins_off], s.slot_src, s.slot_dst, s.score + size_t(b) * s.N_max,
                     s.free_list, s.released_pos, s.map_out, s.rel_out, s.K, s.n, s.x, s.R1, nullptr, hist + wave * 256);
  }
  if (part == s.rel_wgs) {
    __syncthreads();             // head 0's released positions, written by this workgroup
    choice_released(s.sel, s.parts, b, s.released_pos + size_t(b) * s.H * s.R1);
    choice_arrive(s.sel, s.parts, b, dyn, hist);
  }
}

// The H2O mode's release of row bh by the first wave of the workgroup that attended over it: what h2o_release_kernel does, from the
// logits in LDS and the row's (M, L) at hand.  s.x: the rows to keep.
template <int KPL>
__device__ __forceinline__ void h2o_release_role(const AttendArgs &a, int bh, int s_ins, float M, float L, const float *logit, uint32_t *hist) {
  const SchedArgs &s = a.s;
  const int lane = threadIdx.x & 63;
  float *sc = const_cast<float *>(s.score) + size_t(bh) * s.N_max;
  int raw[KPL];
  float held[KPL];
  release_fetch<KPL>(bh, s.slot_src, s.K, raw);
#pragma unroll
  for (int j = 0; j < KPL; ++j) {
    const int k = j * 64 + lane, pos = k == s_ins ? s.n : raw[j];
    held[j] = k < s.K && pos >= 0 && pos != s.n ? sc[pos] : 0.f;
  }
#pragma unroll
  for (int j = 0; j < KPL; ++j) {
    const int k = j * 64 + lane, pos = k == s_ins ? s.n : raw[j];
    if (k >= s.K || pos < 0) continue;
    const float p = exp2f(logit[k] - M) / L;
    held[j] = pos == s.n ? p : held[j] + p;      // the current token starts its score here
    sc[pos] = held[j];
  }
  release_row<KPL>(bh, s_ins, s.slot_src, s.slot_dst, sc, s.free_list, s.released_pos, s.map_out, s.rel_out, s.K, s.n, -1, s.R1, nullptr,
                   hist, raw, s.x, held);
}

// KPL > 0: the H2O mode's whole step, each row's release behind its attention (rows that one workgroup takes whole).
template <typename T, int DH, int U, int WAVES, int KPL = 0>
__global__ __launch_bounds__(64 * WAVES, 4) void attend_kernel(const AttendArgs a) {
  constexpr int EPL = Vec16<T>::EPL;    // elements per lane
  constexpr int LPR = DH / EPL;         // lanes per cache row
  constexpr int RPW = 64 / LPR;         // rows per wave and load
  constexpr int G = WAVES * RPW;        // lane groups (rows in flight) per workgroup
  static_assert(LPR >= 1 && LPR <= 64 && (LPR & (LPR - 1)) == 0, "row must be a power-of-two lane group");
  // merge of the lane groups at the end of a row; a workgroup that carries selections instead keeps its waves'
  // radix histograms there
  __shared__ float s_m[G], s_l[G];
  __shared__ __align__(16) float s_acc[G][DH];
  static_assert(G * DH >= kWideWords && G * DH >= WAVES * 256 && G * DH >= (sizeof(T) == 2 ? kInputTileLds : 4 * JT * NB), "room for one 256-bin histogram per wave, for an input tile's sums");

  extern __shared__ __align__(16) uint64_t dyn_smem[];
  if (KPL == 0 && int(blockIdx.x) < a.n_sel) {   // uniform over the workgroup
    const int e = blockIdx.x;
    uint32_t *hist = reinterpret_cast<uint32_t *>(&s_acc[0][0]);
    if constexpr (WAVES == 4) {
      if (a.s.parts.n_parts > 0) {
        switch (a.s.kpl) {
          case 2: selections_in_parts_role<WAVES, 2>(a, e, dyn_smem, hist); break;
          case 4: selections_in_parts_role<WAVES, 4>(a, e, dyn_smem, hist); break;
          case 8: selections_in_parts_role<WAVES, 8>(a, e, dyn_smem, hist); break;
          default: selections_in_parts_role<WAVES, 16>(a, e, dyn_smem, hist); break;
        }
        return;
      }
    }
    switch (a.s.kpl) {
      case 2: selections_role<WAVES, 2>(a, e, dyn_smem, hist); break;
      case 4: selections_role<WAVES, 4>(a, e, dyn_smem, hist); break;
      case 8: selections_role<WAVES, 8>(a, e, dyn_smem, hist); break;
      default: selections_role<WAVES, 16>(a, e, dyn_smem, hist); break;
    }
    return;
  }
  if (KPL == 0 && int(blockIdx.x) < a.n_sel + a.c.n) {
    step_ctrl_role<T>(a.c, blockIdx.x - a.n_sel, &s_acc[0][0]);
    return;
  }
  const int wg = blockIdx.x - a.n_sel - a.c.n;
  const int bh = wg / a.nsplit;
  const int sp = wg - bh * a.nsplit;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int grp = (tid >> 6) * RPW + lane / LPR;
  const int lig = lane % LPR;

  const T *Kb = static_cast<const T *>(a.Kc) + size_t(bh) * a.K * DH;
  const T *Vb = static_cast<const T *>(a.Vc) + size_t(bh) * a.K * DH;
  const int32_t *sp_row = a.slot_pos + size_t(bh) * a.K;
  const int s_ins = a.insert_slot[size_t(bh) * a.ins_stride + a.ins_off];

  float qf[EPL];
  Vec16<T>::load(static_cast<const T *>(a.q) + size_t(bh) * DH + lig * EPL, qf);
#pragma unroll
  for (int e = 0; e < EPL; ++e) qf[e] *= a.scale_log2;
  // the current token's k, v: every lane group holds them, the one that meets the reserved slot uses them
  const typename Vec16<T>::Raw kn = Vec16<T>::load_raw(static_cast<const T *>(a.k_new) + size_t(bh) * DH + lig * EPL);
  const typename Vec16<T>::Raw vn = Vec16<T>::load_raw(static_cast<const T *>(a.v_new) + size_t(bh) * DH + lig * EPL);

  const int begin = sp * a.chunk;
  const int end = min(a.K, begin + a.chunk);

  float m = -INFINITY, l = 0.f, acc[EPL];
#pragma unroll
  for (int e = 0; e < EPL; ++e) acc[e] = 0.f;

  // cache rows are read whatever they hold (no read waits for the reserved slot's index to arrive), one
  // iteration ahead of their use; the row of the reserved slot is then replaced by the current token's k, v,
  // which are also stored (the slot is marked occupied by the release kernel, which knows the reserved slot too)
  typename Vec16<T>::Raw kr[U], vr[U];
  int spv[U];
#define ATTEND_FETCH(BASE)                                                        \
  _Pragma("unroll") for (int u = 0; u < U; ++u) {                                 \
    const int slot_ = min((BASE) + u * G + grp, end - 1);                         \
    kr[u] = Vec16<T>::load_raw(Kb + size_t(slot_) * DH + lig * EPL);              \
    vr[u] = Vec16<T>::load_raw(Vb + size_t(slot_) * DH + lig * EPL);              \
    spv[u] = sp_row[slot_];                                                       \
  }
  if (begin < end) { ATTEND_FETCH(begin) }
  for (int base = begin; base < end; base += G * U) {
    float logit[U];
    bool valid[U];
    typename Vec16<T>::Raw kc[U], vc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int slot = base + u * G + grp;
      const bool inr = slot < end;
      const bool ins = inr && slot == s_ins;
      if (ins) {
        Vec16<T>::store_raw(const_cast<T *>(Kb) + size_t(slot) * DH + lig * EPL, kn);
        Vec16<T>::store_raw(const_cast<T *>(Vb) + size_t(slot) * DH + lig * EPL, vn);
      }
      kc[u] = ins ? kn : kr[u];
      vc[u] = ins ? vn : vr[u];
      valid[u] = inr && (ins || spv[u] >= 0);
    }
    if (base + G * U < end) { ATTEND_FETCH(base + G * U) }
    float mb = m;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float dot = 0.f;
      if (valid[u]) {
        float kf[EPL];
        Vec16<T>::values(kc[u], kf);
#pragma unroll
        for (int e = 0; e < EPL; ++e) dot = fmaf(qf[e], kf[e], dot);
      }
      dot = group_sum<LPR>(dot);
      logit[u] = valid[u] ? dot : -INFINITY;
      mb = fmaxf(mb, logit[u]);
      if (KPL > 0) {
        if (lig == 0 && base + u * G + grp < end) reinterpret_cast<float *>(dyn_smem)[base + u * G + grp] = logit[u];
      } else if (a.logit_out && lig == 0 && base + u * G + grp < end) {
        a.logit_out[size_t(bh) * a.K + base + u * G + grp] = logit[u];
      }
    }
    if (mb == -INFINITY) continue;  // nothing occupied so far in this lane group
    const float corr = exp2f(m - mb);
    l *= corr;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[e] *= corr;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (valid[u]) {
        const float p = exp2f(logit[u] - mb);
        l += p;
        float vf[EPL];
        Vec16<T>::values(vc[u], vf);
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] = fmaf(p, vf[e], acc[e]);
      }
    }
    m = mb;
  }

#undef ATTEND_FETCH

  // ---- merge the G lane groups of this workgroup ----
  if (lig == 0) s_m[grp] = m;
  __syncthreads();
  float M = -INFINITY;
#pragma unroll
  for (int g = 0; g < G; ++g) M = fmaxf(M, s_m[g]);
  const float f = (m == -INFINITY) ? 0.f : exp2f(m - M);
#pragma unroll
  for (int e = 0; e < EPL; ++e) s_acc[grp][lig * EPL + e] = acc[e] * f;
  if (lig == 0) s_l[grp] = l * f;
  __syncthreads();
  if (tid < DH) {
    float sum = 0.f, L = 0.f;
#pragma unroll 8
    for (int g = 0; g < G; ++g) {
      sum += s_acc[g][tid];
      L += s_l[g];
    }
    if (a.nsplit == 1) {
      a.out[size_t(bh) * DH + tid] = sum / L;   // the current token is always present: L > 0
      if (KPL == 0 && a.ml_out && tid == 0) {
        a.ml_out[size_t(bh) * 2] = M;
        a.ml_out[size_t(bh) * 2 + 1] = L;
      }
    } else {
      float *p = a.part + (size_t(bh) * a.nsplit + sp) * (DH + 2);
      p[tid] = sum;
      if (tid == 0) {
        p[DH] = M;
        p[DH + 1] = L;
      }
    }
  }
  if constexpr (KPL > 0) {
    if (tid >= 64) return;                // (the sums below in the order of the ones above)
    float L = 0.f;
#pragma unroll 8
    for (int g = 0; g < G; ++g) L += s_l[g];
    __shared__ uint32_t s_hist[256];
    h2o_release_role<KPL>(a, bh, s_ins, M, L, reinterpret_cast<const float *>(dyn_smem), s_hist);
  }
}

template <int DH>
__global__ __launch_bounds__(DH) void attend_combine_kernel(const float *part, float *out, int nsplit, float *ml_out) {
  merge_splits(part, out, ml_out, blockIdx.x, threadIdx.x, nsplit, DH);
}

template <typename T, int DH>
hipError_t launch_h2o_typed(adore_ctx *ctx, const AttendArgs &a, int rows) {
  ScopedTimer t(ctx, ADORE_KERNEL_ATTEND, ctx->stream);
  const size_t lds = size_t(a.K) * 4;
  if constexpr (sizeof(T) == 4) {
    // fp32 rows of 256 to 511 slots keep to the eight waves that the attention alone takes (choose_split): with four a lane group adds
    // up twice as many of them (1.71e-7 -> 1.79e-7 off 64 bits at 256 slots, 1.85e-7 -> 2.05e-7 at 500; in bf16 1.91e-7 -> 1.74e-7).
    if (ctx->attend_waves == 8 && a.K <= 512) {
      if (a.K <= 256) ADORE_LAUNCH(t, (attend_kernel<T, DH, 4, 8, 4>), dim3(rows), dim3(512), lds, ctx->stream, a);
      else ADORE_LAUNCH(t, (attend_kernel<T, DH, 4, 8, 8>), dim3(rows), dim3(512), lds, ctx->stream, a);
      return hipGetLastError();
    }
  }
  if (a.K <= 256) ADORE_LAUNCH(t, (attend_kernel<T, DH, 4, 4, 4>), dim3(rows), dim3(256), lds, ctx->stream, a);
  else if (a.K <= 512) ADORE_LAUNCH(t, (attend_kernel<T, DH, 4, 4, 8>), dim3(rows), dim3(256), lds, ctx->stream, a);
  else ADORE_LAUNCH(t, (attend_kernel<T, DH, 4, 4, 16>), dim3(rows), dim3(256), lds, ctx->stream, a);
  return hipGetLastError();
}

template <typename T, int DH>
hipError_t launch_typed(adore_ctx *ctx, const AttendArgs &a, int rows, int waves, int extra_wgs, size_t dyn_lds, bool merge) {
  {
    ScopedTimer t(ctx, ADORE_KERNEL_ATTEND, ctx->stream);
    const dim3 grid(rows * a.nsplit + extra_wgs);
    if (waves == 16)
      ADORE_LAUNCH(t, (attend_kernel<T, DH, 4, 16>), grid, dim3(1024), dyn_lds, ctx->stream, a);
    else if (waves == 8)
      ADORE_LAUNCH(t, (attend_kernel<T, DH, 4, 8>), grid, dim3(512), dyn_lds, ctx->stream, a);
    else
      ADORE_LAUNCH(t, (attend_kernel<T, DH, 4, 4>), grid, dim3(256), dyn_lds, ctx->stream, a);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (a.nsplit > 1 && merge) {
    ScopedTimer t(ctx, ADORE_KERNEL_ATTEND_COMBINE, ctx->stream);
    ADORE_LAUNCH(t, (attend_combine_kernel<DH>), dim3(rows), dim3(DH), 0, ctx->stream, a.part, a.out,
                       a.nsplit, a.ml_out);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace

// The choice in parts (see ChoiceParts): where a workgroup's LDS does not hold a sequence's scores and keys.
int choice_parts(int n) { return (n + kPartTokens - 1) / kPartTokens; }
bool parts_fit(const adore_config &c) {
  const int Rdim = max(c.rebuild_budget, 1), parts = choice_parts(c.max_positions - 1);
  return c.cache_slots <= kMaxSlots && parts <= kMostParts && choice_part_keys(parts, Rdim) <= kMostPartKeys;
}
size_t parts_bytes(const adore_config &c) {
  return size_t(c.batch) * choice_part_keys(choice_parts(c.max_positions - 1), max(c.rebuild_budget, 1)) * 8 + size_t(c.batch) * 4;
}
// Where either is possible the parts win from about 2000 positions on (per step, one workgroup / parts): 1 sequence of 4 heads behind 900
// tokens 14.6 / 17.4 us, 16 of 32 behind 1024 73.8 / 78.3, 3 of 12 behind 2000 21.7 / 20.2, 8 of 32 behind 2000 55.3 / 53.5, 2 of 8 behind 3500
// 21.8 / 19.4, 16 of 16 behind 3500 39.7 / 33.8; with more than 2048 heads in all one workgroup per sequence and four heads a wave
// (hpw) take less from the attention (128 of 32: 258 / 263).  Behind 8192 tokens (4 of 32, K = 1024), where one workgroup's LDS does not
// hold a sequence: 84 us a step with the selections in launches of their own on side streams, whose events hold the host for 77 us,
// 50 in parts (attention and all of it 25 us, projection 26).
bool ride_in_parts(const adore_ctx *ctx, int r) { return ctx->ride_parts && r > 0 && (!ctx->ride_whole || ctx->n >= kPartsFrom); }

// Rows up to which a workgroup releases one head rather than one a wave.  Attention and all it carries (us, a wave / a workgroup): 4
// sequences of 32 heads, K = 1024, behind 8192 tokens 24.1 / 17.8, behind 1500 19.7 / 16.4; 2 of 32, K = 512 13.8 / 12.6; 16 of 16, K = 256
// 12.2 / 12.2; 32 of 8, K = 512 17.9 / 18.5 to 18.9; 16 of 32 the same (the attention is what takes the time).
constexpr int kWideRows = 128;

size_t riding_lds_bytes(int n, int K, int r) {
  return size_t((n + 2) / 2) * 8 + size_t((K + 1) / 2) * 8 + ridden_choice_lds_bytes(r, n);
}

// sel: null, or the selections of this step to carry in the same launch (see SchedArgs); ctrl: null, or (with sel) the first part of its
// controller, in which case tail receives the merge of this launch's splits for the launch that carries the second.
hipError_t launch_attend(adore_ctx *ctx, int layer, const void *q, const void *k_new, const void *v_new,
                         float *out, const RidingSelections *sel, const StepCtrl *ctrl, StepTail *tail) {
  const adore_config &c = ctx->cfg;
  const size_t layer_bytes = size_t(c.batch) * c.heads * c.cache_slots * c.head_dim * elem_size(c);
  AttendArgs a;
  a.q = q; a.k_new = k_new; a.v_new = v_new;
  a.Kc = ctx->cache_k + layer * layer_bytes;
  a.Vc = ctx->cache_v + layer * layer_bytes;
  a.slot_pos = ctx->slot_pos[ctx->cur];
  a.insert_slot = reserved_slots(ctx, ctx->cur);
  a.ins_stride = ctx->ins_stride; a.ins_off = ctx->ins_off;
  a.part = ctx->att_part;
  a.out = out;
  a.logit_out = h2o_mode(ctx) ? ctx->att_logit : nullptr;
  a.ml_out = h2o_mode(ctx) ? ctx->att_ml : nullptr;
  a.K = c.cache_slots; a.chunk = ctx->chunk; a.nsplit = ctx->nsplit;
  a.scale_log2 = 1.4426950408889634f / sqrtf(float(c.head_dim));
  const int rows = c.batch * c.heads;
  a.n_sel = 0;
  a.s.rel_wgs = 0;
  a.c.n = 0;
  int waves = ctx->attend_waves, extra = 0;
  size_t dyn = 0;
  if (sel) {
    // 4 waves per workgroup: half of a compute unit's wave slots and registers then stay free, so the extra
    // workgroups start at once next to the attention's instead of waiting for a round of them to end
    waves = 4;
    if (const char *e = ctrl ? nullptr : getenv("ADORE_RIDE_WAVES")) {   // tuning runs (the controller's part has 4)
      const int v = atoi(e);
      if (v == 4 || v == 8) waves = v;
    }
    SchedArgs &s = a.s;
    s.kpl = c.cache_slots <= 128 ? 2 : c.cache_slots <= 256 ? 4 : c.cache_slots <= 512 ? 8 : 16;
    // four heads to a wave where a row is short (four of them fit a wave's registers) and the role would otherwise
    // take more than a quarter of the chip's wave slots
    s.prio = 3;
    if (const char *e = getenv("ADORE_ROLE_PRIO")) s.prio = atoi(e);   // tuning runs
    s.hpw = s.kpl <= 4 && c.batch * c.heads > 2048 ? 4 : 1;
    if (const char *e = getenv("ADORE_RIDE_HPW")) {   // tests: the four-heads path on a small shape
      if (atoi(e) == 4 && s.kpl <= 4) s.hpw = 4;
    }
    const bool per_head = waves == 4 && s.hpw == 1 && rows <= kWideRows;
    s.rel_wgs = per_head ? c.heads - 1 : (c.heads - 1 + waves * s.hpw - 1) / (waves * s.hpw);
    if (per_head) s.hpw = 0;
    s.slot_src = ctx->slot_pos[ctx->cur]; s.slot_dst = ctx->slot_pos[sel->dst];
    s.score = ctx->score; s.free_list = ctx->free_list[sel->dst];
    s.released_pos = ctx->released_pos; s.map_out = sel->map_out; s.rel_out = sel->rel_out;
    s.H = c.heads; s.K = c.cache_slots; s.N_max = c.max_positions; s.n = ctx->n; s.x = sel->x;
    s.R1 = c.rebuild_budget + 1;
    RebuildSelectArgs &r = s.sel;
    r.slot_pos = ctx->slot_pos[sel->dst]; r.score = ctx->score; r.free_list = ctx->free_list[sel->dst];
    r.rebuilt_pos = ctx->rebuilt_pos[sel->dst]; r.insert_slot = nullptr;
    r.map_out = sel->map_out; r.rb_out = sel->rb_out;
    r.K = c.cache_slots; r.H = c.heads; r.N_max = c.max_positions; r.n = ctx->n; r.r = sel->r;
    r.R1 = c.rebuild_budget + 1; r.Rdim = max(c.rebuild_budget, 1);
    r.words = (c.max_positions + 31) / 32;
    s.parts.n_parts = 0;
    dyn = riding_lds_bytes(ctx->n, c.cache_slots, sel->r);
    if (ride_in_parts(ctx, sel->r)) {
      waves = 4;
      s.hpw = rows <= kWideRows ? 0 : 1;
      s.rel_wgs = s.hpw == 0 ? c.heads - 1 : (c.heads - 1 + waves - 1) / waves;
      s.parts.n_parts = choice_parts(ctx->n);
      s.parts.keys = ctx->part_keys;
      s.parts.arrived = ctx->part_arrived;
      dyn = choice_parts_lds_bytes(s.parts.n_parts, r.Rdim);
    }
    extra = c.batch * (s.rel_wgs + 1 + s.parts.n_parts);
    a.n_sel = extra;
    if (ctrl) {
      a.c = *ctrl;
      extra += ctrl->n;
      tail->part = ctx->att_part;
      tail->out = out;
      tail->rows = ctx->nsplit > 1 ? rows : 0;
      tail->nsplit = ctx->nsplit;
      tail->d = c.head_dim;
    }
  }
  if (c.dtype == ADORE_BF16) {
    return c.head_dim == 128 ? launch_typed<bf16_t, 128>(ctx, a, rows, waves, extra, dyn, !ctrl)
                             : launch_typed<bf16_t, 64>(ctx, a, rows, waves, extra, dyn, !ctrl);
  }
  return c.head_dim == 128 ? launch_typed<float, 128>(ctx, a, rows, waves, extra, dyn, !ctrl)
                           : launch_typed<float, 64>(ctx, a, rows, waves, extra, dyn, !ctrl);
}

// H2O mode: attention, the step's probabilities added to the scores and the release in one launch, where a workgroup takes a whole
// row.  16 sequences of 32 heads, K = 512: 22.5 + 15.5 us (and the logits' way through memory) -> 29 us, the
// step 101 -> 90 us.  With four waves also at 256 to 511 slots in bf16, where the attention alone takes eight: 40 steps 2075 -> 1806 us at 256,
// 2315 -> 1975 at 300, 2839 -> 2362 at 500, 1935 -> 1625 with 40 sequences of 12 heads of 64 and 300.
bool h2o_attend_releases(const adore_ctx *ctx) { return h2o_mode(ctx) && ctx->nsplit == 1; }

hipError_t launch_h2o_attend_release(adore_ctx *ctx, const void *q, const void *k_new, const void *v_new, float *out, int dst,
                                     int32_t *map_out) {
  const adore_config &c = ctx->cfg;
  AttendArgs a = {};
  a.q = q; a.k_new = k_new; a.v_new = v_new;
  a.Kc = ctx->cache_k; a.Vc = ctx->cache_v;
  a.slot_pos = ctx->slot_pos[ctx->cur];
  a.insert_slot = reserved_slots(ctx, ctx->cur);
  a.ins_stride = ctx->ins_stride; a.ins_off = ctx->ins_off;
  a.out = out;
  a.K = c.cache_slots; a.chunk = c.cache_slots; a.nsplit = 1;
  a.scale_log2 = 1.4426950408889634f / sqrtf(float(c.head_dim));
  SchedArgs &s = a.s;
  s.slot_src = ctx->slot_pos[ctx->cur]; s.slot_dst = ctx->slot_pos[dst];
  s.score = ctx->score; s.free_list = ctx->free_list[dst];
  s.released_pos = ctx->released_pos; s.map_out = map_out; s.rel_out = nullptr;
  s.K = c.cache_slots; s.N_max = c.max_positions; s.n = ctx->n;
  s.x = c.cache_slots - c.rebuild_budget - 1; s.R1 = c.rebuild_budget + 1;
  const int rows = c.batch * c.heads;
  if (c.dtype == ADORE_BF16) return c.head_dim == 128 ? launch_h2o_typed<bf16_t, 128>(ctx, a, rows) : launch_h2o_typed<bf16_t, 64>(ctx, a, rows);
  return c.head_dim == 128 ? launch_h2o_typed<float, 128>(ctx, a, rows) : launch_h2o_typed<float, 64>(ctx, a, rows);
}

}  // namespace adore
