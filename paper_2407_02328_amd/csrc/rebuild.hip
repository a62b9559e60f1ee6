// Stage 4: rebuild the K/V states of the chosen released tokens (paper Sec. 2.3)
// by re-projecting their hidden states with W_k / W_v and writing each head's
// slice straight into the slot the schedule assigned to it.
//
//   C[M = B*r, N = 2*H*d] = X_gathered[M, D] * W_kv[N, D]^T     (fp32 accumulate, one rounding)
//
// Row mi of the product is token rho = mi % r of sequence b = mi / r; its source
// row is hidden[b][rebuilt_pos[b][rho]] (gather), its destination rows are
// cache_{k,v}[b][h][free_list[b][h][rho]] (scatter).  No [M,N] tensor is ever
// materialised and nothing is compacted.
//
// bf16 path: a real dense contraction, so it runs on the matrix cores
// (v_mfma_f32_32x32x16_bf16).  Both operands are contiguous along the reduction
// dimension, which is exactly the per-lane operand layout of that instruction
// (8 consecutive k for one row), so tiles go global -> LDS -> registers as
// 16-byte vectors with no transposes.  One kernel template covers a family of
// output tiles; the launcher takes the largest tile that still gives every compute
// unit a workgroup (M = 512 at the 7B shape: 128x128, one tile per unit;
// M >= 2048: 256x256; M = 128: 64x64; M <= 32: 32x32).  Larger tiles move fewer bytes per flop, from the
// L2 to the compute unit and through LDS, and that path is what the 128x128 tile runs into first.  LDS stages
// are XOR-swizzled (conflict-free for 16-byte reads and writes).  The output tile
// is rounded to bf16 into LDS and leaves as 16-byte vectors: a row of the tile is
// a run of contiguous head slices of cache rows.
// fp32 path: tiles of 16x16x4 fp32 matrix instructions (f32_tile_kernel).  bf16 shapes that no tile takes: one wave per output.
#include <algorithm>

#include "ctrl_device.h"

namespace adore {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

// The same tile kernel serves the three projections of the path:
//   REBUILD  C = X[b][rebuilt_pos] . W_kv^T         -> head slices scattered into the freed cache slots
//   QKV      C = X_rows . [W_q ; W_kv]^T            -> query rows to a dense buffer, K/V slices scattered into the
//            slots of the rebuilt tokens and of the current token (rebuild forward, Sec. 2.3)
//   OPROJ    C = O_rows . W_o^T + X_rows (residual) -> dense rows, the next layer's input
// and one more product of the same shape family, the controller's input projection over a prompt chunk:
//   PLAIN    C = X_rows . W^T                        -> dense fp32 rows, no rounding
// TAIL is REBUILD with the workgroups of a StepTail in front (an instance of its own: the others stay as they are).
enum { MODE_REBUILD = 0, MODE_QKV = 1, MODE_OPROJ = 2, MODE_PLAIN = 3, MODE_TAIL = 4 };

struct GemmArgs {
  const void *X;               // A operand: [B][N_max][D] gathered by position, or dense rows [M][D]
  const void *W;               // [N][D]  (QKV: W_kv, the rows of columns >= H*d)
  const void *Wq;              // QKV: [H*d][D], the rows of columns < H*d
  void *Kc, *Vc;               // [B][H][K][d] of this layer
  void *Out;                   // QKV: query rows [M][H*d]; OPROJ: output rows [.][N]; PLAIN: fp32 rows [M][N]
  const void *Res;             // OPROJ: residual rows, gathered by position or dense like X
  const int32_t *rebuilt_pos;  // [B][Rdim]
  const int32_t *free_list;    // [B][H][R1]
  const int32_t *insert_slot;  // [B][H]    QKV: the slot of the current token
  int32_t *map_dst, *map_out;  // REBUILD: slot maps [B][H][K] that get the rebuilt tokens' positions, or null
  int B, H, d, D, K, N_max, r, R1, Rdim, M, N;   // D = length of the contraction
  int tiles_m, tiles_n;
  // Rows.  The tile kernel takes the rebuilt tokens: row mi = (b, j) = (mi / r, mi % r), rank j of sequence b.
  // The current token of every sequence (one row each) goes through cur_rows_kernel.  Dense row buffers hold
  // xrps rows per sequence: rank j at row b * xrps + j, the current token at row b * xrps + r.
  int xrps;
  int cur_pos;                 // position of the current token
  int a_gather, res_gather;    // 1: the row of a token is [b][its position]; 0: its row in a dense buffer
  int out_rps, out_cur;        // OPROJ: rank j is written to row b * out_rps + j, the current token to b * out_rps + out_cur
  int n_cur;                   // QKV / OPROJ: the first n_cur workgroups of the tile launch take the current tokens' rows; TAIL: the tail
  int cur_ks;                  // ... with the contraction cut over cur_ks (1, 2, 4, 8) of a workgroup's waves
  const float2 *rope_cur;      // QKV: the workgroups of the current tokens' rows turn their query and key rows (same
                               // table; null: they do not)
  const float2 *rope;          // tile kernel: [N_max][d/2] (cos, sin), the key (and query) tiles turn their rows by
                               // position as they leave; null: no rotary embedding, or a pass of its own does it
  int tail_at;                 // TAIL: its first workgroup
  StepTail tail;               // TAIL
};

// A rank that stays empty (position -1: fewer tokens were chosen than the launch has rows for) reads row 0 of its
// sequence; nothing of it is written.
__device__ inline size_t row_by_position(const GemmArgs &a, int b, int j) {
  return size_t(b) * a.N_max + max(a.rebuilt_pos[size_t(b) * a.Rdim + j], 0);
}

// The current token's row of every sequence (rebuild forward) as workgroups of the tile kernel's launch.  B rows
// against the same weights are a skinny product that only streams W; the tile launches of the forward leave a
// fifth or more of the compute units without a tile, and these workgroups take them (one workgroup per unit:
// the kernel's LDS sees to that), so the rows cost no launch and no time of their own.  A wave multiplies 16
// sequences x 32 output columns; the 8 waves of a workgroup are cur_ks wide along the contraction and 8 / cur_ks
// wide along the columns (partial sums added through LDS in a fixed order), so that the launcher can make as
// many workgroups as there are units without a tile: what one unit can stream is bounded by what it can keep
// in flight (about 36 GB/s next to the tiles' traffic).  With so few units at work the rows of W must arrive as whole cache lines (operands loaded
// straight into the 16x16x32 operand layout cost the L1 a tag look-up per lane, about 25 GB/s per unit): a wave
// reads its 32 rows x 64 k as four coalesced 16-byte loads per lane, six such chunks in flight, and turns them
// into operands through 4 KB of LDS of its own (XOR-swizzled; only the wave itself reads and writes it, so no
// barrier).  Epilogue as in the tile kernel, one rounding.
constexpr int kCurCols = 256;   // output columns per workgroup in this role when the contraction is not cut
constexpr int kCurLds = 8 * 32 * 8 * 16 + 8 * 2 * 4 * 64 * 4 + 16 * kCurCols * 2;   // the waves' tiles, their sums, the rounded rows

template <int MODE>
__device__ inline void cur_rows_role(const GemmArgs &a, int e, u32x4 *smem) {
  constexpr int U = 6;                                  // chunks of 64 k in flight
  const int ks = a.cur_ks;
  const int wg_cols = kCurCols / ks;
  const int wgs_n = a.N / wg_cols;
  const int sb = e / wgs_n, jn = e - sb * wgs_n;
  const int t0 = sb * 16;
  if (t0 >= a.B) return;                                // workgroups that only pad the launch
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane & 15, g = lane >> 4;
  const int kpart = wave % ks;                          // this wave's part of the contraction
  const int j0 = jn * wg_cols + (wave / ks) * 32;
  const int Hd = a.H * a.d;
  const int bb = min(t0 + c, a.B - 1);                  // padded rows read a valid sequence; dropped at the store
  const size_t xrow = a.a_gather ? size_t(bb) * a.N_max + a.cur_pos : size_t(bb) * a.xrps + a.r;
  const u32x4 *pa = reinterpret_cast<const u32x4 *>(static_cast<const bf16_t *>(a.X) + xrow * a.D) + g;
  // W: lane (row8 = lane / 8, chunk = lane % 8) loads 16 bytes of row 8 i + row8 of the wave's 32 rows
  const int lrow = lane >> 3, lch = lane & 7;
  const u32x4 *pw[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int n = j0 + 8 * i + lrow;
    const bf16_t *wrow = MODE == MODE_QKV && n < Hd ? static_cast<const bf16_t *>(a.Wq) + size_t(n) * a.D
                         : MODE == MODE_QKV         ? static_cast<const bf16_t *>(a.W) + size_t(n - Hd) * a.D
                                                    : static_cast<const bf16_t *>(a.W) + size_t(n) * a.D;
    pw[i] = reinterpret_cast<const u32x4 *>(wrow) + lch;
  }
  u32x4 *tile = smem + wave * (32 * 8);                 // [32 rows][8 chunks of 16 bytes]
  auto swz = [](int row, int chunk) { return row * 8 + (chunk ^ ((row >> 1) & 7)); };
  f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
  const int nchunks = a.D / 64 / ks;                    // chunks of this wave: kpart * nchunks ...
  const int chunk0 = kpart * nchunks;
  u32x4 vw[U][4], va[U][2];
#define CUR_LOAD(SET, CH)                                                                \
  {                                                                                      \
    _Pragma("unroll") for (int i = 0; i < 4; ++i) vw[SET][i] = pw[i][(chunk0 + (CH)) * 8]; \
    va[SET][0] = pa[(chunk0 + (CH)) * 8];                                                \
    va[SET][1] = pa[(chunk0 + (CH)) * 8 + 4];                                            \
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if (u < nchunks) CUR_LOAD(u, u)
  }
  for (int ch0 = 0; ch0 < nchunks; ch0 += U) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int ch = ch0 + u;
      if (ch < nchunks) {
#pragma unroll
        for (int i = 0; i < 4; ++i) tile[swz(8 * i + lrow, lch)] = vw[u][i];
        u32x4 fb[2][2];   // [step of 32 k][tile of 16 columns]
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
          for (int nc = 0; nc < 2; ++nc) fb[st][nc] = tile[swz(nc * 16 + c, st * 4 + g)];
        const u32x4 fa0 = va[u][0], fa1 = va[u][1];
        if (ch + U < nchunks) CUR_LOAD(u, ch + U)
#pragma unroll
        for (int nc = 0; nc < 2; ++nc) {
          acc[nc] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8 *>(&fa0),
                                                            *reinterpret_cast<const bf16x8 *>(&fb[0][nc]), acc[nc], 0, 0, 0);
          acc[nc] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8 *>(&fa1),
                                                            *reinterpret_cast<const bf16x8 *>(&fb[1][nc]), acc[nc], 0, 0, 0);
        }
      }
    }
  }
#undef CUR_LOAD
  const bool turning = MODE == MODE_QKV && a.rope_cur != nullptr;   // uniform over the launch
  if (ks > 1) {   // the parts of the contraction meet in the wave that holds part 0, in order
    float *red = reinterpret_cast<float *>(smem + 8 * (32 * 8));   // [8 waves][2][4][64], behind the waves' tiles
#pragma unroll
    for (int nc = 0; nc < 2; ++nc)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[((wave * 2 + nc) * 4 + v) * 64 + lane] = acc[nc][v];
    __syncthreads();
    if (kpart != 0 && !turning) return;   // (when the rows are turned below, every wave stays for the barrier)
    for (int p = 1; p < (kpart == 0 ? ks : 1); ++p)
#pragma unroll
      for (int nc = 0; nc < 2; ++nc)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[nc][v] += red[(((wave + p) * 2 + nc) * 4 + v) * 64 + lane];
  }
  if (turning) {
    // Rotary embedding: the workgroup's columns are whole heads of one section (launcher).  The rounded results meet
    // in an LDS tile [16 sequences][wg_cols]; then a thread takes 8 planes at a time (the 8-element vectors of
    // elements j.. and j + d/2.. of a head), turns query and key rows to the current position, and stores 16 bytes.
    uint16_t *sT = reinterpret_cast<uint16_t *>(smem + 8 * (32 * 8) + 8 * 2 * 4 * 64 / 4);   // behind tiles and sums
    if (kpart == 0) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int nc = 0; nc < 2; ++nc)
          sT[(4 * g + v) * wg_cols + (wave / ks) * 32 + nc * 16 + c] = f32_to_bf16_rne(acc[nc][v]);
    }
    __syncthreads();
    const int section = (jn * wg_cols) / Hd;             // 0: queries, 1: keys, 2: values
    const int half = a.d / 2;
    const bool turn = section <= 1;
    const int upr = turn ? wg_cols / 16 : wg_cols / 8;   // units per sequence: vector pairs, or single vectors
    for (int idx = tid; idx < 16 * upr; idx += 512) {
      const int seq = idx / upr, uu = idx - seq * upr;
      const int b = t0 + seq;
      if (b >= a.B) continue;
      int col, jp = 0;
      if (turn) {
        const int hv = half / 8, hh = uu / hv;
        jp = (uu - hh * hv) * 8;
        col = hh * a.d + jp;
      } else {
        col = uu * 8;
      }
      const int rem = jn * wg_cols + col - section * Hd;
      const int h = rem / a.d;
      bf16_t *dst;
      if (section == 0) {
        dst = static_cast<bf16_t *>(a.Out) + (size_t(b) * a.xrps + a.r) * Hd + rem;
      } else {
        const int slot = a.insert_slot[size_t(b) * a.H + h];
        dst = static_cast<bf16_t *>(section == 1 ? a.Kc : a.Vc) + ((size_t(b) * a.H + h) * a.K + slot) * a.d + (rem - h * a.d);
      }
      const u32x4 lo = *reinterpret_cast<const u32x4 *>(sT + seq * wg_cols + col);
      if (!turn) {
        *reinterpret_cast<u32x4 *>(dst) = lo;
        continue;
      }
      const u32x4 hi = *reinterpret_cast<const u32x4 *>(sT + seq * wg_cols + col + half);
      const float2 *cs = a.rope_cur + size_t(a.cur_pos) * half + jp;
      uint32_t rl[8], rh[8];
#pragma unroll
      for (int e2 = 0; e2 < 8; ++e2) {
        const float x = __uint_as_float(((lo[e2 / 2] >> (16 * (e2 & 1))) & 0xffffu) << 16);
        const float y = __uint_as_float(((hi[e2 / 2] >> (16 * (e2 & 1))) & 0xffffu) << 16);
        rl[e2] = f32_to_bf16_rne(rope_lo(x, y, cs[e2]));
        rh[e2] = f32_to_bf16_rne(rope_hi(x, y, cs[e2]));
      }
      *reinterpret_cast<u32x4 *>(dst) = u32x4{rl[0] | (rl[1] << 16), rl[2] | (rl[3] << 16), rl[4] | (rl[5] << 16), rl[6] | (rl[7] << 16)};
      *reinterpret_cast<u32x4 *>(dst + half) =
          u32x4{rh[0] | (rh[1] << 16), rh[2] | (rh[3] << 16), rh[4] | (rh[5] << 16), rh[6] | (rh[7] << 16)};
    }
    return;
  }
  // accumulator element v of lane (c, g): sequence 4*g + v of the block, column c of the tile
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int b = t0 + 4 * g + v;
    if (b >= a.B) continue;
#pragma unroll
    for (int nc = 0; nc < 2; ++nc) {
      float val = acc[nc][v];
      const int n = j0 + nc * 16 + c;
      bf16_t *dst;
      if (MODE == MODE_OPROJ) {
        const size_t rrow = a.res_gather ? size_t(b) * a.N_max + a.cur_pos : size_t(b) * a.xrps + a.r;
        val += to_float(static_cast<const bf16_t *>(a.Res)[rrow * a.N + n]);
        dst = static_cast<bf16_t *>(a.Out) + (size_t(b) * a.out_rps + a.out_cur) * a.N + n;
      } else {
        const int section = n / Hd, rem = n - section * Hd;
        const int h = rem / a.d;
        if (section == 0) {
          dst = static_cast<bf16_t *>(a.Out) + (size_t(b) * a.xrps + a.r) * Hd + rem;
        } else {
          const int slot = a.insert_slot[size_t(b) * a.H + h];
          dst = static_cast<bf16_t *>(section == 1 ? a.Kc : a.Vc) + ((size_t(b) * a.H + h) * a.K + slot) * a.d + (rem - h * a.d);
        }
      }
      dst->bits = f32_to_bf16_rne(val);
    }
  }
}

// Workgroup = 8 waves on a BM x BN output tile, k-steps of BK.
//   KG = 1: the waves form a WM x WN grid, each holding (BM/WM) x (BN/WN) of the tile.
//   KG = 2, 4, 8: that many such grids of fewer waves (k-groups); each multiplies its share of every k-step, so the
//           LDS read traffic is that of one grid while every SIMD still has two waves to switch
//           between, and a tile may be small.  The shares are added through LDS at the end, in order.
// A k-step costs a barrier and the trips through LDS behind it, some 500 cycles whatever its length: where a tile has little to multiply
// a step, or much, longer ones pay (N = 8192, D = 4096): M = 2048 133 -> 117 us (256x256, steps of 64 in two stages; 32 in four before).  Behind
// a decode step's attention (us a step): M = 128 44.7 -> 39.2 (64x64, steps of 128, two workgroups a unit; 128x32 of 64 before), 64 36.8 ->
// 30.0 (64x32, 128), 32 36.1 -> 27.5 (32x32, 256; the 128-row tile multiplied padding), 16 x 4096 x 4096 34.0 -> 23.1.  No faster there: 128x128
// and 128x64 in steps of 128 (two stages and three; with cold operands they are, 58.5 -> 54 and 47.5 -> 43.5), 256x128 in two stages or k-groups.
// More groups are shorter chains of fp32 sums: of 524288 rebuilt elements (4 x 32 rows, 16 heads of 128, D = 4096) 142 are not the 64-bit
// product's rounding with one group or two, 97 with four, 93 with eight; of 262144 at D = 2048 46, 25 and 15.
//   global -> registers: NS k-steps ahead (NS register sets, refilled right after they are spilled to LDS)
//   registers -> LDS:    LS stages; the tile of step ks+LS-1 is written while ks is read, one barrier per
//                        k-step.  With LS >= 3 the tile of ks+1 is complete during ks, so the first
//                        fragments of the next step are fetched before the barrier.
//   LDS -> fragments:    one 16-wide k-slice ahead of the MFMAs that use them
// sched_barrier keeps the compiler from sinking the fragment loads below the MFMAs they overlap with.  Where a wave has several
// MFMAs a slice, its LDS reads and writes and its reads from memory go out one behind each of them instead of in front of and
// behind them all (a wave issues in order, and an MFMA waits for the one before it): M = 512 43.0 -> 42.0 us, 1024 73.5 -> 71.8, 2048
// 133.5 -> 130.5, 256 35.0 -> 34.0 at N = 8192, D = 4096; two LDS operations behind each, whatever they are, 131.3 at M = 2048, the
// reads from memory in the last slice 135; with one MFMA a slice (128x32) 24.5 -> 25.5, left as it was.
template <int MODE_, int BM, int BN, int BK, int KG, int WM, int WN, int LS, int NS>
__global__ __launch_bounds__(512, BM * BN <= 64 * 64 && (MODE_ == MODE_REBUILD || MODE_ == MODE_TAIL) ? 4 : 2)   // two workgroups a unit, or one
void rebuild_mfma_kernel(const GemmArgs a) {
  constexpr int MODE = MODE_ == MODE_TAIL ? MODE_REBUILD : MODE_;
  constexpr int CH = BK / 8;             // 16-byte chunks per tile row
  constexpr int RPP = 512 / CH;          // tile rows the workgroup loads per pass
  constexpr int TM = BM / (WM * 32), TN = BN / (WN * 32);   // 32x32 blocks per wave
  static_assert(KG * WM * WN == 8, "eight waves");
  static_assert(TM * WM * 32 == BM && TN * WN * 32 == BN, "tile shape");
  constexpr int NA = BM / RPP, NB = (BN + RPP - 1) / RPP;   // 16-byte loads per thread and k-step
  static_assert(NA * RPP == BM && (NB * RPP == BN || BN < RPP), "tile rows");
  constexpr int KSUB = BK / 16 / KG;     // 16-wide k-slices per wave and k-step
  static_assert(KSUB == 2 || KSUB == 4, "fragment double buffering needs an even number of k-slices");
  constexpr int LEAD = LS - 1;
  constexpr bool kMixed = TM * TN > 1;
  // reads and stores of a k-step's tile all in the first k-slice, or spread over them (256x256: 120 -> 117 us; the others have too few
  // matrix instructions a slice: 64x64 33 -> 34.5)
  constexpr bool kSpread = TM * TN >= 8;
  constexpr int STAGE = (BM + BN) * CH;  // 16-byte units per LDS stage
  constexpr int LOOP_BYTES = LS * STAGE * 16;
  constexpr int RED_BYTES = (KG - 1) * WM * WN * TM * TN * 16 * 64 * 4;
  constexpr int OUT_BYTES = BM * BN * 2;
  constexpr int ROLE_BYTES = MODE_ == MODE_QKV || MODE_ == MODE_OPROJ ? kCurLds : MODE_ == MODE_TAIL ? kStepTailLds * 4 : 0;
  constexpr int SMEM_BYTES = std::max({LOOP_BYTES, RED_BYTES, OUT_BYTES, ROLE_BYTES});
  constexpr int NH_MAX = BN / 64 > 0 ? BN / 64 : 1;
  // one LDS block: the stages during the k-loop, then the upper k-group's accumulators, then the bf16 output tile
  __shared__ u32x4 smem[SMEM_BYTES / 16];
  __shared__ long long s_dst[BM * NH_MAX];   // element offset of each output row slice in its destination, -1 = none
  __shared__ long long s_res[MODE == MODE_OPROJ ? BM : 1];   // element offset of each row's residual, -1 = none
  __shared__ int s_rpos[MODE == MODE_REBUILD || MODE == MODE_QKV ? BM : 1];   // position of each row's token
  // rows are 256 or 512 B (BK = 128, 256), 128 B (64) or 64 B (32): 16 consecutive rows at one chunk index hit 16 different bank groups
  auto swz = [](int row, int chunk) {
    return row * CH + (chunk ^ (CH >= 16 ? row & 15 : CH == 8 ? (row >> 1) & 7 : (row >> 2) & 3));
  };

  int bx = blockIdx.x;
  if constexpr (MODE == MODE_QKV || MODE == MODE_OPROJ) {
    if (bx < a.n_cur) {   // uniform over the workgroup; n_cur is a multiple of 8, so the tiles keep their XCDs
      cur_rows_role<MODE>(a, bx, smem);
      return;
    }
    bx -= a.n_cur;
  }
  if constexpr (MODE_ == MODE_TAIL) {
    // in front of the tiles (n_cur, a multiple of 8) or behind them (n_cur = 0; tail_at); uniform over the workgroup
    const int e = bx - a.tail_at;
    if (e >= 0 && e < max(a.n_cur, a.tail.n)) {
      if (e < a.tail.n) step_tail_role<512>(a.tail, e, reinterpret_cast<float *>(smem));
      return;
    }
    bx -= a.n_cur;
  }
  const int total = a.tiles_m * a.tiles_n;
  const int per_xcd = (total + 7) / 8;
  const int lin = (bx & 7) * per_xcd + (bx >> 3);
  if (lin >= total) return;
  // the tiles of a W panel on one XCD; PLAIN, whose X is the larger operand and N a few tiles: those of a panel of X
  const int tn = MODE == MODE_PLAIN ? lin % a.tiles_n : lin / a.tiles_m, tm = MODE == MODE_PLAIN ? lin / a.tiles_n : lin - tn * a.tiles_m;
  const int m0 = tm * BM, n0 = tn * BN;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kgrp = wave / (WM * WN), wm = (wave / WN) % WM, wn = wave % WN;

  const int Hd = a.H * a.d;
  const int lchunk = tid % CH, lrow = tid / CH;   // rows lrow + RPP*i
  const bool b_on = BN >= RPP || lrow < BN;       // narrow tiles: only some threads load W rows
  const u32x4 *gA[NA], *gB[NB];
  const bf16_t *X = static_cast<const bf16_t *>(a.X);
  const bf16_t *W = MODE == MODE_QKV ? (n0 < Hd ? static_cast<const bf16_t *>(a.Wq) + size_t(n0) * a.D
                                                  : static_cast<const bf16_t *>(a.W) + size_t(n0 - Hd) * a.D)
                                     : static_cast<const bf16_t *>(a.W) + size_t(n0) * a.D;
  // Rotary embedding: the tiles of the sections that are turned hold whole planes.  One that is narrower than a head takes half of its
  // columns from the head's lower half and half of them, d / 2 further on, from its upper one (a pass of its own behind the launch: 18.3 ->
  // 15.8 us a step at 3 sequences of 12 heads of 64, 28.5 -> 26.0 at 16 of 16 heads of 128, 42.3 -> 39.2 at 4 of 32).
  const int section = MODE == MODE_OPROJ || MODE == MODE_PLAIN ? 0 : n0 / Hd;   // REBUILD: K, V; QKV: Q, K, V (a tile lies in one)
  const bool turn = (MODE == MODE_REBUILD ? section == 0 : MODE == MODE_QKV ? section <= 1 : false) && a.rope != nullptr;
  const bool paired = turn && BN < a.d;
  const int piece = paired ? n0 % a.d / BN : 0;   // which part of the head's planes
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    int nrow = b_on ? lrow + RPP * i : 0;
    if (paired) nrow += nrow < BN / 2 ? -piece * (BN / 2) : a.d / 2 - (piece + 1) * (BN / 2);   // (counted from the head's column piece * BN)
    gB[i] = reinterpret_cast<const u32x4 *>(W + ptrdiff_t(nrow) * a.D) + lchunk;
  }
  const int nk = a.D / BK;
  u32x4 ra[NS][NA], rb[NS][NB];
#define SA(ST) (smem + (ST) * STAGE)
#define SB(ST) (smem + (ST) * STAGE + BM * CH)
// PART: all of a tile's rows (-1), or the share of k-slice PART of a step
#define IN_PART(I, PART) ((PART) < 0 || (I) * KSUB / (NA + NB) == (PART))
#define GLOAD_A(SET, KS, PART)                                                           \
  { _Pragma("unroll") for (int i = 0; i < NA; ++i) if (IN_PART(i, PART)) ra[SET][i] = gA[i][(KS) * CH]; }
#define GLOAD_B(SET, KS, PART)                                                           \
  { _Pragma("unroll") for (int i = 0; i < NB; ++i) if (IN_PART(NA + i, PART)) rb[SET][i] = gB[i][(KS) * CH]; }
#define GLOAD(SET, KS, PART) { GLOAD_A(SET, KS, PART) GLOAD_B(SET, KS, PART) }
#define LSTORE(SET, ST, PART)                                                            \
  {                                                                                      \
    _Pragma("unroll") for (int i = 0; i < NA; ++i)                                       \
      if (IN_PART(i, PART)) SA(ST)[swz(lrow + RPP * i, lchunk)] = ra[SET][i];            \
    if (b_on) {                                                                          \
      _Pragma("unroll") for (int i = 0; i < NB; ++i)                                     \
        if (IN_PART(NA + i, PART)) SB(ST)[swz(lrow + RPP * i, lchunk)] = rb[SET][i];     \
    }                                                                                    \
  }
#define FRAGS(BUF, ST, KK)                                                               \
  {                                                                                      \
    const int ch_ = (KK) * 2 + (lane >> 5);                                              \
    _Pragma("unroll") for (int i = 0; i < TM; ++i) {                                     \
      const u32x4 va_ = SA(ST)[swz((wm * TM + i) * 32 + (lane & 31), ch_)];              \
      fa[BUF][i] = *reinterpret_cast<const bf16x8 *>(&va_);                              \
    }                                                                                    \
    _Pragma("unroll") for (int j = 0; j < TN; ++j) {                                     \
      const u32x4 vb_ = SB(ST)[swz((wn * TN + j) * 32 + (lane & 31), ch_)];              \
      fb[BUF][j] = *reinterpret_cast<const bf16x8 *>(&vb_);                              \
    }                                                                                    \
  }
#define MFMAS(BUF)                                                                       \
  _Pragma("unroll") for (int i = 0; i < TM; ++i)                                         \
    _Pragma("unroll") for (int j = 0; j < TN; ++j)                                       \
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[BUF][i], fb[BUF][j], acc[i][j], 0, 0, 0);

  // prologue: tiles 0 .. LEAD-1 to LDS, tiles LEAD .. LEAD+NS-1 into the register sets (set of tile t = t % NS).
  // Everything read from memory here is issued before anything is waited for: the W rows of the first NS tiles
  // (they depend on nothing), the positions of the gathered rows, the A rows, the destination slots.  (A read of
  // what the previous kernel wrote takes a microsecond or two; one after the other they cost a tenth of the launch.)
#pragma unroll
  for (int t = 0; t < NS; ++t) {
    if (t < nk) { GLOAD_B(t, t, -1) }
  }
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int mi = m0 + lrow + RPP * i;
    size_t src_row = 0;
    if (mi < a.M) {
      const int b = mi / a.r, j = mi - b * a.r;
      src_row = a.a_gather ? row_by_position(a, b, j) : size_t(b) * a.xrps + j;
    }
    gA[i] = reinterpret_cast<const u32x4 *>(X + src_row * a.D) + lchunk;
  }
#pragma unroll
  for (int t = 0; t < NS; ++t) {
    if (t < nk) { GLOAD_A(t, t, -1) }
  }
  // where every row of the output tile goes: looked up now, used after the k-loop
  const int sw = MODE == MODE_OPROJ ? BN : a.d;   // width of a contiguous piece of an output row
  const int nh = BN / sw > 0 ? BN / sw : 1;       // pieces in one tile row
  for (int t = tid; MODE != MODE_PLAIN && t < BM * nh; t += 512) {
    const int row = t / nh, hh = t - row * nh;
    const int mi = m0 + row;
    long long off = -1;
    if (mi < a.M) {
      const int b = mi / a.r, j = mi - b * a.r;
      if (MODE == MODE_OPROJ) {
        off = (long long)(size_t(b) * a.out_rps + j) * a.N + n0;
      } else {
        const int rem = (n0 + hh * a.d) % Hd;
        const int h = rem / a.d;
        if (MODE == MODE_QKV && section == 0) {
          off = (long long)(size_t(b) * a.xrps + j) * Hd + rem - piece * (BN / 2);
        } else {
          const int slot = a.free_list[(size_t(b) * a.H + h) * a.R1 + j];
          off = ((long long)(size_t(b) * a.H + h) * a.K + slot) * a.d + (rem - h * a.d) - piece * (BN / 2);
          // no slot: the head still holds this token's row (heads with maps of their own), or the rank is empty
          if (MODE == MODE_REBUILD && (slot < 0 || a.rebuilt_pos[size_t(b) * a.Rdim + j] < 0)) off = -1;
          if (MODE == MODE_REBUILD && a.map_dst && section == 0) {   // the K half's tiles visit every (token, head)
            const int pos = a.rebuilt_pos[size_t(b) * a.Rdim + j];
            a.map_dst[(size_t(b) * a.H + h) * a.K + slot] = pos;
            if (a.map_out) a.map_out[(size_t(b) * a.H + h) * a.K + slot] = pos;
          }
        }
      }
    }
    s_dst[t] = off;
  }
  if ((MODE == MODE_REBUILD || MODE == MODE_QKV) && a.rope) {
    for (int row = tid; row < BM; row += 512) {
      const int mi = min(m0 + row, a.M - 1);
      s_rpos[row] = max(a.rebuilt_pos[size_t(mi / a.r) * a.Rdim + (mi % a.r)], 0);
    }
  }
  if (MODE == MODE_OPROJ) {
    for (int row = tid; row < BM; row += 512) {
      const int mi = m0 + row;
      long long ro = -1;
      if (mi < a.M) {
        const int b = mi / a.r, j = mi - b * a.r;
        ro = (long long)(a.res_gather ? row_by_position(a, b, j) : size_t(b) * a.xrps + j) * a.N + n0;
      }
      s_res[row] = ro;
    }
  }
#pragma unroll
  for (int t = 0; t < LEAD; ++t) {
    if (t < nk) { LSTORE(t % NS, t, -1) }
    if (t + NS < nk) { GLOAD(t % NS, t + NS, -1) }   // the set just stored takes the tile NS further on
  }
  __syncthreads();

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // k-slice kk of this wave's k-group.  Of two groups each takes 32 of every 64 k, whatever the step: tiles of two groups all add up alike.
  auto slice = [&](int kk) { return KG == 2 ? (kk / 2) * 4 + kgrp * 2 + kk % 2 : KSUB * kgrp + kk; };
  bf16x8 fa[2][TM], fb[2][TN];     // double-buffered fragments
  FRAGS(0, 0, slice(0))
  int st = 0;                      // LDS stage of tile ks
  // One k-step.  IF(c) guards the parts that run out near the end; it is empty in the steady loop so
  // that the loop body is a single basic block (the wait counters are then tracked exactly).
#define KSTEP(U, KS, IF)                                                                 \
  {                                                                                      \
    const int st1 = st == LS - 1 ? 0 : st + 1;                                           \
    const int stw = st + LEAD >= LS ? st + LEAD - LS : st + LEAD;                        \
    _Pragma("unroll") for (int kk = 0; kk < KSUB; ++kk) {                                \
      if (kk + 1 < KSUB) {                                                               \
        FRAGS((kk + 1) & 1, st, slice(kk + 1))                                          \
      } else if (LS > 2) {                                                               \
        IF((KS) + 1 < nk) { FRAGS(0, st1, slice(0)) }                                       \
      }                                                                                  \
      if (!kMixed) {                                                                     \
        __builtin_amdgcn_sched_barrier(0);                                               \
        MFMAS(kk & 1)                                                                    \
        __builtin_amdgcn_sched_barrier(0);                                               \
      }                                                                                  \
      if (kSpread || kk == 0) {                                                          \
        IF((KS) + LEAD < nk) { LSTORE(((U) + LEAD) % NS, stw, kSpread ? kk : -1) }       \
        IF((KS) + LEAD + NS < nk) { GLOAD(((U) + LEAD) % NS, (KS) + LEAD + NS, kSpread ? kk : -1) } \
      }                                                                                  \
      if (kMixed) {                                                                      \
        MFMAS(kk & 1)                                                                    \
        _Pragma("unroll") for (int q = 0; q < TM * TN; ++q) {                            \
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   /* a matrix instruction */ \
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   /* an LDS read */          \
          __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);   /* an LDS write */         \
          __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   /* a read from memory */   \
        }                                                                                \
        __builtin_amdgcn_sched_barrier(0);                                               \
      }                                                                                  \
    }                                                                                    \
    __syncthreads();                                                                     \
    if (LS == 2) { IF((KS) + 1 < nk) { FRAGS(0, st1, slice(0)) } }                          \
    st = st1;                                                                            \
  }
#define ALWAYS(c)
#define GUARDED(c) if (c)
  const int nk_main = nk >= NS + LEAD ? (nk - NS - LEAD) / NS * NS : 0;   // k-steps that need no guard
  int ks0 = 0;
  for (; ks0 < nk_main; ks0 += NS) {
#pragma unroll
    for (int u = 0; u < NS; ++u) KSTEP(u, ks0 + u, ALWAYS)
  }
  for (; ks0 < nk; ks0 += NS) {
#pragma unroll
    for (int u = 0; u < NS; ++u) {
      if (ks0 + u < nk) KSTEP(u, ks0 + u, GUARDED)   // uniform over the workgroup: the barrier inside is safe
    }
  }
#undef KSTEP
#undef ALWAYS
#undef GUARDED
#undef GLOAD
#undef IN_PART
#undef GLOAD_A
#undef GLOAD_B
#undef LSTORE
#undef FRAGS
#undef MFMAS
#undef SA
#undef SB

  // ---- add the k-groups: all but the first hand their accumulators over through LDS ----
  if (KG > 1) {
    constexpr int kGroup = WM * WN * TM * TN * 16 * 64;
    float *red = reinterpret_cast<float *>(smem) + (wave % (WM * WN)) * (TM * TN * 16 * 64) + lane;
    if (kgrp > 0) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) red[(kgrp - 1) * kGroup + ((i * TN + j) * 16 + v) * 64] = acc[i][j][v];
    }
    __syncthreads();
    if (kgrp == 0) {
#pragma unroll
      for (int g = 0; g < KG - 1; ++g)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] += red[g * kGroup + ((i * TN + j) * 16 + v) * 64];
    }
    __syncthreads();   // the output tile below overwrites what was just read
  }
  if (MODE == MODE_PLAIN) {   // fp32 rows straight from the accumulators: 32 consecutive columns per row and block
    float *out = static_cast<float *>(a.Out);
    if (kgrp == 0) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int mi = m0 + (wm * TM + i) * 32 + 8 * (v / 4) + 4 * (lane >> 5) + (v % 4);
            if (mi < a.M) out[size_t(mi) * a.N + n0 + (wn * TN + j) * 32 + (lane & 31)] = acc[i][j][v];
          }
    }
    return;
  }
  // ---- round once to bf16 into a row-major LDS tile ----
  // accumulator element v of lane L: row 8*(v/4) + 4*(L/32) + v%4, column L%32 of its 32x32 block
  uint16_t *sOut = reinterpret_cast<uint16_t *>(smem);   // [BM][BN] bf16
  if (kgrp == 0) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int row = (wm * TM + i) * 32 + 8 * (v / 4) + 4 * (lane >> 5) + (v % 4);
          const int col = (wn * TN + j) * 32 + (lane & 31);
          float val = acc[i][j][v];
          if (MODE == MODE_OPROJ) {   // the residual joins before the one rounding
            const long long ro = s_res[row];
            if (ro >= 0) val += to_float(static_cast<const bf16_t *>(a.Res)[ro + col]);
          }
          sOut[row * BN + col] = f32_to_bf16_rne(val);
        }
  }
  __syncthreads();
  // ---- scatter: every output row slice is contiguous in the cache; 16 bytes per lane ----
  bf16_t *dst_half = static_cast<bf16_t *>(MODE == MODE_OPROJ ? a.Out
                                           : MODE == MODE_QKV ? (section == 0 ? a.Out : section == 1 ? a.Kc : a.Vc)
                                                              : (section == 0 ? a.Kc : a.Vc));
  // Rotary embedding (query and key tiles): the rounded row is turned by its
  // token's position on the way out, in fp32, and rounded again.  A thread takes 8 planes at a time: the 8-element
  // vectors of elements j and j + d/2 of a head, which share their angles; the angles of two such pairs are fetched
  // before either is used (a fetch costs a trip to the L2).
  if (turn) {
    constexpr int PV = BM * BN / 16;           // pairs of vectors in the tile
    const int half = a.d / 2;
    const int width = paired ? BN : a.d, hv = width / 16;   // columns of a head in the tile, pairs of vectors among them
    const int per_row = BN / 16;
    for (int i0 = 0; i0 < (PV + 511) / 512; i0 += 2) {
      float2 cs[2][8];
      u32x4 lo[2], hi[2];
      long long offv[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int idx = tid + (i0 + u) * 512;
        offv[u] = -1;
        if (idx < PV) {
          const int row = idx / per_row, rem = idx - row * per_row;
          const int hh = rem / hv, v = rem - hh * hv;
          const long long off = s_dst[row * nh + hh];
          if (off >= 0) {
            offv[u] = off + v * 8;
            const float2 *src = a.rope + size_t(s_rpos[row]) * half + piece * (BN / 2) + v * 8;
#pragma unroll
            for (int e = 0; e < 8; ++e) cs[u][e] = src[e];
            lo[u] = *reinterpret_cast<const u32x4 *>(sOut + row * BN + hh * width + v * 8);
            hi[u] = *reinterpret_cast<const u32x4 *>(sOut + row * BN + hh * width + width / 2 + v * 8);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (offv[u] < 0) continue;
        uint32_t rl[8], rh[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float x = __uint_as_float(((lo[u][e / 2] >> (16 * (e & 1))) & 0xffffu) << 16);
          const float y = __uint_as_float(((hi[u][e / 2] >> (16 * (e & 1))) & 0xffffu) << 16);
          rl[e] = f32_to_bf16_rne(rope_lo(x, y, cs[u][e]));
          rh[e] = f32_to_bf16_rne(rope_hi(x, y, cs[u][e]));
        }
        *reinterpret_cast<u32x4 *>(dst_half + offv[u]) =
            u32x4{rl[0] | (rl[1] << 16), rl[2] | (rl[3] << 16), rl[4] | (rl[5] << 16), rl[6] | (rl[7] << 16)};
        *reinterpret_cast<u32x4 *>(dst_half + offv[u] + half) =
            u32x4{rh[0] | (rh[1] << 16), rh[2] | (rh[3] << 16), rh[4] | (rh[5] << 16), rh[6] | (rh[7] << 16)};
      }
    }
    return;
  }
  constexpr int VPR = BN / 8;   // 16-byte vectors per tile row
  for (int idx = tid; idx < BM * VPR; idx += 512) {
    const int row = idx / VPR, vec = idx - row * VPR;
    const long long off = s_dst[row * nh + (vec * 8) / sw];
    if (off >= 0) {
      const u32x4 val = *reinterpret_cast<const u32x4 *>(sOut + row * BN + vec * 8);
      *reinterpret_cast<u32x4 *>(dst_half + off + (vec * 8) % sw) = val;
    }
  }
}

// The same product in fp32, on the fp32 matrix instructions; also the controller's input projection over a prompt (PLAIN).
// A workgroup owns a tile of 16 MT rows x 16 NT columns; its four waves take every fourth step of 16 k.  Lane (c, g) reads the
// 4 values at k = 16 s + 4 g of rows c of both operands (64-byte runs of every row; both sides use the same assignment, so
// the order of k does not matter), U steps in flight, straight into the operands: with four waves on different k the tile's
// rows pass the L1 once, and 4 MT NT instructions of 32 cycles per step hide the MT + NT reads.  Element e of the four goes to
// accumulator e, and after two steps (chains of eight products) the four are added up in 64 bits, as are the waves' sums at the
// end (chains through the whole row were further from 64 bits than the kernel before: 1.5e-7 against 1.0e-7 at k = 1024).
// One wave per output element, which read both rows from the L1 for every output, reached 4 to 6 TFLOP/s.  Before / on these
// tiles: 32 rows x 1024 columns x 512 13.7 / 5.7 us, 160 x 2048 x 1024 119 / 25 us (27 TFLOP/s), 128 x 4096 x 1024 189 / 26 us, 256 x 8192 x
// 4096 4440 / 288 us (60 TFLOP/s).  TAIL is an instance of its own here too: the tail's role inside REBUILD took the 16x16 tile from 52
// registers and 7 waves a SIMD to 115 and 3, the 32x32 one from 97 and 4 to 115 and 3 (256 x 4096 x 2048 71 -> 75 us, 32 x 1024 x 512 5.9 -> 6.3).
template <int MODE_, int MT, int NT, int U>
__global__ __launch_bounds__(256) void f32_tile_kernel(const GemmArgs a) {
  constexpr int MODE = MODE_ == MODE_TAIL ? MODE_REBUILD : MODE_;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane & 15, g = lane >> 4;
  __shared__ double red[4][MT * NT][16][17];
  int bx = blockIdx.x;
  if constexpr (MODE_ == MODE_TAIL) {
    static_assert(sizeof(red) >= kStepTailLds * sizeof(float), "room for the tail");
    if (bx < a.n_cur) {
      step_tail_role<256>(a.tail, bx, reinterpret_cast<float *>(red));
      return;
    }
    bx -= a.n_cur;
  }
  const int tm = bx / a.tiles_n, tn = bx - tm * a.tiles_n;
  const int m0 = tm * (16 * MT), n0 = tn * (16 * NT);
  const float *pa[MT], *pb[NT];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const int mi = min(m0 + 16 * i + c, a.M - 1);         // padded rows read a valid one; dropped at the store
    const int b = mi / a.r, j = mi - b * a.r;
    const size_t row = MODE == MODE_REBUILD ? row_by_position(a, b, j) : size_t(b) * a.xrps + j;
    pa[i] = static_cast<const float *>(a.X) + row * a.D;
  }
#pragma unroll
  for (int i = 0; i < NT; ++i) pb[i] = static_cast<const float *>(a.W) + size_t(min(n0 + 16 * i + c, a.N - 1)) * a.D;
  static_assert(U % 2 == 0, "sums are taken over two steps");
  double sum[MT][NT][4];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) sum[i][j][v] = 0.0;
  for (int k0 = wave * 16 + g * 4; k0 - g * 4 < a.D; k0 += 64 * U) {   // uniform over the wave; D is a multiple of 4
    f32x4 va[U][MT], vb[U][NT];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = k0 + 64 * u;
      const bool in = k < a.D;                            // behind the end of a row both operands are zero
#pragma unroll
      for (int i = 0; i < MT; ++i) va[u][i] = in ? *reinterpret_cast<const f32x4 *>(pa[i] + k) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < NT; ++i) vb[u][i] = in ? *reinterpret_cast<const f32x4 *>(pb[i] + k) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int u = 0; u < U; u += 2)
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          f32x4 acc[4];
#pragma unroll
          for (int e = 0; e < 4; ++e)
            acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(va[u][i][e], vb[u][j][e], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(va[u + 1][i][e], vb[u + 1][j][e], acc[e], 0, 0, 0);
#pragma unroll
          for (int v = 0; v < 4; ++v)
            sum[i][j][v] += (double(acc[0][v]) + double(acc[1][v])) + (double(acc[2][v]) + double(acc[3][v]));
        }
  }
  // sum v of lane (c, g): row 4*g + v, column c of its tile
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) {
#pragma unroll
      for (int v = 0; v < 4; ++v) red[wave][i * NT + j][4 * g + v][c] = sum[i][j][v];
    }
  __syncthreads();
  const int m = tid >> 4, nn = tid & 15;
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const int mi = m0 + 16 * i + m;
    if (mi >= a.M) continue;
    const int b = mi / a.r, rho = mi - b * a.r;
    const int pos = MODE == MODE_REBUILD ? a.rebuilt_pos[size_t(b) * a.Rdim + rho] : 0;
    if (pos < 0) continue;                                // an empty rank
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int n = n0 + 16 * j + nn, t = i * NT + j;
      if (n >= a.N) continue;
      const float val = float((red[0][t][m][nn] + red[1][t][m][nn]) + (red[2][t][m][nn] + red[3][t][m][nn]));
      if (MODE == MODE_PLAIN) {
        static_cast<float *>(a.Out)[size_t(mi) * a.N + n] = val;
        continue;
      }
      const int Hd = a.H * a.d;
      const int half = n / Hd, rem = n - half * Hd;
      const int h = rem / a.d, cc = rem - h * a.d;
      const int slot = a.free_list[(size_t(b) * a.H + h) * a.R1 + rho];
      if (slot < 0) continue;                             // the head still holds this token's row
      static_cast<float *>(half ? a.Vc : a.Kc)[((size_t(b) * a.H + h) * a.K + slot) * a.d + cc] = val;
      if (a.map_dst && half == 0 && cc == 0) {
        a.map_dst[(size_t(b) * a.H + h) * a.K + slot] = pos;
        if (a.map_out) a.map_out[(size_t(b) * a.H + h) * a.K + slot] = pos;
      }
    }
  }
}

// One wave per output element: dot of a gathered hidden row with one W row.
template <typename T>
__global__ __launch_bounds__(256) void rebuild_dot_kernel(const GemmArgs a) {
  constexpr int EPL = Vec16<T>::EPL;
  const size_t wid = (size_t(blockIdx.x) * blockDim.x + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (wid >= size_t(a.M) * a.N) return;
  const int mi = int(wid / a.N), nf = int(wid - size_t(mi) * a.N);
  const int b = mi / a.r, rho = mi - b * a.r;
  const int pos = a.rebuilt_pos[size_t(b) * a.Rdim + rho];
  if (pos < 0) return;   // an empty rank (uniform over the wave)
  const T *x = static_cast<const T *>(a.X) + (size_t(b) * a.N_max + pos) * a.D;
  const T *wrow = static_cast<const T *>(a.W) + size_t(nf) * a.D;
  float s = 0.f;
  for (int c = lane * EPL; c < a.D; c += 64 * EPL) {
    float xf[EPL], wf[EPL];
    Vec16<T>::load(x + c, xf);
    Vec16<T>::load(wrow + c, wf);
#pragma unroll
    for (int e = 0; e < EPL; ++e) s = fmaf(xf[e], wf[e], s);
  }
  s = wave_sum(s);
  if (lane == 0) {
    const int Hd = a.H * a.d;
    const int half = nf / Hd, rem = nf - half * Hd;
    const int h = rem / a.d, cc = rem - h * a.d;
    const int slot = a.free_list[(size_t(b) * a.H + h) * a.R1 + rho];
    if (slot < 0) return;   // the head still holds this token's row
    T *dst = static_cast<T *>(half ? a.Vc : a.Kc) + ((size_t(b) * a.H + h) * a.K + slot) * a.d + cc;
    store_elem(dst, s);
    if (a.map_dst && half == 0 && cc == 0) {
      a.map_dst[(size_t(b) * a.H + h) * a.K + slot] = pos;
      if (a.map_out) a.map_out[(size_t(b) * a.H + h) * a.K + slot] = pos;
    }
  }
}

// The forward's two projections (QKV, OPROJ) for storage types and widths the tile kernel does not take (fp32
// storage, widths that are no multiples of 128): one wave per output element, all r + 1 rows of a sequence alike
// (rank j < r, the current token at j = r).  fp32 products and sums, one rounding to the storage type.
template <typename T, int MODE>
__global__ __launch_bounds__(256) void proj_dot_kernel(const GemmArgs a) {
  constexpr int EPL = Vec16<T>::EPL;
  const size_t wid = (size_t(blockIdx.x) * blockDim.x + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  const int rps = a.r + 1;
  if (wid >= size_t(a.B) * rps * a.N) return;
  const int mi = int(wid / a.N), nf = int(wid - size_t(mi) * a.N);
  const int b = mi / rps, j = mi - b * rps;
  const bool cur = j == a.r;
  const int pos = cur ? a.cur_pos : a.rebuilt_pos[size_t(b) * a.Rdim + j];
  if (pos < 0) return;   // an empty rank (uniform over the wave)
  const int Hd = a.H * a.d;
  const size_t xrow = a.a_gather ? size_t(b) * a.N_max + pos : size_t(b) * a.xrps + j;
  const T *x = static_cast<const T *>(a.X) + xrow * a.D;
  const T *wrow = MODE == MODE_QKV && nf < Hd ? static_cast<const T *>(a.Wq) + size_t(nf) * a.D
                  : MODE == MODE_QKV          ? static_cast<const T *>(a.W) + size_t(nf - Hd) * a.D
                                              : static_cast<const T *>(a.W) + size_t(nf) * a.D;
  float s = 0.f;
  for (int c = lane * EPL; c < a.D; c += 64 * EPL) {
    float xf[EPL], wf[EPL];
    Vec16<T>::load(x + c, xf);
    Vec16<T>::load(wrow + c, wf);
#pragma unroll
    for (int e = 0; e < EPL; ++e) s = fmaf(xf[e], wf[e], s);
  }
  s = wave_sum(s);
  if (lane != 0) return;
  if (MODE == MODE_OPROJ) {
    const size_t rrow = a.res_gather ? size_t(b) * a.N_max + pos : size_t(b) * a.xrps + j;
    s += to_float(static_cast<const T *>(a.Res)[rrow * a.N + nf]);
    store_elem(static_cast<T *>(a.Out) + (size_t(b) * a.out_rps + (cur ? a.out_cur : j)) * a.N + nf, s);
    return;
  }
  const int section = nf / Hd, rem = nf - section * Hd;
  if (section == 0) {
    store_elem(static_cast<T *>(a.Out) + (size_t(b) * a.xrps + j) * Hd + rem, s);
    return;
  }
  const int h = rem / a.d, cc = rem - h * a.d;
  const int slot = cur ? a.insert_slot[size_t(b) * a.H + h] : a.free_list[(size_t(b) * a.H + h) * a.R1 + j];
  store_elem(static_cast<T *>(section == 1 ? a.Kc : a.Vc) + ((size_t(b) * a.H + h) * a.K + slot) * a.d + cc, s);
}

// The current token's row of every sequence (rebuild forward): B rows against the same weights, a skinny product
// that only streams W.  One workgroup owns 16 sequences x NC*16 output columns; its 4 waves cut the contraction
// into quarters (summed through LDS in a fixed order).  16x16x32 tiles; lane (c, g) holds, for matrix instruction
// s, the 8 values at k = (4*s + g)*8 of its quarter for row c, so every row is read in 64-byte runs (both operands
// use the same assignment, so the order of k does not matter).  Epilogue as in the tile kernel.
template <int MODE, int NC>
__global__ __launch_bounds__(256) void cur_rows_kernel(const GemmArgs a) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane & 15, g = lane >> 4;
  const int j0 = blockIdx.x * (16 * NC), t0 = blockIdx.y * 16;
  const int Hd = a.H * a.d;
  const int kw = a.D / 4;                               // k-range of one wave, a multiple of 32
  const int bb = min(t0 + c, a.B - 1);                  // padded rows read a valid sequence; dropped at the store
  const size_t xrow = a.a_gather ? size_t(bb) * a.N_max + a.cur_pos : size_t(bb) * a.xrps + a.r;
  const u32x4 *pa = reinterpret_cast<const u32x4 *>(static_cast<const bf16_t *>(a.X) + xrow * a.D + wave * kw) + g;
  const u32x4 *pb[NC];
#pragma unroll
  for (int nc = 0; nc < NC; ++nc) {
    const int n = j0 + nc * 16 + c;                     // N is a multiple of 16 * NC
    const bf16_t *wrow = MODE == MODE_QKV && n < Hd ? static_cast<const bf16_t *>(a.Wq) + size_t(n) * a.D
                         : MODE == MODE_QKV         ? static_cast<const bf16_t *>(a.W) + size_t(n - Hd) * a.D
                                                    : static_cast<const bf16_t *>(a.W) + size_t(n) * a.D;
    pb[nc] = reinterpret_cast<const u32x4 *>(wrow + wave * kw) + g;
  }
  f32x4 acc[NC];
#pragma unroll
  for (int nc = 0; nc < NC; ++nc) acc[nc] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int steps = kw / 32;
#define CUR_STEP(VA, VB)                                                                                     \
  _Pragma("unroll") for (int nc = 0; nc < NC; ++nc)                                                          \
    acc[nc] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8 *>(&(VA)),              \
                                                      *reinterpret_cast<const bf16x8 *>(&(VB)[nc]), acc[nc], 0, 0, 0);
  int s = 0;
  for (; s + 4 <= steps; s += 4) {          // four steps' loads in flight
    u32x4 va[4], vb[4][NC];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      va[u] = pa[(s + u) * 4];
#pragma unroll
      for (int nc = 0; nc < NC; ++nc) vb[u][nc] = pb[nc][(s + u) * 4];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) { CUR_STEP(va[u], vb[u]) }
  }
  for (; s < steps; ++s) {
    u32x4 va = pa[s * 4], vb[NC];
#pragma unroll
    for (int nc = 0; nc < NC; ++nc) vb[nc] = pb[nc][s * 4];
    CUR_STEP(va, vb)
  }
#undef CUR_STEP
  // accumulator element v of lane (c, g): sequence 4*g + v, column c
  __shared__ float red[4][NC][16][17];
#pragma unroll
  for (int nc = 0; nc < NC; ++nc)
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave][nc][4 * g + v][c] = acc[nc][v];
  __syncthreads();
  const int m = tid >> 4, nn = tid & 15;
  const int b = t0 + m;
  if (b >= a.B) return;
#pragma unroll
  for (int nc = 0; nc < NC; ++nc) {
    float val = (red[0][nc][m][nn] + red[1][nc][m][nn]) + (red[2][nc][m][nn] + red[3][nc][m][nn]);
    const int n = j0 + nc * 16 + nn;
    bf16_t *dst;
    if (MODE == MODE_OPROJ) {
      const size_t rrow = a.res_gather ? size_t(b) * a.N_max + a.cur_pos : size_t(b) * a.xrps + a.r;
      val += to_float(static_cast<const bf16_t *>(a.Res)[rrow * a.N + n]);
      dst = static_cast<bf16_t *>(a.Out) + (size_t(b) * a.out_rps + a.out_cur) * a.N + n;
    } else {
      const int section = n / Hd, rem = n - section * Hd;
      const int h = rem / a.d;
      if (section == 0) {
        dst = static_cast<bf16_t *>(a.Out) + (size_t(b) * a.xrps + a.r) * Hd + rem;
      } else {
        const int slot = a.insert_slot[size_t(b) * a.H + h];
        dst = static_cast<bf16_t *>(section == 1 ? a.Kc : a.Vc) + ((size_t(b) * a.H + h) * a.K + slot) * a.d + (rem - h * a.d);
      }
    }
    dst->bits = f32_to_bf16_rne(val);
  }
}

// The tile shapes the launcher chooses from.  The first five multiply any contraction that is a multiple of 64 (or 32) and are the ones the
// rebuild forward counts with (pick_with_riders).
struct TileShape {
  int bm, bn, bk;
  int per_unit;                // workgroups that share a compute unit
};
constexpr TileShape kTiles[] = {{256, 256, 32, 1}, {256, 128, 64, 1}, {128, 128, 64, 1}, {128, 64, 64, 1}, {128, 32, 64, 2},
                                {256, 256, 64, 1}, {64, 64, 128, 2}, {64, 32, 128, 2}, {32, 32, 256, 2}};
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]), kForwardTiles = 5;
bool takes_tail(int tile) { return tile >= 0 && kTiles[tile].bm <= 128; }   // short steps take none of the 256-wide ones

// kdim = length of the contraction; scatter modes write head slices (section = H*d columns of one kind)
bool tile_fits(const TileShape &t, int kdim, int section, int head_dim, bool dense) {
  if (kdim % t.bk != 0 || section % t.bn != 0) return false;
  return dense || t.bn % head_dim == 0 || head_dim % t.bn == 0;
}

// Time of one workgroup on its tile in microseconds at a contraction length of 4096, measured with one tile per
// compute unit; the launch takes ceil(tiles / 256) rounds of that.  The tile with the lowest
// estimate is used: a launch that fills three quarters of the units once (256x128 at M = 512, N = 12288: 192 tiles,
// 64 us) beats one that fills all of them one and a half times (128x128: 384 tiles, 88 us).
// Small products (us): 128 rows x 2048 columns x 1024 on 64 tiles of 128x32 12.5, on 256 of 32x32 8.4; 39 x 1536 x 768 11.0 / 7.8;
// 16 x 4096 x 4096 35 / 19.  The estimate counts shapes of which two share a unit like the others: 64x64 tiles between one and two a unit are
// charged twice, and lose M = 160 and 192 at N = 8192 to 128x64 (42.4 and 43.2 us a step, 40.8 and 41.2 on 64x64); 256x256 against 128x128 at M
// = 1280 127 / 157, 1536 141 / 181, and 98 / 119 with D = 2048.
constexpr float kTileMicros[kNumTiles] = {125.f, 66.f, 41.f, 40.f, 25.f, 112.f, 21.f, 17.f, 12.f};

// extra: workgroups that ride in the launch and need a compute unit each (the current tokens' rows); of the first `among` shapes
int pick_tile(int M, int N, int kdim, int section, int head_dim, bool dense, int extra = 0, int among = kNumTiles) {
  int pick = -1;
  float best = 0.f;
  for (int i = 0; i < among; ++i) {
    if (!tile_fits(kTiles[i], kdim, section, head_dim, dense)) continue;
    const long long tiles = (long long)((M + kTiles[i].bm - 1) / kTiles[i].bm) * (N / kTiles[i].bn);
    const float est = float((tiles + extra + 255) / 256) * kTileMicros[i];
    if (pick < 0 || est < best) {
      pick = i;
      best = est;
    }
  }
  if (const char *e = getenv("ADORE_GEMM_TILE")) {   // tuning runs: force a tile shape by index
    const int v = atoi(e);
    if (v >= 0 && v < among && tile_fits(kTiles[v], kdim, section, head_dim, dense)) pick = v;
  }
  return pick;
}

// 32x32 tiles where there are enough of them for every compute unit, otherwise 16x16 ones.
template <int MODE>
void launch_f32_tile(ScopedTimer &t, hipStream_t stream, GemmArgs &a) {
  const long long big = (long long)((a.M + 31) / 32) * ((a.N + 31) / 32);
  const int side = big >= 256 ? 32 : 16;
  a.tiles_m = (a.M + side - 1) / side;
  a.tiles_n = (a.N + side - 1) / side;
  const dim3 grid(unsigned(a.tiles_m) * unsigned(a.tiles_n) + (MODE == MODE_TAIL ? unsigned(a.n_cur) : 0u)), block(256);
  if (side == 32) ADORE_LAUNCH(t, (f32_tile_kernel<MODE, 2, 2, 2>), grid, block, 0, stream, a);
  else ADORE_LAUNCH(t, (f32_tile_kernel<MODE, 1, 1, 4>), grid, block, 0, stream, a);
}

template <int MODE>
void launch_tile(ScopedTimer &t, hipStream_t stream, int pick, GemmArgs &a) {
  a.tiles_m = (a.M + kTiles[pick].bm - 1) / kTiles[pick].bm;
  a.tiles_n = a.N / kTiles[pick].bn;
  const int total = a.tiles_m * a.tiles_n;
  a.tail_at = 0;
  const bool behind = MODE == MODE_TAIL && a.n_cur == 0;
  if (behind) a.tail_at = (total + 7) / 8 * 8;
  const dim3 grid((total + 7) / 8 * 8 + (behind ? a.tail.n : a.n_cur)), block(512);
#define TILE(...) ADORE_LAUNCH(t, (rebuild_mfma_kernel<MODE, __VA_ARGS__>), grid, block, 0, stream, a)
  constexpr bool kStep = MODE == MODE_REBUILD || MODE == MODE_TAIL;   // the forward takes none of the shapes guarded by it
  if constexpr (MODE != MODE_TAIL) {
    switch (pick) {
      //             BM   BN   BK KG WM WN LS NS
      case 0: if constexpr (kStep) TILE(256, 256, 32, 1, 2, 4, 4, 2); return;
      case 1: TILE(256, 128,  64, 1, 4, 2, 3, 2); return;
      case 5: TILE(256, 256,  64, 1, 2, 4, 2, 1); return;
    }
  }
  switch (pick) {
    case 2: TILE(128, 128,  64, 2, 2, 2, 3, 4); return;
    case 3: TILE(128,  64,  64, 2, 2, 2, 3, 4); return;
    case 4: if constexpr (kStep) TILE(128, 32, 64, 2, 4, 1, 3, 4); return;
    case 6: TILE(64,   64, 128, 2, 2, 2, 2, 3); return;
  }
  if constexpr (kStep) {
    if (pick == 7) TILE(64, 32, 128, 4, 2, 1, 2, 3);
    else TILE(32, 32, 256, 8, 1, 1, 2, 2);
  }
#undef TILE
}

void fill_common(adore_ctx *ctx, GemmArgs &a, int lists, int r) {
  const adore_config &c = ctx->cfg;
  a.Wq = nullptr; a.Out = nullptr; a.Res = nullptr; a.map_dst = a.map_out = nullptr;
  a.rebuilt_pos = ctx->rebuilt_pos[lists];
  a.free_list = ctx->free_list[lists];
  a.insert_slot = ctx->insert_slot[lists];
  a.B = c.batch; a.H = c.heads; a.d = c.head_dim; a.D = c.hidden; a.K = c.cache_slots;
  a.N_max = c.max_positions; a.r = r; a.R1 = c.rebuild_budget + 1; a.Rdim = max(c.rebuild_budget, 1);
  a.xrps = r; a.cur_pos = 0; a.a_gather = 1; a.res_gather = 0; a.out_rps = 0; a.out_cur = 0;
  a.tiles_m = a.tiles_n = 0;
  a.n_cur = 0;
  a.cur_ks = 1;
  a.rope = nullptr;
  a.rope_cur = nullptr;
  a.tail.n = 0;
  a.tail_at = 0;
}

}  // namespace

namespace {
// Workgroups of `threads` threads that a step's tail takes: a cell per sequence, and the rows whose splits are merged.
int step_tail_wgs(const adore_ctx *ctx, int threads) {
  const adore_config &c = ctx->cfg;
  const int per_wg = threads / c.head_dim;
  return c.batch + (ctx->nsplit > 1 ? (c.batch * c.heads + per_wg - 1) / per_wg : 0);
}
}  // namespace

// About how long a full rebuild (R tokens of every sequence, one layer) takes, in microseconds.
float rebuild_gemm_micros(const adore_config &c) {
  const int M = c.batch * c.rebuild_budget, Hd = c.heads * c.head_dim;
  if (M == 0) return 0.f;
  const int pick = c.dtype == ADORE_BF16 ? pick_tile(M, 2 * Hd, c.hidden, Hd, c.head_dim, false) : -1;
  if (pick < 0) return float(4.0 * M * Hd * c.hidden / (c.dtype == ADORE_F32 ? 40e6 : 6e6));   // 40 (27 to 60, see f32_tile_kernel) and 6 TFLOP/s
  const long long tiles = (long long)((M + kTiles[pick].bm - 1) / kTiles[pick].bm) * (2 * Hd / kTiles[pick].bn);
  return float((tiles + 255) / 256) * kTileMicros[pick] * c.hidden / 4096.f;
}

namespace {
// Tile of a launch that carries a tail of `wgs` workgroups: the same as without, so that the step's rows have the same bits either
// way.  The tail goes in front of the tiles where the chip holds all of them at once (14: both parts of the grid are padded to multiples of
// 8), otherwise behind them, where it starts as the first tiles end.
int pick_tile_with_tail(const adore_config &c, int M, int wgs, bool *front) {
  const int Hd = c.heads * c.head_dim, pick = pick_tile(M, 2 * Hd, c.hidden, Hd, c.head_dim, false);
  *front = false;
  if (pick < 0) return pick;
  const long long tiles = (long long)((M + kTiles[pick].bm - 1) / kTiles[pick].bm) * (2 * Hd / kTiles[pick].bn);
  *front = tiles + wgs + 14 <= 256 * kTiles[pick].per_unit;
  return pick;
}
}  // namespace

bool rebuild_gemm_takes_tail(const adore_ctx *ctx, int r, bool *beside) {
  const adore_config &c = ctx->cfg;
  bool front = false;
  const bool takes = r > 0 && (c.dtype == ADORE_F32 || takes_tail(pick_tile_with_tail(c, c.batch * r, step_tail_wgs(ctx, 512), &front)));
  if (beside) *beside = takes && front;
  return takes;
}

hipError_t launch_rebuild_gemm(adore_ctx *ctx, int layer, const void *hidden_layer, int lists, int r,
                               int32_t *map_dst, int32_t *map_out, const StepTail *tail) {
  const adore_config &c = ctx->cfg;
  if (r <= 0) return hipSuccess;
  const size_t es = elem_size(c);
  const size_t layer_bytes = size_t(c.batch) * c.heads * c.cache_slots * c.head_dim * es;
  GemmArgs a;
  fill_common(ctx, a, lists, r);
  a.X = hidden_layer;
  a.W = static_cast<const char *>(ctx->w.w_kv) + size_t(layer) * 2 * c.heads * c.head_dim * c.hidden * es;
  a.Kc = ctx->cache_k + layer * layer_bytes;
  a.Vc = ctx->cache_v + layer * layer_bytes;
  a.M = c.batch * r; a.N = 2 * c.heads * c.head_dim;
  a.map_dst = map_dst; a.map_out = map_out;
  ScopedTimer t(ctx, ADORE_KERNEL_REBUILD_GEMM, ctx->stream);
  bool front = false;
  const int pick = c.dtype != ADORE_BF16 ? -1
                   : tail ? pick_tile_with_tail(c, a.M, step_tail_wgs(ctx, 512), &front)
                          : pick_tile(a.M, a.N, c.hidden, c.heads * c.head_dim, c.head_dim, false);
  // the key tiles turn their rows themselves; behind the other kernels a pass of its own follows
  const bool rope = c.rope_base > 0.f;
  const bool turned = rope && pick >= 0;
  if (turned) a.rope = ctx->rope_f;
  if (tail) {
    a.tail = *tail;
    a.tail.n = step_tail_wgs(ctx, pick >= 0 ? 512 : 256);
    a.n_cur = pick < 0 ? a.tail.n : front ? (a.tail.n + 7) / 8 * 8 : 0;
  }
  if (pick >= 0 && tail) {
    launch_tile<MODE_TAIL>(t, ctx->stream, pick, a);
  } else if (pick >= 0) {
    launch_tile<MODE_REBUILD>(t, ctx->stream, pick, a);
  } else if (c.dtype == ADORE_F32 && tail) {
    launch_f32_tile<MODE_TAIL>(t, ctx->stream, a);
  } else if (c.dtype == ADORE_F32) {
    launch_f32_tile<MODE_REBUILD>(t, ctx->stream, a);
  } else {
    const size_t waves = size_t(a.M) * a.N;
    const unsigned blocks = unsigned((waves + 3) / 4);
    ADORE_LAUNCH(t, (rebuild_dot_kernel<bf16_t>), dim3(blocks), dim3(256), 0, ctx->stream, a);
  }
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && rope && !turned) e = launch_rope_rows(ctx, layer, lists, r, 0, r, false, 0);
  return e;
}

// ---- rebuild forward: the two projections around the attention of a layer ----------------------------
// Whether the tile kernels take both projections of this configuration; otherwise the forward runs them as one
// wave per output element (proj_dot_kernel).
bool fwd_gemm_supported(const adore_config &c) {
  const int Hd = c.heads * c.head_dim;
  return c.dtype == ADORE_BF16 && c.hidden % 128 == 0 && Hd % 128 == 0 &&
         pick_tile(1, 3 * Hd, c.hidden, Hd, c.head_dim, false) >= 0 &&
         pick_tile(1, c.hidden, Hd, c.hidden, c.head_dim, true) >= 0;
}

namespace {

// Workgroups that take the current tokens' rows inside the tile launch (a multiple of 8; see cur_rows_role) when
// the contraction is cut ks ways inside a workgroup, or 0 when the rows go through a launch of their own: a
// width that is no multiple of the role's 256 columns, or ADORE_FWD_CUR_SEPARATE=1 (for comparison runs).
int cur_row_riders(const GemmArgs &a, int ks) {
  if (a.N % kCurCols != 0 || a.D % (64 * ks) != 0) return 0;
  if (const char *e = getenv("ADORE_FWD_CUR_SEPARATE")) {
    if (atoi(e) != 0) return 0;
  }
  const int n = ((a.B + 15) / 16) * (a.N / (kCurCols / ks));
  return (n + 7) / 8 * 8;
}

// Tile shape and cut for a forward projection: the cheapest launch by pick_tile's estimate, with the rows of the
// current tokens spread over as many of the remaining units as a cut of the contraction allows.
int pick_with_riders(GemmArgs &a, int kdim, int section, int head_dim, bool dense) {
  a.n_cur = 0;
  a.cur_ks = 1;
  const int base = cur_row_riders(a, 1);
  const int pick = pick_tile(a.M, a.N, kdim, section, head_dim, dense, base, kForwardTiles);
  // The rows of a layer are the next one's input, without a norm between them here, and a last bit that falls the other way in an
  // early layer can be another key's softmax in a late one: so the choice is made among the shapes that were always there, and a
  // newer one stands in whose sums are the same (one k-group for one, two for two) and which fits wherever the old one does, widths and
  // contractions being multiples of 128 here (fwd_gemm_supported).  How finely the current tokens' rows are cut decides their sums as
  // well: it goes by the old shape's number of tiles.
  static_assert(kTiles[5].bn == kTiles[0].bn && 128 % kTiles[5].bk == 0 && 128 % kTiles[6].bk == 0 && 64 % kTiles[6].bn == 0, "the stand-ins fit");
  const int tile = pick == 0 ? 5 : pick == 4 ? 6 : pick;
  if (pick < 0 || base == 0) return tile;
  const int tiles = ((a.M + kTiles[pick].bm - 1) / kTiles[pick].bm) * (a.N / kTiles[pick].bn);
  const int rounds = (tiles + base + 255) / 256;
  int ks = 1;
  while (ks < 8 && cur_row_riders(a, ks * 2) > 0 && (tiles + cur_row_riders(a, ks * 2) + 255) / 256 <= rounds) ks *= 2;
  a.cur_ks = ks;
  a.n_cur = cur_row_riders(a, ks);
  return tile;
}

template <int MODE>
void launch_proj_dot(ScopedTimer &t, hipStream_t stream, bool bf16, const GemmArgs &a) {
  const size_t waves = size_t(a.B) * (a.r + 1) * a.N;
  const dim3 grid(unsigned((waves + 3) / 4)), block(256);
  if (bf16) {
    ADORE_LAUNCH(t, (proj_dot_kernel<bf16_t, MODE>), grid, block, 0, stream, a);
  } else {
    ADORE_LAUNCH(t, (proj_dot_kernel<float, MODE>), grid, block, 0, stream, a);
  }
}

template <int MODE>
void launch_cur_rows(ScopedTimer &t, hipStream_t stream, const GemmArgs &a) {
  const int seq_blocks = (a.B + 15) / 16;
  if (a.N % 32 == 0 && (a.N / 32) * seq_blocks >= 256) {
    ADORE_LAUNCH(t, (cur_rows_kernel<MODE, 2>), dim3(a.N / 32, seq_blocks), dim3(256), 0, stream, a);
  } else {
    ADORE_LAUNCH(t, (cur_rows_kernel<MODE, 1>), dim3(a.N / 16, seq_blocks), dim3(256), 0, stream, a);
  }
}

}  // namespace

// q, k, v of the r rebuilt tokens and the current token of every sequence.  x_rows: the rows entering this layer,
// either the embedding table [B][N_max][D] (by_position) or the dense rows [B][r+1][D] the previous layer wrote.
hipError_t launch_fwd_qkv(adore_ctx *ctx, int layer, const void *w_q_layer, const void *x_rows, bool by_position,
                          int r) {
  const adore_config &c = ctx->cfg;
  const int Hd = c.heads * c.head_dim;
  const size_t es = elem_size(c);
  const size_t layer_bytes = size_t(c.batch) * Hd * c.cache_slots * es;
  GemmArgs a;
  fill_common(ctx, a, ctx->cur, r);
  a.X = x_rows;
  a.W = static_cast<const char *>(ctx->w.w_kv) + size_t(layer) * 2 * Hd * c.hidden * es;
  a.Wq = w_q_layer;
  a.Kc = ctx->cache_k + layer * layer_bytes;
  a.Vc = ctx->cache_v + layer * layer_bytes;
  a.Out = ctx->fwd_q;
  a.xrps = r + 1; a.cur_pos = ctx->n; a.a_gather = by_position ? 1 : 0;
  a.M = c.batch * r; a.N = 3 * Hd;
  bool turned = false;   // the tiles turned the rebuilt tokens' query and key rows themselves
  bool cur_turned = false;   // ... and the workgroups of the current tokens' rows theirs
  if (!fwd_gemm_supported(c)) {   // all r + 1 rows of every sequence, one wave per output element
    {
      ScopedTimer t(ctx, ADORE_KERNEL_FWD_QKV, ctx->stream);
      launch_proj_dot<MODE_QKV>(t, ctx->stream, c.dtype == ADORE_BF16, a);
    }
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = launch_rope_rows(ctx, layer, ctx->cur, r, 0, r + 1, true, ctx->n);
    return e;
  }
  if (r > 0) {
    ScopedTimer t(ctx, ADORE_KERNEL_FWD_QKV, ctx->stream);
    const int pick = pick_with_riders(a, c.hidden, Hd, c.head_dim, false);
    if (pick < 0) return hipErrorInvalidValue;
    turned = c.rope_base > 0.f;
    if (turned) a.rope = ctx->rope_f;
    // the current tokens' rows riding in this launch turn themselves when a workgroup's columns are whole heads
    cur_turned = c.rope_base > 0.f && a.n_cur > 0 && (kCurCols / a.cur_ks) % c.head_dim == 0;
    if (cur_turned) a.rope_cur = ctx->rope_f;
    launch_tile<MODE_QKV>(t, ctx->stream, pick, a);
  }
  if (a.n_cur == 0) {
    ScopedTimer t(ctx, ADORE_KERNEL_FWD_QKV_CUR, ctx->stream);
    launch_cur_rows<MODE_QKV>(t, ctx->stream, a);
  }
  hipError_t e = hipGetLastError();
  // rotary embedding: whatever rows the launch above did not turn itself
  if (e == hipSuccess) e = launch_rope_rows(ctx, layer, ctx->cur, r, turned ? r : 0, cur_turned ? r : r + 1, true, ctx->n);
  return e;
}

// x' = round(x + W_o . o): residual rows like launch_fwd_qkv's x_rows; output rows at out[b * out_rps + j] for
// rank j and out[b * out_rps + out_cur] for the current token.
hipError_t launch_fwd_oproj(adore_ctx *ctx, const void *w_o_layer, const void *x_rows, bool by_position, void *out,
                            int out_rps, int out_cur, int r) {
  const adore_config &c = ctx->cfg;
  const int Hd = c.heads * c.head_dim;
  GemmArgs a;
  fill_common(ctx, a, ctx->cur, r);
  a.X = ctx->fwd_o;
  a.W = w_o_layer;
  a.Kc = a.Vc = nullptr;
  a.Out = out;
  a.Res = x_rows;
  a.D = Hd;
  a.xrps = r + 1; a.cur_pos = ctx->n; a.a_gather = 0; a.res_gather = by_position ? 1 : 0;
  a.out_rps = out_rps; a.out_cur = out_cur;
  a.M = c.batch * r; a.N = c.hidden;
  if (!fwd_gemm_supported(c)) {
    ScopedTimer t(ctx, ADORE_KERNEL_FWD_OPROJ, ctx->stream);
    launch_proj_dot<MODE_OPROJ>(t, ctx->stream, c.dtype == ADORE_BF16, a);
    return hipGetLastError();
  }
  if (r > 0) {
    ScopedTimer t(ctx, ADORE_KERNEL_FWD_OPROJ, ctx->stream);
    const int pick = pick_with_riders(a, Hd, c.hidden, c.head_dim, true);
    if (pick < 0) return hipErrorInvalidValue;
    launch_tile<MODE_OPROJ>(t, ctx->stream, pick, a);
  }
  if (a.n_cur == 0) {
    ScopedTimer t(ctx, ADORE_KERNEL_FWD_OPROJ_CUR, ctx->stream);
    launch_cur_rows<MODE_OPROJ>(t, ctx->stream, a);
  }
  return hipGetLastError();
}
// gi[tok][j] = W_ih[j][:] . x_tok for the ntok tokens of a prompt chunk (token b * per_seq + i at row
// b * seq_rows + i of x), fp32 sums: fp32 storage on the fp32 tiles, bf16 on the 128-wide tiles.  False if the shape does not
// fit them.
bool launch_plain_projection(adore_ctx *ctx, ScopedTimer &t, hipStream_t st, const void *x, const void *W, float *out,
                             int ntok, int per_seq, int seq_rows, int N, int D) {
  // 256 x 128 x 64 where its rounds over the compute units come out shorter than those of 128 x 128 x 64 (65536 tokens x 384 rows of 4096: 401 ->
  // 242 us, with the order of the tiles below; 8192 tokens, one round of either: 54 us for 66).  Its two groups of four waves cut D as the
  // narrow tile's do, so that a sum is the same either way (all of D in one chain per wave, twice as long: no faster);
  // one set of tiles on its way in registers is what that leaves room for (two: 26 registers spilled, 330 us).
  // (128-wide steps for both, which the wide one has no room for, or for one of them, would be other sums.)
  const long long wide = ((ntok + 255) / 256) * (N / 128), narrow = ((ntok + 127) / 128) * (N / 128);
  const int kTile = float((wide + 255) / 256) * kTileMicros[1] < float((narrow + 255) / 256) * kTileMicros[2] ? 1 : 2;
  const bool bf16 = ctx->cfg.dtype == ADORE_BF16;
  if (bf16 && (N % kTiles[kTile].bn != 0 || D % kTiles[kTile].bk != 0)) return false;
  GemmArgs a;
  fill_common(ctx, a, 0, per_seq);
  a.X = x; a.W = W; a.Out = out;
  a.Kc = a.Vc = nullptr;
  a.D = D; a.M = ntok; a.N = N;
  a.xrps = seq_rows; a.a_gather = 0;
  if (!bf16) {
    launch_f32_tile<MODE_PLAIN>(t, st, a);
    return true;
  }
  a.tiles_m = (a.M + kTiles[kTile].bm - 1) / kTiles[kTile].bm;
  a.tiles_n = a.N / kTiles[kTile].bn;
  const dim3 grid((a.tiles_m * a.tiles_n + 7) / 8 * 8), block(512);
  if (kTile == 1)
    ADORE_LAUNCH(t, (rebuild_mfma_kernel<MODE_PLAIN, 256, 128, 64, 2, 2, 2, 3, 1>), grid, block, 0, st, a);
  else
    ADORE_LAUNCH(t, (rebuild_mfma_kernel<MODE_PLAIN, 128, 128, 64, 2, 2, 2, 3, 4>), grid, block, 0, st, a);
  return true;
}

}  // namespace adore
