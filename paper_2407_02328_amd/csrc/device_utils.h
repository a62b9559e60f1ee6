// Device helpers: 16-byte storage loads, bf16 conversion, the ranking key.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "adore_internal.h"

namespace adore {

// ---- storage access: one 16-byte vector -> EPL floats ----------------------
template <typename T>
struct Vec16;

template <>
struct Vec16<float> {
  static constexpr int EPL = 4;  // elements per 16-byte load
  __device__ static __forceinline__ void load(const float *p, float (&f)[4]) {
    const float4 v = *reinterpret_cast<const float4 *>(p);
    f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
  }
  __device__ static __forceinline__ void copy(float *dst, const float *src) {
    *reinterpret_cast<float4 *>(dst) = *reinterpret_cast<const float4 *>(src);
  }
  // the same in two steps: the 16 bytes as they are, and their values
  typedef float4 Raw;
  __device__ static __forceinline__ Raw load_raw(const float *p) { return *reinterpret_cast<const float4 *>(p); }
  __device__ static __forceinline__ void store_raw(float *p, const Raw &v) { *reinterpret_cast<float4 *>(p) = v; }
  __device__ static __forceinline__ void values(const Raw &v, float (&f)[4]) {
    f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
  }
};

template <>
struct Vec16<bf16_t> {
  static constexpr int EPL = 8;
  __device__ static __forceinline__ void load(const bf16_t *p, float (&f)[8]) {
    const uint4 v = *reinterpret_cast<const uint4 *>(p);
    f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xffff0000u);
    f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xffff0000u);
    f[4] = __uint_as_float(v.z << 16); f[5] = __uint_as_float(v.z & 0xffff0000u);
    f[6] = __uint_as_float(v.w << 16); f[7] = __uint_as_float(v.w & 0xffff0000u);
  }
  __device__ static __forceinline__ void copy(bf16_t *dst, const bf16_t *src) {
    *reinterpret_cast<uint4 *>(dst) = *reinterpret_cast<const uint4 *>(src);
  }
  typedef uint4 Raw;
  __device__ static __forceinline__ Raw load_raw(const bf16_t *p) { return *reinterpret_cast<const uint4 *>(p); }
  __device__ static __forceinline__ void store_raw(bf16_t *p, const Raw &v) { *reinterpret_cast<uint4 *>(p) = v; }
  __device__ static __forceinline__ void values(const Raw &v, float (&f)[8]) {
    f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xffff0000u);
    f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xffff0000u);
    f[4] = __uint_as_float(v.z << 16); f[5] = __uint_as_float(v.z & 0xffff0000u);
    f[6] = __uint_as_float(v.w << 16); f[7] = __uint_as_float(v.w & 0xffff0000u);
  }
};

__device__ __forceinline__ float to_float(float v) { return v; }
__device__ __forceinline__ float to_float(bf16_t v) { return __uint_as_float(uint32_t(v.bits) << 16); }

// fp32 -> bf16, round to nearest, ties to even.  NaN stays NaN.
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return uint16_t((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return uint16_t(u >> 16);
}

// Rotary embedding of one plane: (lo, hi) = elements j and j + d/2 of a head, cs = (cos, sin) of the angle.
// fp64 for fp32 storage.  For bf16 storage fp32 is enough (its error is a thousandth of the spacing of the storage
// values); written with explicit fused operations so that every kernel that turns a row gets the same bits.
__device__ __forceinline__ double rope_lo(double lo, double hi, double2 cs) { return lo * cs.x - hi * cs.y; }
__device__ __forceinline__ double rope_hi(double lo, double hi, double2 cs) { return lo * cs.y + hi * cs.x; }
__device__ __forceinline__ float rope_lo(float lo, float hi, float2 cs) { return fmaf(lo, cs.x, -(hi * cs.y)); }
__device__ __forceinline__ float rope_hi(float lo, float hi, float2 cs) { return fmaf(lo, cs.y, hi * cs.x); }
__device__ __forceinline__ void store_elem(float *p, float v) { *p = v; }
__device__ __forceinline__ void store_elem(bf16_t *p, float v) { p->bits = f32_to_bf16_rne(v); }

// ---- ranking key ------------------------------------------------------------
// Tokens of one sequence are ranked by sigma (higher is better) and, between
// equal sigma, by position (lower is better).  The 64-bit key is monotone in
// that order: larger key = better token.  Keys of distinct positions differ.
// -0 is folded into +0, NaN is treated as 0.  A valid key is never 0.
__device__ __forceinline__ uint64_t rank_key(float sigma, int pos) {
  sigma = (sigma != sigma) ? 0.0f : sigma + 0.0f;
  uint32_t u = __float_as_uint(sigma);
  u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return (uint64_t(u) << 32) | uint64_t(0xffffffffu - uint32_t(pos));
}
__device__ __forceinline__ int key_pos(uint64_t key) { return int(0xffffffffu - uint32_t(key & 0xffffffffu)); }

// ---- wave helpers (64 lanes) ------------------------------------------------
// A shuffle is a trip through LDS; a lane's neighbours within its row of 16 come with the instruction that uses them (DPP), and rows
// and halves change places in registers (permlane swaps): the same sums in the same order.  All of these need their partners active.
// Shuffles before: attention launches with both selections 28.1 -> 26.5 us (16 sequences of 32 heads, H2O), 25.5 -> 24.8 (scores), 8.7 ->
// 7.5 (1 of 4 heads), the H2O choice 13.2 -> 12.3, the controller's cell on its side stream 14 -> 12.
template <int CTRL>
__device__ __forceinline__ float lane_dpp(uint32_t v) {
  return __uint_as_float(uint32_t(__builtin_amdgcn_update_dpp(0, int(v), CTRL, 0xf, 0xf, true)));
}
// v + the value of lane ^ OFF
template <int OFF>
__device__ __forceinline__ float add_lane_xor(float v) {
  static_assert(OFF == 1 || OFF == 2 || OFF == 4 || OFF == 8 || OFF == 16 || OFF == 32, "one bit of the lane");
  const uint32_t u = __float_as_uint(v);
  if constexpr (OFF == 32) {
    const auto s = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
  } else if constexpr (OFF == 16) {
    const auto s = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
  } else if constexpr (OFF == 8) {
    return v + lane_dpp<0x128>(u);                               // row_ror:8
  } else if constexpr (OFF == 4) {
    const int up = __builtin_amdgcn_update_dpp(0, int(u), 0x104, 0xf, 0x5, false);                       // row_shl:4 into quads 0 and 2
    return v + __uint_as_float(uint32_t(__builtin_amdgcn_update_dpp(up, int(u), 0x114, 0xf, 0xa, false)));   // row_shr:4 into 1 and 3
  } else {
    return v + lane_dpp<OFF == 2 ? 0x4e : 0xb1>(u);              // quad_perm
  }
}
// the larger of v and the value of lane ^ OFF
template <int OFF>
__device__ __forceinline__ float max_lane_xor(float v) {
  static_assert(OFF == 16 || OFF == 32, "rows or halves");
  const uint32_t u = __float_as_uint(v);
  if constexpr (OFF == 32) {
    const auto s = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1]));
  } else {
    const auto s = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1]));
  }
}
// Sum over groups of N lanes, in all of them: pairs N/2 apart first.
template <int N>
__device__ __forceinline__ float group_sum(float v) {
  if constexpr (N > 1) return group_sum<N / 2>(add_lane_xor<N / 2>(v));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) { return group_sum<64>(v); }

// Inclusive sum of lanes 0 .. own; all 64 lanes active.
__device__ __forceinline__ int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1, 2, 4, 8
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
  return v;
}
// All lanes' bits together; all 64 lanes active.  Wave-uniform.
__device__ __forceinline__ uint32_t wave_or(uint32_t u) {
  int v = int(u);
  v |= __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
  v |= __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v |= __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v |= __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v |= __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
  v |= __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
  return uint32_t(__builtin_amdgcn_readlane(v, 63));
}
__device__ __forceinline__ uint32_t wave_and(uint32_t u) { return ~wave_or(~u); }

// Scan of a 256-bin histogram from the top bin down: the bin in which the rank `need` (1 = the largest) falls, the
// rank left inside it, and how many entries it holds.  Lane l owns bins 255 - 4l .. 252 - 4l.  Wave-uniform results.
__device__ __forceinline__ void pick_bin(int c0, int c1, int c2, int c3, int lane, int need, int &bin, int &rest, int &inbin) {
  const int own = c0 + c1 + c2 + c3;
  const int incl = wave_scan(own), excl = incl - own;
  const bool mine = excl < need && need <= incl;   // exactly one lane: need <= the number of candidates
  int b = 252 - 4 * lane, r = need - excl - c0 - c1 - c2, n = c3;
  if (need <= excl + c0) {
    b = 255 - 4 * lane; r = need - excl; n = c0;
  } else if (need <= excl + c0 + c1) {
    b = 254 - 4 * lane; r = need - excl - c0; n = c1;
  } else if (need <= excl + c0 + c1 + c2) {
    b = 253 - 4 * lane; r = need - excl - c0 - c1; n = c2;
  }
  const int src = __builtin_ctzll(__builtin_amdgcn_ballot_w64(mine) | (uint64_t(1) << 63));
  bin = __builtin_amdgcn_readlane(b, src);
  rest = __builtin_amdgcn_readlane(r, src);
  inbin = __builtin_amdgcn_readlane(n, src);
}
// hist: 256 words, 16-byte aligned
__device__ __forceinline__ void pick_bin(const uint32_t *hist, int lane, int need, int &bin, int &rest, int &inbin) {
  const uint4 hq = *reinterpret_cast<const uint4 *>(hist + 252 - 4 * lane);
  pick_bin(int(hq.w), int(hq.z), int(hq.y), int(hq.x), lane, need, bin, rest, inbin);
}

// One wave's LDS operations run in order; this keeps the compiler from moving them across the point.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

}  // namespace adore
