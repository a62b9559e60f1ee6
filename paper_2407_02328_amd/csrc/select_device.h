// Device code of the two selections of a decode step, shared by the stand-alone selection kernels and by the
// attention launch that carries them as extra workgroups.
//
// Ranking uses the 64-bit integer key of device_utils.h, so every selection has exactly one answer and is
// reproducible bit for bit.  Release is a wave-level binary radix select over the K keys of a row held in
// registers (K <= 1024).  The per-sequence choice is a most-significant-digit radix select over up to N_max
// keys with 8-bit digits and an LDS histogram; it stops as soon as the digit bucket holding the r-th key is
// taken whole.
#pragma once

#include "device_utils.h"

namespace adore {

// Radix select.  key_of(i) for i in [0, ncand) returns the key of candidate i or 0
// if i is not a candidate.  Finds (*thr, *shift) such that exactly c candidates
// have (key >> shift) >= thr.  Needs 1 <= c <= number of candidates.
// s_hist: 256 uints; s_ctl: 4 uint64.  All threads of the block (whole waves) must call it.
// The first digit starts at the highest bit in which two candidates differ: scores of one sequence share most of their
// exponent, so that a digit from the top of the key would put nearly all of them into one or two bins (atomics on one
// address, 64 in turn per wave) and tell nothing.  4 sequences of 8200 tokens: release 22.4 -> 19.0 us, choice 19.2 -> 17.1 us.
template <class KeyFn>
__device__ __forceinline__ void radix_select(KeyFn key_of, int ncand, int c, uint32_t *s_hist, uint64_t *s_ctl,
                                    uint64_t *thr, int *shift_out) {
  uint32_t *s_or = reinterpret_cast<uint32_t *>(s_ctl + 3), *s_and = s_or + 1;   // upper words of all candidates
  if (threadIdx.x == 0) {
    *s_or = 0u;
    *s_and = ~0u;
  }
  __syncthreads();
  uint32_t or_hi = 0u, and_hi = ~0u;
  for (int i = threadIdx.x; i < ncand; i += blockDim.x) {
    const uint64_t key = key_of(i);
    if (key != 0) {
      or_hi |= uint32_t(key >> 32);
      and_hi &= uint32_t(key >> 32);
    }
  }
  or_hi = wave_or(or_hi);
  and_hi = wave_and(and_hi);
  if ((threadIdx.x & 63) == 0) {
    atomicOr(s_or, or_hi);
    atomicAnd(s_and, and_hi);
  }
  __syncthreads();
  const uint32_t diff = *s_or & ~*s_and;
  // bits from `prev` up are decided; equal scores: the positions decide (below 2^24, so the key's lower word starts 0xff)
  int prev = diff ? 64 - __clz(int(diff)) : 24;
  uint64_t prefix = prev == 64 ? 0 : ((uint64_t(*s_and) << 32) | 0xff000000u) >> prev;
  int remaining = c;
  int shift = 0;
  for (;;) {
    shift = max(prev - 8, 0);
    const uint32_t digits = (1u << (prev - shift)) - 1u;
    for (int t = threadIdx.x; t < 256; t += blockDim.x) s_hist[t] = 0;
    __syncthreads();
    for (int i = threadIdx.x; i < ncand; i += blockDim.x) {
      const uint64_t key = key_of(i);
      if (key != 0 && (prev == 64 || (key >> prev) == prefix)) {
        atomicAdd(&s_hist[uint32_t(key >> shift) & digits], 1u);
      }
    }
    __syncthreads();
    // four waves find the bin each by itself, without an exchange and its barrier; of sixteen one does
    const int lane = threadIdx.x & 63;
    const bool all = blockDim.x <= 256;
    int digit = 0, rest = 0, inbin = 0;
    if (all || threadIdx.x < 64) {
      const uint32_t *top = s_hist + 252 - 4 * lane;
      pick_bin(int(top[3]), int(top[2]), int(top[1]), int(top[0]), lane, remaining, digit, rest, inbin);
      if (!all && lane == 0) {
        s_ctl[0] = uint64_t(uint32_t(digit));
        s_ctl[1] = uint64_t(uint32_t(rest));
        s_ctl[2] = uint64_t(uint32_t(inbin));
      }
    }
    if (!all) {
      __syncthreads();
      digit = int(s_ctl[0]);
      rest = int(s_ctl[1]);
      inbin = int(s_ctl[2]);
    }
    prefix = (prefix << (prev - shift)) | uint32_t(digit);
    remaining = rest;
    const bool whole_bucket = inbin == rest;
    __syncthreads();                              // the bins are read before the next pass clears them
    prev = shift;
    if (whole_bucket || shift == 0) break;   // the last digit used: keys are distinct, the bucket held one key
  }
  *thr = prefix;
  *shift_out = shift;
}

// Gathers the c selected keys (those with (key >> shift) >= thr) into s_keys in any
// order, then writes their positions best first to out_pos[0..c).  s_count: one int.
template <class KeyFn>
__device__ __forceinline__ void collect_sorted(KeyFn key_of, int ncand, int c, uint64_t thr, int shift,
                                      uint64_t *s_keys, int *s_count, int32_t *out_pos) {
  if (threadIdx.x == 0) *s_count = 0;
  __syncthreads();
  for (int i = threadIdx.x; i < ncand; i += blockDim.x) {
    const uint64_t key = key_of(i);
    if (key != 0 && (key >> shift) >= thr) {
      const int idx = atomicAdd(s_count, 1);
      if (idx < c) s_keys[idx] = key;
    }
  }
  __syncthreads();
  for (int t = threadIdx.x; t < c; t += blockDim.x) {
    const uint64_t mine = s_keys[t];
    int rank = 0;
#pragma unroll 8
    for (int j = 0; j < c; ++j) rank += s_keys[j] > mine;
    out_pos[rank] = key_pos(mine);
  }
  __syncthreads();
}

// The best r of few: radix_select and collect_sorted meet at a barrier four times a digit and three more, which is what a short
// choice costs (5 us for 32 of 1024).  Here each of the workgroup's four waves finds the best r of its quarter alone, and the at most
// 4 r that are left are ranked against each other (3 us).
constexpr int kFewRanks = 64;        // r up to here: 4 r threads rank 4 r keys

// One wave: leaves the best r of the keys [first, end) (0: none) in out[0 .. r), in any order, and zeros behind them where there are
// fewer.  hist: 256 words of the wave's own, 16-byte aligned.
__device__ __forceinline__ void wave_best(const uint64_t *s_key, int first, int end, int r, uint32_t *hist, uint64_t *out) {
  const int lane = threadIdx.x & 63;
  uint32_t or_hi = 0u, and_hi = ~0u;
  int count = 0;
  for (int i0 = first; i0 < end; i0 += 64) {                    // (the whole wave, for the ballots)
    const uint64_t key = i0 + lane < end ? s_key[i0 + lane] : 0;
    if (key != 0) {
      or_hi |= uint32_t(key >> 32);
      and_hi &= uint32_t(key >> 32);
    }
    count += __popcll(__ballot(key != 0));
  }
  uint64_t thr = 0;
  int shift = 0;
  if (count > r) {
    or_hi = wave_or(or_hi);
    and_hi = wave_and(and_hi);
    const uint32_t diff = or_hi & ~and_hi;                      // as in radix_select from here on
    int prev = diff ? 64 - __clz(int(diff)) : 24, remaining = r;
    uint64_t prefix = prev == 64 ? 0 : ((uint64_t(and_hi) << 32) | 0xff000000u) >> prev;
    for (;;) {
      shift = max(prev - 8, 0);
      const uint32_t digits = (1u << (prev - shift)) - 1u;
      *reinterpret_cast<uint4 *>(hist + 4 * lane) = uint4{0u, 0u, 0u, 0u};
      wave_lds_fence();
      for (int i = first + lane; i < end; i += 64) {
        const uint64_t key = s_key[i];
        if (key != 0 && (prev == 64 || (key >> prev) == prefix)) atomicAdd(&hist[uint32_t(key >> shift) & digits], 1u);
      }
      wave_lds_fence();
      int digit, rest, inbin;
      pick_bin(hist, lane, remaining, digit, rest, inbin);
      wave_lds_fence();                                         // the bins are read before the next pass clears them
      prefix = (prefix << (prev - shift)) | uint32_t(digit);
      remaining = rest;
      prev = shift;
      if (inbin == rest || shift == 0) break;
    }
    thr = prefix;
  }
  int taken = 0;
  for (int i0 = first; i0 < end; i0 += 64) {
    const uint64_t key = i0 + lane < end ? s_key[i0 + lane] : 0;
    const bool in = key != 0 && (key >> shift) >= thr;
    const uint64_t mask = __ballot(in);
    if (in) out[taken + __popcll(mask & ((uint64_t(1) << lane) - 1))] = key;
    taken += __popcll(mask);
  }
  for (int t = taken + lane; t < r; t += 64) out[t] = 0;
}

// 256 threads: positions of the best r of the keys [0, n) to out_pos[0 .. r), best first.  list: 4 r keys, 16-byte aligned.  hist: 4 x 256
// words, 16-byte aligned.  Needs at least r keys and r <= kFewRanks; the keys are complete (barrier).
__device__ __forceinline__ void best_of_few(const uint64_t *s_key, int n, int r, uint32_t *hist, uint64_t *list, int32_t *out_pos) {
  const int tid = threadIdx.x, wave = tid >> 6, per = (n + 3) / 4;
  wave_best(s_key, wave * per, min(n, (wave + 1) * per), r, hist + wave * 256, list + wave * r);
  __syncthreads();
  if (tid < 4 * r) {
    const uint64_t mine = list[tid];
    int rank = 0;
    const ulonglong2 *two = reinterpret_cast<const ulonglong2 *>(list);
#pragma unroll 8
    for (int j = 0; j < 2 * r; ++j) {
      const ulonglong2 v = two[j];
      rank += (v.x > mine) + (v.y > mine);
    }
    if (mine != 0 && rank < r) out_pos[rank] = key_pos(mine);
  }
  __syncthreads();
}

// ---- release -------------------------------------------------------------------
// One wave per (b,h) row, no barriers; s_ins is the slot the attention of this step filled with token n;
// sc: the scores of the row's sequence by position (global memory or a copy in LDS);
// row_copy, if not null, receives the row as it stands after the release (K ints, e.g. in LDS);
// raw, if not null, holds what release_fetch read of the row earlier (so that the read is under way
// while something else is waited for).
// Lane L holds the keys of slots L, L+64, ...
// (KPL per lane).  The x lowest keys (x < 0: as many as leave m_keep rows) are found by a radix select, 8 bits a
// pass, with a histogram of the wave's own in LDS (hist: 256 words); digits on which all candidates agree are
// skipped.  Keys are distinct, so exactly x are taken.  (A bit-by-bit search with ballots, up to 64 passes of
// KPL ballots each, took 9 us of a 21 us chain next to the attention.)
// This lane's share of row `row` as it stands in memory: raw[j] = slot j*64 + lane (anything beyond K).
template <int KPL>
__device__ __forceinline__ void release_fetch(int row, const int32_t *__restrict__ slot_src, int K, int (&raw)[KPL]) {
  const int lane = threadIdx.x & 63;
  const int32_t *sp = slot_src + size_t(row) * K;
#pragma unroll
  for (int j = 0; j < KPL; ++j) {
    const int k = j * 64 + lane;
    raw[j] = k < K ? sp[k] : -1;
  }
}

template <int KPL>
__device__ __forceinline__ void release_row(int row, int s_ins, const int32_t *__restrict__ slot_src,
                                   int32_t *__restrict__ slot_dst, const float *sc,
                                   int32_t *__restrict__ free_list, int32_t *__restrict__ released_pos,
                                   int32_t *__restrict__ map_out, int32_t *__restrict__ rel_out, int K,
                                   int n, int x, int R1, int32_t *row_copy, uint32_t *hist, const int *raw = nullptr,
                                   int m_keep = 0, const float *held = nullptr) {
  const int lane = threadIdx.x & 63;
  const int32_t *sp = slot_src + size_t(row) * K;

  int pos[KPL];
  uint32_t khi[KPL], klo[KPL];
  uint32_t cand = 0;                            // bit j: slot j*64+lane holds a releasable token
  uint32_t or_hi = 0, or_lo = 0, and_hi = ~0u, and_lo = ~0u;
#pragma unroll
  for (int j = 0; j < KPL; ++j) {
    const int k = j * 64 + lane;
    pos[j] = k < K ? (k == s_ins ? n : (raw ? raw[j] : sp[k])) : -1;
  }
#pragma unroll
  for (int j = 0; j < KPL; ++j) {
    khi[j] = klo[j] = 0;
    if (pos[j] >= 0 && pos[j] != n) {
      const uint64_t key = rank_key(held ? held[j] : sc[pos[j]], pos[j]);
      khi[j] = uint32_t(key >> 32);
      klo[j] = uint32_t(key);
      cand |= 1u << j;
      or_hi |= khi[j]; or_lo |= klo[j];
      and_hi &= khi[j]; and_lo &= klo[j];
    }
  }
  or_hi = wave_or(or_hi);
  or_lo = wave_or(or_lo);
  and_hi = wave_and(and_hi);
  and_lo = wave_and(and_lo);
  const uint32_t diff_hi = or_hi & ~and_hi, diff_lo = or_lo & ~and_lo;   // bits that tell candidates apart

  uint32_t active = cand, sel = 0;
  int need = x;
  int nactive = 0;                              // candidates still in play, whole row
#pragma unroll
  for (int j = 0; j < KPL; ++j) nactive += __popcll(__ballot((cand >> j) & 1u));
  // x < 0: the row counts for itself how many rows it has to give up to be left with m_keep (the current token
  // included): heads that hold different numbers of rows (H2O mode) cannot be told from the host
  if (x < 0) need = max(0, nactive + 1 - m_keep);
  if (need > 0 && nactive > need) {
    // The `need` lowest keys are the `need` largest of the inverted keys: radix select on those, 8 bits a pass from
    // the top, the wave's own 256-bin histogram in LDS.  Every digit starts at a bit in which candidates differ (bytes from
    // the top would put the candidates, which share most of their exponent, into a bin or two first); the search ends
    // as soon as the bin the rank falls into is taken whole (keys are distinct, so after the last digit at the latest).
    bool done = false;
#pragma unroll 1
    for (int word = 1; word >= 0 && !done; --word) {
      uint32_t diff = word ? diff_hi : diff_lo;
#pragma unroll 1
      while (diff != 0u && !done) {
        const int shift = max(24 - __clz(int(diff)), 0);   // a digit from the highest bit that tells two candidates apart
        diff &= (1u << shift) - 1u;
        *reinterpret_cast<uint4 *>(hist + 4 * lane) = uint4{0u, 0u, 0u, 0u};
        wave_lds_fence();
#pragma unroll
        for (int j = 0; j < KPL; ++j) {
          const uint32_t kw = ~(word ? khi[j] : klo[j]);
          if ((active >> j) & 1u) atomicAdd(&hist[(kw >> shift) & 0xffu], 1u);
        }
        wave_lds_fence();
        int bin, rest, inbin;
        pick_bin(hist, lane, need, bin, rest, inbin);
        wave_lds_fence();                       // the reads above come before the next pass clears the bins
#pragma unroll
        for (int j = 0; j < KPL; ++j) {
          if (!((active >> j) & 1u)) continue;
          const int dgt = int(((~(word ? khi[j] : klo[j])) >> shift) & 0xffu);
          if (dgt > bin) sel |= 1u << j;        // above the bin: among the `need` largest for certain
          if (dgt != bin) active &= ~(1u << j);
        }
        need = rest;
        nactive = inbin;
        done = nactive == need;
      }
    }
  }
  if (need > 0) sel |= active;                  // what is left is exactly `need` keys

  // ascending slot order = j major, lane minor
  int nfree = 0, nrel = 0;
  int32_t *dp = slot_dst + size_t(row) * K;
#pragma unroll
  for (int j = 0; j < KPL; ++j) {
    const int k = j * 64 + lane;
    const bool rel = (sel >> j) & 1u;
    const bool free_after = k < K && (pos[j] < 0 || rel);
    const uint64_t bf = __ballot(free_after), br = __ballot(rel);
    const uint64_t below = (uint64_t(1) << lane) - 1;
    if (free_after) {
      const int idx = nfree + __popcll(bf & below);
      if (idx < R1) free_list[size_t(row) * R1 + idx] = k;
    }
    if (rel) {
      const size_t at = size_t(row) * R1 + nrel + __popcll(br & below);
      released_pos[at] = pos[j];
      if (rel_out) rel_out[at] = pos[j];
    }
    if (k < K) {
      if (row_copy) row_copy[k] = rel ? -1 : pos[j];
      dp[k] = rel ? -1 : pos[j];
      if (map_out) map_out[size_t(row) * K + k] = rel ? -1 : pos[j];   // the caller's copy; rebuilt slots follow
    }
    nfree += __popcll(bf);
    nrel += __popcll(br);
  }
  for (int t = nrel + lane; t < R1; t += 64) {
    released_pos[size_t(row) * R1 + t] = -1;
    if (rel_out) rel_out[size_t(row) * R1 + t] = -1;
  }
}

// The same by a workgroup of 256 threads, for rows that are few: thread t holds the keys of slots t, t + 256, ... (KPL of them).  A wave
// alone works 16 keys a lane through every pass and through the compaction, 15 us of a chain of 17 at K = 1024; this takes 5.
// red: kWideWords words of LDS, 16-byte aligned.  x >= 0.  All threads; row_copy is complete behind a barrier.
constexpr int kWideWords = 2 * 256 + 4 * 5 + 4 * 4 * 2;
template <int KPL>
__device__ __forceinline__ void release_fetch_wide(int row, const int32_t *__restrict__ slot_src, int K, int (&raw)[KPL]) {
  const int32_t *sp = slot_src + size_t(row) * K;
#pragma unroll
  for (int j = 0; j < KPL; ++j) {
    const int k = j * 256 + int(threadIdx.x);
    raw[j] = k < K ? sp[k] : -1;
  }
}
template <int KPL>
__device__ __forceinline__ void release_row_wide(int row, int s_ins, int32_t *__restrict__ slot_dst, const float *sc,
                                                 int32_t *__restrict__ free_list, int32_t *__restrict__ released_pos,
                                                 int32_t *__restrict__ map_out, int32_t *__restrict__ rel_out, int K, int n, int x, int R1,
                                                 int32_t *row_copy, uint32_t *red, const int (&raw)[KPL]) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t *hist = red, *s_bits = red + 512, *s_count = s_bits + 20;   // [2][256]; [4 waves][5]; [KPL][4 waves][2]
  int pos[KPL];
  uint32_t khi[KPL], klo[KPL], cand = 0;
  uint32_t or_hi = 0, or_lo = 0, and_hi = ~0u, and_lo = ~0u;
#pragma unroll
  for (int j = 0; j < KPL; ++j) {
    const int k = j * 256 + tid;
    pos[j] = k < K ? (k == s_ins ? n : raw[j]) : -1;
    khi[j] = klo[j] = 0;
  }
  int nactive = 0;
#pragma unroll
  for (int j = 0; j < KPL; ++j) {
    const bool in = pos[j] >= 0 && pos[j] != n;
    if (in) {
      const uint64_t key = rank_key(sc[pos[j]], pos[j]);
      khi[j] = uint32_t(key >> 32);
      klo[j] = uint32_t(key);
      cand |= 1u << j;
      or_hi |= khi[j]; or_lo |= klo[j];
      and_hi &= khi[j]; and_lo &= klo[j];
    }
    nactive += __popcll(__ballot(in));
  }
  or_hi = wave_or(or_hi);
  or_lo = wave_or(or_lo);
  and_hi = wave_and(and_hi);
  and_lo = wave_and(and_lo);
  if (lane == 0) {
    s_bits[wave * 5] = or_hi; s_bits[wave * 5 + 1] = or_lo;
    s_bits[wave * 5 + 2] = and_hi; s_bits[wave * 5 + 3] = and_lo;
    s_bits[wave * 5 + 4] = uint32_t(nactive);
  }
  hist[tid] = 0u;
  __syncthreads();
  or_hi = or_lo = 0u;
  and_hi = and_lo = ~0u;
  nactive = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    or_hi |= s_bits[w * 5]; or_lo |= s_bits[w * 5 + 1];
    and_hi &= s_bits[w * 5 + 2]; and_lo &= s_bits[w * 5 + 3];
    nactive += int(s_bits[w * 5 + 4]);
  }
  const uint32_t diff_hi = or_hi & ~and_hi, diff_lo = or_lo & ~and_lo;
  uint32_t active = cand, sel = 0;
  int need = x, cur = 0;
  if (need > 0 && nactive > need) {              // as in release_row; everything but the lanes' own keys is the same in all threads
    bool done = false;
#pragma unroll 1
    for (int word = 1; word >= 0 && !done; --word) {
      uint32_t diff = word ? diff_hi : diff_lo;
#pragma unroll 1
      while (diff != 0u && !done) {
        const int shift = max(24 - __clz(int(diff)), 0);
        diff &= (1u << shift) - 1u;
        uint32_t *bins = hist + cur * 256;
#pragma unroll
        for (int j = 0; j < KPL; ++j) {
          const uint32_t kw = ~(word ? khi[j] : klo[j]);
          if ((active >> j) & 1u) atomicAdd(&bins[(kw >> shift) & 0xffu], 1u);
        }
        cur ^= 1;
        hist[cur * 256 + tid] = 0u;              // the other one's, last read before the barrier of the pass before
        __syncthreads();
        int bin, rest, inbin;
        pick_bin(bins, lane, need, bin, rest, inbin);
#pragma unroll
        for (int j = 0; j < KPL; ++j) {
          if (!((active >> j) & 1u)) continue;
          const int dgt = int(((~(word ? khi[j] : klo[j])) >> shift) & 0xffu);
          if (dgt > bin) sel |= 1u << j;
          if (dgt != bin) active &= ~(1u << j);
        }
        need = rest;
        done = inbin == rest;
        __syncthreads();
      }
    }
  }
  if (need > 0) sel |= active;

  // ascending slot order: j, then the wave, then the lane
  uint64_t bf[KPL], br[KPL];
#pragma unroll
  for (int j = 0; j < KPL; ++j) {
    const bool rel = (sel >> j) & 1u;
    bf[j] = __ballot(j * 256 + tid < K && (pos[j] < 0 || rel));
    br[j] = __ballot(rel);
    if (lane == 0) {
      s_count[(j * 4 + wave) * 2] = uint32_t(__popcll(bf[j]));
      s_count[(j * 4 + wave) * 2 + 1] = uint32_t(__popcll(br[j]));
    }
  }
  __syncthreads();
  int nfree = 0, nrel = 0;
  int32_t *dp = slot_dst + size_t(row) * K;
  const uint64_t below = (uint64_t(1) << lane) - 1;
#pragma unroll
  for (int j = 0; j < KPL; ++j) {
    int free_at = nfree, rel_at = nrel;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int f = int(s_count[(j * 4 + w) * 2]), r = int(s_count[(j * 4 + w) * 2 + 1]);
      if (w < wave) {
        free_at += f;
        rel_at += r;
      }
      nfree += f;
      nrel += r;
    }
    const int k = j * 256 + tid;
    const bool rel = (sel >> j) & 1u;
    if ((bf[j] >> lane) & 1u) {
      const int idx = free_at + __popcll(bf[j] & below);
      if (idx < R1) free_list[size_t(row) * R1 + idx] = k;
    }
    if (rel) {
      const size_t at = size_t(row) * R1 + rel_at + __popcll(br[j] & below);
      released_pos[at] = pos[j];
      if (rel_out) rel_out[at] = pos[j];
    }
    if (k < K) {
      if (row_copy) row_copy[k] = rel ? -1 : pos[j];
      dp[k] = rel ? -1 : pos[j];
      if (map_out) map_out[size_t(row) * K + k] = rel ? -1 : pos[j];
    }
  }
  for (int t = nrel + tid; t < R1; t += 256) {
    released_pos[size_t(row) * R1 + t] = -1;
    if (rel_out) rel_out[size_t(row) * R1 + t] = -1;
  }
}

// ---- per-sequence choice of the tokens to rebuild -------------------------------
struct RebuildSelectArgs {
  int32_t *slot_pos;           // [B][H][K]
  const float *score;          // [B][N_max]
  const int32_t *free_list;    // [B][H][R1]
  int32_t *rebuilt_pos;        // [B][Rdim]
  int32_t *insert_slot;        // [B][H]
  int32_t *map_out;            // [B][H][K] caller's slot map (already holds the map after the release), or null
  int32_t *rb_out;             // [B][Rdim] caller's copy of rebuilt_pos, or null
  int K, H, N_max, n, r, R1, Rdim, words;
};

// The keys of tokens 0 .. n are kept in LDS for the passes of the per-sequence choice as long as they fit into
// 56 KB next to the residency bitmap; longer sequences recompute them from the scores in every pass.
__host__ __device__ inline bool choice_keys_cached(int n, int words) {
  return size_t(n + 1) * 8 + size_t(words) * 4 <= 56 * 1024;
}
// Beyond that a copy of the scores themselves (4 bytes a token, the key is made from it on the fly) still fits the
// LDS a workgroup may ask for (the stand-alone choice does; the limit leaves room for its other arrays): one read
// of the scores instead of one per pass up to about 33000 tokens.
constexpr size_t kChoiceLdsLimit = 152 * 1024;
__host__ __device__ inline bool choice_scores_cached(int n, int words) {
  return !choice_keys_cached(n, words) && size_t(n + 1) * 4 + size_t(words) * 4 + 16384 <= kChoiceLdsLimit;
}

// The choice for sequence b by one workgroup of any size.  res_row: the positions held by head 0 of the sequence
// after the release (uniform policy: every head of a sequence holds the same positions).  assign_heads: also
// enter the chosen positions into the slot maps of all heads and reserve the next free slot (otherwise whoever
// writes the rebuilt rows does that).  smem64: dynamic LDS of rebuild_choice_lds_bytes().
__device__ __forceinline__ void rebuild_choice_block(const RebuildSelectArgs &a, int b, const int32_t *res_row,
                                            bool assign_heads, uint64_t *smem64) {
  const bool cached = choice_keys_cached(a.n, a.words);
  const bool sc_cached = choice_scores_cached(a.n, a.words);
  uint64_t *s_cache = smem64;                                   // [n + 1] keys, 0 = resident (if cached)
  float *s_score = reinterpret_cast<float *>(smem64);           // or [n + 1] scores (if sc_cached), padded to 8 bytes
  uint64_t *s_keys = smem64 + (cached ? a.n + 1 : sc_cached ? (a.n + 2) / 2 : 0);   // [max(r,1)]
  uint64_t *s_ctl = s_keys + max(a.r, 1);                       // [4]
  uint32_t *s_hist = reinterpret_cast<uint32_t *>(s_ctl + 4);   // [256]
  uint32_t *s_bits = s_hist + 256;                              // [words] residency bitmap
  int *s_sel = reinterpret_cast<int *>(s_bits + a.words);       // [max(r,1)] chosen positions, best first
  int *s_count = s_sel + max(a.r, 1);
  const int tid = threadIdx.x;
  const int r = a.r;

  if (r > 0) {
    for (int wd = tid; wd < a.words; wd += blockDim.x) s_bits[wd] = 0;
    __syncthreads();
    for (int k = tid; k < a.K; k += blockDim.x) {
      const int p = res_row[k];
      if (p >= 0) atomicOr(&s_bits[p >> 5], 1u << (p & 31));
    }
    __syncthreads();
    const float *sc = a.score + size_t(b) * a.N_max;
    auto key_of = [&](int i) -> uint64_t {
      return (s_bits[i >> 5] >> (i & 31)) & 1u ? uint64_t(0) : rank_key(sc[i], i);
    };
    uint64_t thr;
    int shift;
    if (cached) {   // one read of the scores instead of one per pass
      for (int i = tid; i <= a.n; i += blockDim.x) s_cache[i] = key_of(i);
      __syncthreads();
      auto key_c = [&](int i) -> uint64_t { return s_cache[i]; };
      radix_select(key_c, a.n + 1, r, s_hist, s_ctl, &thr, &shift);
      collect_sorted(key_c, a.n + 1, r, thr, shift, s_keys, s_count, s_sel);
    } else if (sc_cached) {   // the scores once, the keys from the copy in every pass
      for (int i = tid; i <= a.n; i += blockDim.x) s_score[i] = sc[i];
      __syncthreads();
      auto key_s = [&](int i) -> uint64_t {
        return (s_bits[i >> 5] >> (i & 31)) & 1u ? uint64_t(0) : rank_key(s_score[i], i);
      };
      radix_select(key_s, a.n + 1, r, s_hist, s_ctl, &thr, &shift);
      collect_sorted(key_s, a.n + 1, r, thr, shift, s_keys, s_count, s_sel);
    } else {
      radix_select(key_of, a.n + 1, r, s_hist, s_ctl, &thr, &shift);
      collect_sorted(key_of, a.n + 1, r, thr, shift, s_keys, s_count, s_sel);
    }
    for (int t = tid; t < r; t += blockDim.x) {
      a.rebuilt_pos[size_t(b) * a.Rdim + t] = s_sel[t];
      if (a.rb_out) a.rb_out[size_t(b) * a.Rdim + t] = s_sel[t];
    }
    if (assign_heads) {
      // rebuilt rank rho takes the rho-th lowest free slot of every head
      for (int idx = tid; idx < a.H * r; idx += blockDim.x) {
        const int h = idx / r, rho = idx - h * r;
        const int slot = a.free_list[(size_t(b) * a.H + h) * a.R1 + rho];
        a.slot_pos[(size_t(b) * a.H + h) * a.K + slot] = s_sel[rho];
        if (a.map_out) a.map_out[(size_t(b) * a.H + h) * a.K + slot] = s_sel[rho];
      }
    }
  }
  for (int t = r + tid; t < a.Rdim; t += blockDim.x) {
    a.rebuilt_pos[size_t(b) * a.Rdim + t] = -1;
    if (a.rb_out) a.rb_out[size_t(b) * a.Rdim + t] = -1;
  }
  if (assign_heads) {
    // the next free slot is reserved for the next token
    for (int h = tid; h < a.H; h += blockDim.x) {
      a.insert_slot[size_t(b) * a.H + h] = a.free_list[(size_t(b) * a.H + h) * a.R1 + r];
    }
  }
}

// The same choice in two parts, for a workgroup that finds out which positions head 0 keeps while it is
// already at work: choice_fill_keys needs only the scores (any subset of the workgroup's threads may run it, with
// their own tid / nthreads), choice_from_keys then drops the residents (res_row) and picks.  Requires
// choice_keys_cached(n, 0); LDS of ridden_choice_lds_bytes() at smem64.
__device__ __forceinline__ void choice_fill_keys(const float *sc, int n, uint64_t *s_cache, int tid, int nthreads) {
  for (int i = tid; i <= n; i += nthreads) s_cache[i] = rank_key(sc[i], i);
}

// hist: 4 x 256 words, 16-byte aligned; list: room for n_list keys, 16-byte aligned, or null (then, and where the workgroup has not 256
// threads, the keys are ranked by all of them together)
__device__ __forceinline__ void choice_from_keys(const RebuildSelectArgs &a, int b, const int32_t *res_row, uint64_t *smem64, uint32_t *hist,
                                                 uint64_t *list, int n_list) {
  uint64_t *s_cache = smem64;                                   // [n + 1]
  uint64_t *s_keys = smem64 + a.n + 1;                          // [max(r,1)]
  uint64_t *s_ctl = s_keys + max(a.r, 1);                       // [4]
  uint32_t *s_hist = reinterpret_cast<uint32_t *>(s_ctl + 4);   // [256]
  int *s_sel = reinterpret_cast<int *>(s_hist + 256);           // [max(r,1)]
  int *s_count = s_sel + max(a.r, 1);
  const int tid = threadIdx.x;
  const int r = a.r;
  if (r > 0) {
    for (int k = tid; k < a.K; k += blockDim.x) {
      const int p = res_row[k];
      if (p >= 0) s_cache[p] = 0;                               // a resident is no candidate
    }
    __syncthreads();
    if (blockDim.x == 256 && r <= kFewRanks && 4 * r <= n_list) {   // uniform over the launch
      best_of_few(s_cache, a.n + 1, r, hist, list, s_sel);
    } else {
      auto key_c = [&](int i) -> uint64_t { return s_cache[i]; };
      uint64_t thr;
      int shift;
      radix_select(key_c, a.n + 1, r, s_hist, s_ctl, &thr, &shift);
      collect_sorted(key_c, a.n + 1, r, thr, shift, s_keys, s_count, s_sel);
    }
    for (int t = tid; t < r; t += blockDim.x) {
      a.rebuilt_pos[size_t(b) * a.Rdim + t] = s_sel[t];
      if (a.rb_out) a.rb_out[size_t(b) * a.Rdim + t] = s_sel[t];
    }
  }
  for (int t = r + tid; t < a.Rdim; t += blockDim.x) {
    a.rebuilt_pos[size_t(b) * a.Rdim + t] = -1;
    if (a.rb_out) a.rb_out[size_t(b) * a.Rdim + t] = -1;
  }
}

// The choice in parts, for sequences too long for one workgroup.  After the release the candidates are the tokens that held no row before
// it and the released ones, so nothing of it but the last step has to wait for the release: workgroups of 256 threads take kPartTokens
// tokens each and leave the best r of those without a row, the workgroup that releases head 0 leaves what it released, and the one
// of them that comes last picks the best r of all.  None waits for another: the last is told by a counter, which it clears for the
// next launch.  Keys and counter pass between the workgroups (and XCDs) as agent-scope atomics.
constexpr int kPartTokens = 1024, kMostParts = 64, kMostPartKeys = 4096;
struct ChoiceParts {
  uint64_t *keys;              // [B][n_parts * max(R, 1) + R1], 0 = none
  int32_t *arrived;            // [B], 0 between launches
  int n_parts;                 // 0: the choice is not made in parts
};
__host__ __device__ inline int choice_part_keys(int n_parts, int Rdim) { return n_parts * Rdim + Rdim + 1; }
inline size_t choice_parts_lds_bytes(int n_parts, int Rdim) {
  const int total = choice_part_keys(n_parts, Rdim), most = total > kPartTokens ? total : kPartTokens;
  return size_t(most) * 8 + size_t(Rdim) * 8 + 4 * 8 + 256 * 4 + kPartTokens / 32 * 4 + size_t(Rdim) * 4 + 16;
}

__device__ __forceinline__ void put_part_key(uint64_t *p, uint64_t key) {
  __hip_atomic_store(p, key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One part: tokens part * kPartTokens .. below a.n.  row: head 0's positions before the release (the current token is not among them).
__device__ __forceinline__ void choice_part(const RebuildSelectArgs &a, const ChoiceParts &c, int b, int part, const int32_t *row, uint64_t *smem64) {
  uint64_t *s_key = smem64;                                     // [kPartTokens]
  uint64_t *s_ctl = s_key + kPartTokens;                        // [4]
  uint32_t *s_hist = reinterpret_cast<uint32_t *>(s_ctl + 4);   // [256]
  uint32_t *s_bits = s_hist + 256;                              // [kPartTokens / 32] tokens that hold a row
  int *s_count = reinterpret_cast<int *>(s_bits + kPartTokens / 32);   // [2] candidates, keys left behind
  constexpr int TPT = kPartTokens / 256, SPT = kMaxSlots / 256;
  const int tid = threadIdx.x, t0 = part * kPartTokens, count = min(kPartTokens, a.n - t0);
  const float *sc = a.score + size_t(b) * a.N_max + t0;
  float v[TPT];
  int pos[SPT];
#pragma unroll
  for (int u = 0; u < TPT; ++u) v[u] = sc[min(tid + 256 * u, count - 1)];
#pragma unroll
  for (int u = 0; u < SPT; ++u) pos[u] = tid + 256 * u < a.K ? row[tid + 256 * u] : -1;
  if (tid < kPartTokens / 32) s_bits[tid] = 0;
  if (tid < 2) s_count[tid] = 0;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < SPT; ++u) {
    const int p = pos[u] - t0;
    if (pos[u] >= 0 && p >= 0 && p < count) atomicOr(&s_bits[p >> 5], 1u << (p & 31));
  }
  __syncthreads();
  int mine = 0;
#pragma unroll
  for (int u = 0; u < TPT; ++u) {
    const int i = tid + 256 * u;
    const bool free = i < count && !((s_bits[i >> 5] >> (i & 31)) & 1u);
    s_key[i] = free ? rank_key(v[u], t0 + i) : uint64_t(0);
    mine += free;
  }
  if (mine) atomicAdd(&s_count[0], mine);
  __syncthreads();
  auto key_of = [&](int i) -> uint64_t { return s_key[i]; };
  uint64_t thr = 0;
  int shift = 0;
  if (s_count[0] > a.r) radix_select(key_of, count, a.r, s_hist, s_ctl, &thr, &shift);   // uniform over the workgroup
  uint64_t *out = c.keys + size_t(b) * choice_part_keys(c.n_parts, a.Rdim) + size_t(part) * a.Rdim;
#pragma unroll
  for (int u = 0; u < TPT; ++u) {
    const uint64_t key = s_key[tid + 256 * u];
    if (key != 0 && (key >> shift) >= thr) {
      const int idx = atomicAdd(&s_count[1], 1);
      if (idx < a.Rdim) put_part_key(out + idx, key);
    }
  }
  __syncthreads();
  for (int i = s_count[1] + tid; i < a.Rdim; i += 256) put_part_key(out + i, 0);
}

// The keys of the n_rel released tokens of head 0 (LDS or global memory written by this workgroup behind a barrier).
__device__ __forceinline__ void choice_released(const RebuildSelectArgs &a, const ChoiceParts &c, int b, const int32_t *released) {
  uint64_t *out = c.keys + size_t(b) * choice_part_keys(c.n_parts, a.Rdim) + size_t(c.n_parts) * a.Rdim;
  const float *sc = a.score + size_t(b) * a.N_max;
  for (int i = threadIdx.x; i < a.Rdim + 1; i += blockDim.x) {
    const int p = i < a.R1 ? released[i] : -1;
    put_part_key(out + i, p >= 0 ? rank_key(sc[p], p) : uint64_t(0));
  }
}

// Behind either of the two: the last workgroup of the sequence to get here chooses.
// hist: 4 x 256 words, 16-byte aligned.
__device__ __forceinline__ void choice_arrive(const RebuildSelectArgs &a, const ChoiceParts &c, int b, uint64_t *smem64, uint32_t *hist) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");              // this wave's keys are where the others will look for them
  __syncthreads();
  const int total = choice_part_keys(c.n_parts, a.Rdim);
  uint64_t *s_key = smem64;                                     // [total]
  uint64_t *s_keys = s_key + total;                             // [Rdim]
  uint64_t *s_ctl = s_keys + a.Rdim;                            // [4]
  uint32_t *s_hist = reinterpret_cast<uint32_t *>(s_ctl + 4);   // [256]
  int *s_sel = reinterpret_cast<int *>(s_hist + 256);           // [Rdim]
  int *s_count = s_sel + a.Rdim;                                // [2]
  const int tid = threadIdx.x;
  if (tid == 0) {
    const int before = __hip_atomic_fetch_add(c.arrived + b, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_count[1] = before == c.n_parts;                           // n_parts parts and the release
    if (before == c.n_parts) __hip_atomic_store(c.arrived + b, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (s_count[1] == 0) return;                                  // uniform over the workgroup
  const uint64_t *in = c.keys + size_t(b) * total;
  for (int i = tid; i < total; i += blockDim.x) s_key[i] = __hip_atomic_load(in + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  const int list = (total + 1) / 2 * 2;                         // (behind the keys, within what a part takes: choice_parts_lds_bytes)
  int *sel = s_sel;
  if (a.r <= kFewRanks && list + 4 * a.r + kFewRanks / 2 <= kPartTokens) {
    sel = reinterpret_cast<int *>(s_key + list + 4 * a.r);      // (s_sel lies where the list does)
    best_of_few(s_key, total, a.r, hist, s_key + list, sel);
  } else {
    auto key_of = [&](int i) -> uint64_t { return s_key[i]; };
    uint64_t thr;
    int shift;
    radix_select(key_of, total, a.r, s_hist, s_ctl, &thr, &shift);
    collect_sorted(key_of, total, a.r, thr, shift, s_keys, s_count, s_sel);
  }
  for (int t = tid; t < a.Rdim; t += blockDim.x) {
    const int p = t < a.r ? sel[t] : -1;
    a.rebuilt_pos[size_t(b) * a.Rdim + t] = p;
    if (a.rb_out) a.rb_out[size_t(b) * a.Rdim + t] = p;
  }
}

inline size_t ridden_choice_lds_bytes(int r, int n) {
  const size_t rr = size_t(r > 0 ? r : 1);
  return size_t(n + 1) * 8 + rr * 8 + 4 * 8 + 256 * 4 + rr * 4 + 8;
}

// n: position of the current token (keys of tokens 0 .. n)
inline size_t rebuild_choice_lds_bytes(int r, int words, int n) {
  const size_t rr = size_t(r > 0 ? r : 1);
  const size_t cache = choice_keys_cached(n, words) ? size_t(n + 1) * 8
                       : choice_scores_cached(n, words) ? size_t((n + 2) / 2) * 8 : 0;
  return cache + rr * 8 + 4 * 8 + 256 * 4 + size_t(words) * 4 + rr * 4 + 8;
}

}  // namespace adore
