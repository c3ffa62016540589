// tc_select.hpp -- exact TopK threshold selection on register-resident keys.
//
// TopK (Sec. 2.3 of the paper) keeps the k entries of largest magnitude.  On
// the device the magnitude is the 31-bit key of mag_key(); the k-th largest
// key T and the tie quota r = k - #(key > T) define the kept set:
//   key > T, or key == T and the entry is among the r lowest-index ties.
//
// Shared pieces: bin search over histograms in LDS, and the one-wavefront
// strategy for short segments (a token row).  The several-workgroup strategy is
// in tc_group.hpp.
#pragma once

#include "tc_device.hpp"

namespace tc {

constexpr int HIST_BINS = 4096;   // 12-bit digits for the first two passes
constexpr int LAST_BINS = 128;    // 7-bit digit for the last pass

__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

struct SelResult {
  uint32_t T;          // threshold key (0xFFFFFFFF when k == 0: nothing kept)
  uint32_t r;          // ties at T to keep over the whole segment
  uint32_t gt_before;  // keys > T in lower-indexed workgroups of the segment
  uint32_t eq_before;  // keys == T in lower-indexed workgroups of the segment
};

// Find the bin b of a histogram with  sum_{c > b} h[c] < need <= sum_{c >= b} h[c]
// (1 <= need <= sum h), given each thread's BPT consecutive bins in loc[]
// (thread t owns bins [t*BPT, t*BPT + BPT)).  Writes (b, sum_{c > b} h[c])
// to found[].
template <int NT, int BPT>
__device__ __forceinline__ void find_bin_loc(const uint32_t (&loc)[BPT], uint32_t need, uint32_t* scratch,
                                             uint32_t* found) {
  const int t = (int)threadIdx.x;
  uint32_t sum = 0;
#pragma unroll
  for (int i = 0; i < BPT; ++i) sum += loc[i];
  uint32_t total;
  const uint32_t pre = block_excl_scan<NT>(sum, scratch, total);
  uint32_t acc = total - pre - sum;           // keys in bins owned by higher threads
  if (acc < need && need <= acc + sum) {
#pragma unroll
    for (int i = BPT - 1; i >= 0; --i) {
      if (acc + loc[i] >= need) { found[0] = (uint32_t)(t * BPT + i); found[1] = acc; break; }
      acc += loc[i];
    }
  }
  __syncthreads();
}

// ... with the histogram in LDS
template <int NT, int NB>
__device__ __forceinline__ void find_bin(const uint32_t* h, uint32_t need, uint32_t* scratch, uint32_t* found) {
  constexpr int BPT = (NB + NT - 1) / NT;
  uint32_t loc[BPT];
#pragma unroll
  for (int i = 0; i < BPT; ++i) {
    const int b = (int)threadIdx.x * BPT + i;
    loc[i] = (b < NB) ? h[b] : 0u;
  }
  find_bin_loc<NT, BPT>(loc, need, scratch, found);
}

// ... with a small histogram in LDS, searched by the first wavefront alone
// (every thread calls; all meet at the closing barrier)
template <int NB>
__device__ __forceinline__ void find_bin_wave(const uint32_t* h, uint32_t need, uint32_t* found) {
  static_assert(NB % WAVE == 0, "whole bins per lane");
  constexpr int BPL = NB / WAVE;
  if (threadIdx.x < WAVE) {
    const int l = lane_id();
    uint32_t loc[BPL], sum = 0;
#pragma unroll
    for (int i = 0; i < BPL; ++i) {
      loc[i] = h[l * BPL + i];
      sum += loc[i];
    }
    const uint32_t incl = wave_incl_scan(sum);
    uint32_t acc = (uint32_t)__builtin_amdgcn_readlane((int)incl, WAVE - 1) - incl;   // bins of higher lanes
    if (acc < need && need <= acc + sum) {
#pragma unroll
      for (int i = BPL - 1; i >= 0; --i) {
        if (acc + loc[i] >= need) { found[0] = (uint32_t)(l * BPL + i); found[1] = acc; break; }
        acc += loc[i];
      }
    }
  }
  __syncthreads();
}

template <int NT>
__device__ __forceinline__ void zero_lds(uint32_t* h, int n) {
  for (int b = (int)threadIdx.x; b < n; b += NT) h[b] = 0u;
}

// Exact threshold for a segment held by one wavefront, V keys per lane (keys
// past the segment's L are 0 and come after it): the k-th largest key T, or
// any T' with exactly k keys at or above it.  Four rows share a SIMD, so what
// counts is instructions issued.  A first guess t0 places a window of two
// octaves on either side of it, 512 bins of 1/128 octave (one to four keys of a
// row each around T), counted with LDS atomics (keys below the window in a word
// per lane, so that they do not meet in one).  T's bin then gives up its keys
// from the nearer end, a wavefront reduction each: at once where it holds a
// few, and once in any case, as values that repeat fill a bin with one key.
// What is left, or what lies beyond the window when it missed T, is split into
// 512 bins again (five or six instructions per key for nine bits of T, at most
// six such passes for any input).  4096 x 768 bfloat16 with EF, 10 %: 17
// distinct values 19.7 us, values with a gap at T 15.6 when trial keys stood in
// place of these passes (two instructions per key for about a bit each), 12.2
// and 10.0 now; normal data 9.8 both ways.  Two cases go without the window:
// k up to 2 takes the largest keys (every key in one bin, k = 1: 16.7 us with
// it, 6 to 7 without), and where the lanes' first keys share a bin the keys
// are taken to be nearly alike (all of a bin's lanes add to one word in turn).
// Keys are multiples of 2^tz (tz <= RW_SHIFT), and so are lo and hi: 16-bit
// inputs need no search below their last bit.  1 <= k <= L.
constexpr uint32_t RW_BINS = 512, RW_SHIFT = 16;            // 2^25: four octaves
constexpr uint32_t RW_WIDE = 27;                            // 2^27: 16 octaves
constexpr uint32_t RW_WORDS = RW_BINS + WAVE;               // LDS words (16-byte aligned)

// T's bin, the keys in larger bins and its own keys, of 512 bins in which
// `need` is the rank from the top; false when they do not reach it (above:
// what they hold)
__device__ __forceinline__ bool row_find_bin(const uint32_t* bins, uint32_t need, uint32_t& bin, uint32_t& above,
                                             uint32_t& cnt) {
  const uint32_t lane = (uint32_t)lane_id();
  const u32x4 h0 = reinterpret_cast<const u32x4*>(bins)[2 * lane], h1 = reinterpret_cast<const u32x4*>(bins)[2 * lane + 1];
  const uint32_t h[8] = {h0.x, h0.y, h0.z, h0.w, h1.x, h1.y, h1.z, h1.w};
  const uint32_t sum = ((h[0] + h[1]) + (h[2] + h[3])) + ((h[4] + h[5]) + (h[6] + h[7]));
  const uint32_t incl = wave_incl_scan(sum);
  const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)incl, WAVE - 1);
  uint32_t acc = all - incl;          // keys in bins of higher lanes
  const uint64_t here = __ballot(acc < need && need <= acc + sum);
  above = all;
  if (!here) return false;
  const int src = __builtin_ctzll(here);
  uint32_t ab = acc, bi = 0u, cn = 0u;
#pragma unroll
  for (int c = 7; c >= 0; --c) {
    const bool on = acc < need;       // the last such bin, from the top, is T's
    ab = on ? acc : ab;
    bi = on ? (uint32_t)c : bi;
    cn = on ? h[c] : cn;
    acc += h[c];
  }
  bin = 8u * (uint32_t)src + (uint32_t)__builtin_amdgcn_readlane((int)bi, src);
  above = (uint32_t)__builtin_amdgcn_readlane((int)ab, src);
  cnt = (uint32_t)__builtin_amdgcn_readlane((int)cn, src);
  return true;
}

template <int V>
__device__ __forceinline__ uint32_t wave_select_key(const uint32_t (&key)[V], uint32_t k, uint32_t tz, uint32_t t0,
                                                    uint32_t* hist) {
  const uint32_t lane = (uint32_t)lane_id(), unit = 1u << tz;
  uint32_t* const bins = hist + WAVE;
  const int below = -1 - (int)lane;   // this lane's word for keys that are not counted
  auto clear = [&] {
    reinterpret_cast<u32x4*>(bins)[lane] = u32x4{0u, 0u, 0u, 0u};
    reinterpret_cast<u32x4*>(bins)[lane + WAVE] = u32x4{0u, 0u, 0u, 0u};
    __builtin_amdgcn_wave_barrier();
  };
  // the bracket of T: C(t) = #(key >= t) is ch < k at hi and, once counted,
  // cl >= k at lo; lo is 0 or above it
  uint32_t lo = 0u, hi = 0x80000000u, cl = 0u, ch = 0u;
  uint32_t bin, above, cnt;
  bool split = true;                  // the bracket is to be split before its keys are looked at
  const uint32_t base = (t0 - min(t0, 2u << 23)) & ~((1u << RW_SHIFT) - 1u);
  const int b0 = (int)(key[0] - base) >> RW_SHIFT;
  if (k <= 2u) {
    split = false;                    // the largest keys
  } else if (__ballot(b0 == __builtin_amdgcn_readfirstlane(b0)) == ~0ull) {
    // (nearly) one value throughout: its lanes would all meet in one word;
    // from the smallest key that is not 0 to the largest instead
    uint32_t small = ~0u, large = 0u;
#pragma unroll
    for (int i = 0; i < V; ++i) {
      small = min(small, key[i] - 1u);
      large = max(large, key[i]);
    }
    lo = wave_uminmax<false>(small) + 1u;
    hi = wave_uminmax<true>(large) + unit;
  } else {
    clear();
#pragma unroll
    for (int i = 0; i < V; ++i) {
      const int b = (int)(key[i] - base) >> RW_SHIFT;
      atomicAdd(&bins[min(max(b, below), (int)RW_BINS - 1)], 1u);
    }
    __builtin_amdgcn_wave_barrier();
    if (row_find_bin(bins, k, bin, above, cnt)) {
      // (the last bin has no upper end; one that starts at key 0 counts the
      // keys past the segment's end)
      lo = base + (bin << RW_SHIFT);
      hi = (bin < RW_BINS - 1u) ? lo + (1u << RW_SHIFT) : hi;
      cl = above + cnt;
      split = lo == 0u;
    } else {
      hi = base;
    }
    ch = above;
  }
  bool once = true;
  uint32_t wide = RW_WIDE;
  for (;;) {
    if (!split) {
      if (cl == k || hi - lo <= unit) return lo;
      // (k - ch is 1 at least; a bracket from 0 on gives up keys at its top only)
      const uint32_t up = k - ch, dn = (lo > 0u) ? cl - k : 0xFFFFFFFFu;
      split = min(up, dn) > 3u && !once;
      once = false;
      if (!split) {
        uint32_t T, m = 0;
        const bool top = up <= dn;
        if (top) {
          // the largest key below hi: differences wrap for those below
          uint32_t best = 0u;
#pragma unroll
          for (int i = 0; i < V; ++i) best = max(best, key[i] - hi);
          T = wave_uminmax<true>(best) + hi;
          if (up == 1u) return T;
        } else {
          // the smallest key from lo on: differences wrap for those below
          uint32_t best = 0xFFFFFFFFu;
#pragma unroll
          for (int i = 0; i < V; ++i) best = min(best, key[i] - lo);
          T = wave_uminmax<false>(best) + lo;
        }
#pragma unroll
        for (int i = 0; i < V; ++i) m += (uint32_t)__popcll(__ballot(key[i] == T));
        if (m > dn || (top && m >= up)) return T;
        hi = top ? T : hi;
        ch += top ? m : 0u;
        lo = top ? lo : T + unit;
        cl -= top ? 0u : m;
        continue;
      }
    }
    // ---- the bracket's keys into 512 bins, the zeros (and the keys past the
    // segment's end) into none: 0 is T when the others do not reach its rank.
    // A bracket from 0 on is tried in its 16 octaves at the top first.
    uint32_t from = max(lo, unit);
    const bool part = lo == 0u && hi - from > (1u << wide);
    from = part ? hi - (1u << wide) : from;
    const uint32_t w = hi - from, bits = 32u - (uint32_t)__builtin_clz((w - 1u) | 1u);
    const uint32_t sh = max(tz, bits - min(bits, 9u));
    clear();
#pragma unroll
    for (int i = 0; i < V; ++i) {
      const uint32_t d = key[i] - from;
      atomicAdd(&bins[d < w ? (int)(d >> sh) : below], 1u);
    }
    __builtin_amdgcn_wave_barrier();
    split = !row_find_bin(bins, k - ch, bin, above, cnt);
    if (split) {
      if (!part) return 0u;
      hi = from;
      wide = 31u;
    } else {
      lo = from + (bin << sh);
      hi = min(hi, lo + (1u << sh));
      cl = ch + above + cnt;
    }
    ch += above;
  }
}

}  // namespace tc
