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

// The threshold by counting: C(t) = #(key >= t) over the segment for a few
// trial keys t, which narrow a bracket lo < hi with C(lo) > k > C(hi) (or lo
// = 0, hi = 2^31).  Every lane holds the same values, on the scalar unit but
// for the guess itself.  Trials are guessed from the counts: the first as if
// magnitudes were exponentially distributed around their mean mu, then by
// interpolation of log C between the ends, in value where the bracket spans
// octaves (a heavy tail or a mass at zero bends log C there), in key
// otherwise.  From the eighth trial on each halves the bracket in key, which
// bounds the search at 39 trials for any input.  Keys are multiples of 2^tz,
// and so are lo and hi: 16-bit inputs need no search below their last bit.
// Only which t is tried depends on floating point; the counts decide.
struct CountSearch {
  uint32_t lo = 0u, hi = 0x80000000u;   // trial keys: C(lo) = cl, C(hi) = ch
  uint32_t cl, ch = 0u, n = 0u;
  uint32_t k, tz;
  float mu, lk, la, lb = -1.0f;         // log2 of k, cl, ch (of 1/2 for ch = 0)
  __device__ __forceinline__ CountSearch(uint32_t L, uint32_t k_, uint32_t tz_, float mu_, float lk_, float lL)
      : cl(L), k(k_), tz(tz_), mu(mu_), lk(lk_), la(lL) {}
  __device__ __forceinline__ bool closed() const { return hi - lo <= (1u << tz); }   // T = lo, k - ch ties kept
  // a key strictly inside the bracket, a multiple of 2^tz, near t
  __device__ __forceinline__ uint32_t inside(uint32_t t) const {
    const uint32_t g = 1u << tz;
    t = (uint32_t)__builtin_amdgcn_readfirstlane((int)t);
    t = min(max(t, lo), hi - 1u);
    t = lo + max(g, ((t - lo) >> tz) << tz);
    return min(t, hi - g);
  }
  // lg = 0.95 ln(L / k + 0.15)
  __device__ __forceinline__ uint32_t first(float lg) const { return inside(__float_as_uint(mu * lg)); }
  __device__ __forceinline__ void update(uint32_t t, uint32_t c) {
    const float l = c ? __builtin_amdgcn_logf((float)c) : -1.0f;
    // (selects, one per member: branches would leave the object in memory)
    const bool low = c > k;
    lo = low ? t : lo;
    cl = low ? c : cl;
    la = low ? l : la;
    hi = low ? hi : t;
    ch = low ? ch : c;
    lb = low ? lb : l;
    ++n;
  }
  __device__ __forceinline__ uint32_t next() const {
    constexpr float LN2 = 0.6931472f;
    if (n >= 8u) return inside(lo + ((hi - lo) >> 1));
    if (hi == 0x80000000u)                // no upper end yet: out by the mean, doubling
      return inside(__float_as_uint(__uint_as_float(lo) + mu * LN2 * (la - lk) * (float)(1u << (n - 1u))));
    if (lo == 0u) {                       // no lower end yet: down once, then "not zero"
      if (n >= 2u) return inside(1u);
      const float h = __uint_as_float(hi);
      return inside(__float_as_uint(fmaxf(h - 1.1f * mu * LN2 * (lk - lb), 0.25f * h)));
    }
    const float f = (la - lk) * __builtin_amdgcn_rcpf(la - lb);
    if (hi - lo > (1u << 24) && (n & 1u) == 0u) {
      const float l = __uint_as_float(lo);
      return inside(__float_as_uint(l + (__uint_as_float(hi) - l) * f));
    }
    return inside(lo + (uint32_t)((float)(hi - lo) * f));
  }
};

// Exact threshold for a segment held by one wavefront, V keys per lane (keys
// past the segment's L are 0 and come after it): the k-th largest key T, or
// any T' with exactly k keys at or above it.  Four rows share a SIMD, so what
// counts is instructions issued: a trial key costs two per key for one bit of
// T, a histogram five for nine bits.  So the first guess places a window of
// two octaves on either side of it, 512 bins of 1/128 octave (one to four keys
// of a row each around T), counted with LDS atomics (keys below the window in
// a word per lane, so that they do not meet in one); T's bin then gives up
// its keys from the nearer end, a wavefront reduction each.  A window that
// missed T, or a bin with many keys, leaves the rest to trial keys.
// 1 <= k <= L; tz as above, at most RW_SHIFT.
constexpr uint32_t RW_BINS = 512, RW_SHIFT = 16;            // 2^25: four octaves
constexpr uint32_t RW_WORDS = RW_BINS + WAVE;               // LDS words (16-byte aligned)
struct RowLogs {
  float lk, lL, lg;   // log2 k, log2 L, the first guess's factor
};
template <int V>
__device__ __forceinline__ uint32_t wave_select_key(const uint32_t (&key)[V], uint32_t L, uint32_t k, uint32_t tz,
                                                    float mu, const RowLogs& lg, uint32_t* hist) {
  CountSearch s(L, k, tz, mu, lg.lk, lg.lL);
  const uint32_t t0 = s.first(lg.lg);
  const uint32_t lane = (uint32_t)lane_id();
  {
    const uint32_t base = (t0 - min(t0, 2u << 23)) & ~((1u << RW_SHIFT) - 1u);
    uint32_t* const bins = hist + WAVE;
    reinterpret_cast<u32x4*>(bins)[lane] = u32x4{0u, 0u, 0u, 0u};
    reinterpret_cast<u32x4*>(bins)[lane + WAVE] = u32x4{0u, 0u, 0u, 0u};
    __builtin_amdgcn_wave_barrier();
    const int below = -1 - (int)lane;
#pragma unroll
    for (int i = 0; i < V; ++i) {
      const int b = (int)(key[i] - base) >> RW_SHIFT;
      atomicAdd(&bins[min(max(b, below), (int)RW_BINS - 1)], 1u);
    }
    __builtin_amdgcn_wave_barrier();
    const u32x4 h0 = reinterpret_cast<const u32x4*>(bins)[2 * lane], h1 = reinterpret_cast<const u32x4*>(bins)[2 * lane + 1];
    const uint32_t h[8] = {h0.x, h0.y, h0.z, h0.w, h1.x, h1.y, h1.z, h1.w};
    const uint32_t sum = ((h[0] + h[1]) + (h[2] + h[3])) + ((h[4] + h[5]) + (h[6] + h[7]));
    const uint32_t incl = wave_incl_scan(sum);
    uint32_t acc = (uint32_t)__builtin_amdgcn_readlane((int)incl, WAVE - 1) - incl;   // keys in bins of higher lanes
    const uint64_t here = __ballot(acc < k && k <= acc + sum);
    if (here) {
      const int src = __builtin_ctzll(here);
      uint32_t above = acc, bin = 0u, cnt = 0u;
#pragma unroll
      for (int c = 7; c >= 0; --c) {
        const bool on = acc < k;          // the last such bin, from the top, is T's
        above = on ? acc : above;
        bin = on ? (uint32_t)c : bin;
        cnt = on ? h[c] : cnt;
        acc += h[c];
      }
      bin = 8u * (uint32_t)src + (uint32_t)__builtin_amdgcn_readlane((int)bin, src);
      above = (uint32_t)__builtin_amdgcn_readlane((int)above, src);
      cnt = (uint32_t)__builtin_amdgcn_readlane((int)cnt, src);
      const uint32_t lo = base + (bin << RW_SHIFT);
      // (the last bin has no upper end; one that starts at key 0 counts the
      // keys past the segment's end)
      if (bin < RW_BINS - 1u && lo > 0u) {
        if (above + cnt == k) return lo;
        s.update(lo, above + cnt);
        s.update(lo + (1u << RW_SHIFT), above);
      }
    }
  }
  for (;;) {
    for (;;) {
      if (s.closed()) return s.lo;
      const uint32_t near = (s.n < 5u) ? 3u : 6u;
      const uint32_t up = k - s.ch, dn = (s.lo > 0u) ? s.cl - k : 0xFFFFFFFFu;
      if (min(up, dn) > near) break;
      uint32_t T, m = 0;
      if (up <= dn) {
        // the largest key below hi: differences wrap for those below
        uint32_t best = 0u;
#pragma unroll
        for (int i = 0; i < V; ++i) best = max(best, key[i] - s.hi);
        T = wave_uminmax<true>(best) + s.hi;
        if (up == 1u) return T;
      } else {
        // the smallest key from lo on: differences wrap for those below
        uint32_t best = 0xFFFFFFFFu;
#pragma unroll
        for (int i = 0; i < V; ++i) best = min(best, key[i] - s.lo);
        T = wave_uminmax<false>(best) + s.lo;
      }
#pragma unroll
      for (int i = 0; i < V; ++i) m += (uint32_t)__popcll(__ballot(key[i] == T));
      const bool top = up <= dn;
      if (m > dn || (top && m >= up)) return T;
      if (!top && m == dn) return T + 1u;
      s.hi = top ? T : s.hi;
      s.ch += top ? m : 0u;
      s.lo = top ? s.lo : T + (1u << tz);
      s.cl -= top ? 0u : m;
    }
    // a trial key: a lane counts its own keys and the lanes' counts are added
    // once (the scalar unit would take a population count and an addition per key)
    const uint32_t t = s.n ? s.next() : t0;
    uint32_t under = 0;      // a bit per key below t
#pragma unroll
    for (int i = 0; i < V; ++i) under = __builtin_amdgcn_alignbit(under, key[i] - t, 31);
    const uint32_t c = (uint32_t)WAVE * V - wave_sum((uint32_t)__builtin_popcount(under));
    if (c == k) return t;
    s.update(t, c);
  }
}

}  // namespace tc
