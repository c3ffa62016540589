// tc_group.hpp -- exact TopK threshold for a segment spread over P
// workgroups whose values stay in registers (the group engine).
//
// TopK (Sec. 2.3 of the paper) keeps the k entries of largest magnitude.  The
// magnitude is the 31-bit key of mag_key(); the k-th largest key T and the
// tie quota r = k - #(key > T) define the kept set: key > T, or key == T and
// the entry is among the r lowest-index ties.
//
// Layout: workgroup `part` of a group owns the chunk [part*CH, part*CH + CH)
// of its segment; thread t holds R runs of E consecutive elements, run j at
// offset (j*NT + t)*E of the chunk (striped, so that every load and store
// instruction of a wavefront covers 1 KiB of contiguous memory).
//
// Two cross-workgroup exchanges per segment in the common case:
//   A. every workgroup guesses, from its own histogram of key bits 30..19 (at
//      the rank its share of the segment gives), the bin of the k-th largest
//      key, and adds its counts from an octave below that bin upwards into the
//      group's histogram, its guess into the group's smallest and largest
//      guess, and 32 finer counts (bits 18..14) of the guessed bin and its two
//      neighbours (bins 0 to 2 when it guesses bin 0).  After the barrier, one read of the merged counts gives the
//      bin b1 (exact when no guess lies more than an octave above it: then no
//      count at or above b1 is missing) and, when every guess was within one
//      bin of b1, the 17-bit prefix of T.
//   B. every workgroup publishes a record: its count of keys above that
//      prefix and the distinct keys that share it with their multiplicities
//      (a few; 16-bit inputs repeat values, so one key may stand for many
//      entries).  After the barrier each workgroup reads all records in one
//      round trip and finds T, the tie quota and what precedes it by itself.
// When a guess was further off (values with a gap around T, as AQ-SGD's changes
// have once an example's activations repeat; or chunks that differ), one pass
// over the next 8 bits, merged through device memory, gives a 20-bit prefix
// for exchange B instead.  When too many distinct keys share the prefix, the
// group goes on with a digit pass and one exchange of per-workgroup counts of
// the last digit: exact for any input.
#pragma once

#include "tc_select.hpp"

namespace tc {

constexpr int GRP_NT = 512;
constexpr uint32_t REC_W = 32;            // words per record: header, then distinct keys
constexpr uint32_t REC_KEYS = REC_W - 1;
constexpr uint32_t REC_OVF = 0xFFu;       // header: more distinct keys than a record holds
constexpr uint32_t FINE_BITS = 5;         // finer digit of exchange A (bits 18..14)
constexpr uint32_t FINE_N = 1u << FINE_BITS;
constexpr uint32_t FINE_SLOTS = 128;      // fine counts kept for bins b1 mod 128
constexpr uint32_t LOW_BITS = 19 - FINE_BITS;   // key bits below the fine prefix (at most that many in a record's entry)
static_assert(LOW_BITS == 14 && LAST_BINS == 128, "two 7-bit digits below the fine prefix");
constexpr uint32_t DIG_BINS = 256;        // digits of the fallback passes: up to 8 bits
constexpr uint32_t CNT_BINS = 64, CNT_W = CNT_BINS + 1;   // last digit of the fallback: at most 6 bits
constexpr uint32_t REC_P_MAX = 256;       // workgroups per segment of the record exchange
constexpr uint32_t A_MARGIN = 16;         // bins added below the guessed one's neighbour (an octave)
constexpr uint32_t RLE_SLOTS = 64;        // hash table of a workgroup's distinct keys on the prefix
constexpr uint32_t RLE_PROBES = 8;

// Device memory owned by one group (inside the caller's workspace; zero on
// entry and left zero on exit), as word offsets from the group's base:
//   ctl[64]               [0] barrier arrivals (monotone during a launch), [1] exits,
//                         [32 + par], [34 + par] largest guess + 1, 4096 - smallest guess
//   hist1[2][4096]        first-digit histograms, by segment parity
//   fine[2][128][32]      bits 18..14 of the keys in guessed bins, by bin mod 128
//   hist2[4][256]         digit pass p: hist2(p)
//   rec[P][32]            exchange B records
//   cnt[P][65]            last digit's counts and keys above its prefix per workgroup (fallback)
// The size keeps the words that earlier layouts used per workgroup (64 for
// the record, 257 rows of digit slots): callers size their workspaces, and
// the allocation-free entry point its refusals, by it.
namespace gm_off {
constexpr uint32_t CTL = 0, HIST1 = 64, FINE = HIST1 + 2 * HIST_BINS, HIST2 = FINE + 2 * FINE_SLOTS * FINE_N + 512,
                   REC = HIST2 + 4 * DIG_BINS;
static_assert(REC % 4 == 0, "records are 16-byte aligned");
}  // namespace gm_off

__host__ __device__ constexpr uint64_t grp_mem_words(uint32_t P) {
  return gm_off::REC + (uint64_t)P * 64u + 257ull * ((P + 7u) & ~7u);
}
static_assert(REC_W + CNT_W <= 64u + 257u, "records and counts fit");

// the group's memory: one base pointer, pieces at fixed offsets
struct GrpMem {
  uint32_t* base;
  uint32_t P;
  __device__ __forceinline__ uint32_t* ctl() const { return base + gm_off::CTL; }
  __device__ __forceinline__ uint32_t* hist1(uint32_t par) const { return base + gm_off::HIST1 + par * HIST_BINS; }
  __device__ __forceinline__ uint32_t* fine(uint32_t par) const { return base + gm_off::FINE + par * FINE_SLOTS * FINE_N; }
  __device__ __forceinline__ uint32_t* hist2(uint32_t q) const { return base + gm_off::HIST2 + q * DIG_BINS; }
  __device__ __forceinline__ uint32_t* rec() const { return base + gm_off::REC; }
  __device__ __forceinline__ uint32_t* cnt() const { return base + gm_off::REC + P * REC_W; }
};

__device__ __forceinline__ GrpMem grp_mem(uint32_t* ws, uint32_t group, uint32_t P) {
  GrpMem g;
  g.base = ws + (uint64_t)group * grp_mem_words(P);
  g.P = P;
  return g;
}

// Barrier among the P workgroups of a group: arrivals are counted in one
// word that only grows during a launch, so the n-th barrier waits for n*P
// arrivals and nobody has to reset anything in flight.  Each wave's device-
// scope stores and atomics complete before its workgroup arrives.  Arrival
// and wait are separate calls so that a workgroup can do work of its own in
// between.  The wait is bounded (co-residency violated): it then raises
// KERR_TIMEOUT and returns.
__device__ __forceinline__ void group_arrive(uint32_t* ctr) {
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void group_wait(uint32_t* ctr, uint32_t target) {
  if (threadIdx.x == 0) {
    uint32_t spins = 0;
    while (ld_agent(ctr) < target) {
      __builtin_amdgcn_s_sleep(0);
      ++spins;
      if ((spins & 1023u) == 0u &&
          (__hip_atomic_load(&g_kernel_errors, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & KERR_TIMEOUT))
        break;
      if (spins > BARRIER_SPIN_LIMIT) { raise_error(KERR_TIMEOUT); break; }
    }
  }
  __syncthreads();
}
__device__ __forceinline__ void group_sync(uint32_t* ctr, uint32_t target) {
  group_arrive(ctr);
  group_wait(ctr, target);
}

// Exclusive scans of R values per thread across the workgroup in one pass;
// tot[j] = workgroup total of value j.  scratch: R * NT/64 words.
template <int NT, int R>
__device__ __forceinline__ void block_excl_scan_multi(const uint32_t (&v)[R], uint32_t (&ex)[R],
                                                      uint32_t (&tot)[R], uint32_t* scratch) {
  constexpr int NW = NT / WAVE;
  const int w = (int)threadIdx.x / WAVE;
  uint32_t incl[R];
#pragma unroll
  for (int j = 0; j < R; ++j) incl[j] = wave_incl_scan(v[j]);
  if (lane_id() == WAVE - 1) {
#pragma unroll
    for (int j = 0; j < R; ++j) scratch[j * NW + w] = incl[j];
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < R; ++j) {
    uint32_t pre = 0, t = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const uint32_t x = scratch[j * NW + i];
      pre += (i < w) ? x : 0u;
      t += x;
    }
    ex[j] = pre + incl[j] - v[j];
    tot[j] = t;
  }
  __syncthreads();
}

// The thread's index.  In the loop over segments (LOOP) what follows from it is
// computed where it is used: hoisted out of the loop it took all 256 registers
// and, in the widest layouts, up to 50 more in scratch, where a straight path
// needs about 140.  Two segments per group, AQ-SGD 30 %, 16 x 393,216: binary16
// 49.1 -> 45.8 us, binary32 62.2 -> 54.1.
template <bool LOOP>
__device__ __forceinline__ uint32_t grp_thread() {
  uint32_t t = threadIdx.x;
  if constexpr (LOOP) asm volatile("" : "+v"(t));
  return t;
}

// LDS of the group engine's selection
struct GrpSelShared {
  uint32_t hist[HIST_BINS + WAVE];   // histograms (the last WAVE words: per-lane dummies)
};

struct GrpSmall {
  uint32_t scratch[8 * (GRP_NT / WAVE)];
  uint32_t found[4];
  uint32_t red[DIG_BINS];            // one digit's counts, copies summed
  uint32_t fwin[3 * FINE_N + WAVE];  // this workgroup's fine counts of its window
  uint32_t fmrg[GRP_NT];             // the group's merged fine counts of that window, largest and smallest window
  uint32_t h7a[LAST_BINS + WAVE], h7b[LAST_BINS + WAVE];  // last two 7-bit digits of T (plus per-lane dummies)
  uint32_t hk[RLE_SLOTS], hc[RLE_SLOTS];   // distinct keys on the prefix (low bits + 1) and multiplicities
  uint32_t rec[REC_W];               // this workgroup's record
  uint32_t misc[16];
  // this workgroup's keys on the 17-bit prefix, in index order (exchange B,
  // at most WAVE of them): key, chunk offset, staged payload position
  uint32_t ckey[WAVE], coff[WAVE], cpos[WAVE];
  uint32_t rem[WAVE];                // staged positions dropped after exchange B, less their rank
};

// The known leading bits of T, and the keys still to place below them.  fine:
// exchange A found the 17-bit prefix (every workgroup's window covered the bin
// of the k-th key).
struct SelA {
  uint32_t prefix, pbits, need;
  bool fine;
};

// Per-workgroup state carried across the segments a group handles.
struct GrpState {
  uint32_t nbar = 0;       // barriers passed (equal in all workgroups of the group)
  uint32_t iter = 0;       // segments handled
  bool used_cnt = false;   // the fallback ran (its counts must be cleared on exit)
};

// Histogram copies for digit counts: values that repeat (differences of
// 16-bit numbers often do) would make the lanes of one wave hit one LDS
// address; with a copy per lane group (lane mod CP), spaced by an odd stride
// so that one bin's copies sit in distinct banks, at most 64/CP lanes meet.
// Word HS-1 of each copy absorbs lanes with nothing to count.
constexpr int DIG_CP = 16, DIG_HS = 257;
static_assert(DIG_CP * DIG_HS <= HIST_BINS + WAVE, "histogram copies fit the selection histogram");

template <int NT>
__device__ __forceinline__ void dig_zero(uint32_t* hist) {
  for (int i = (int)threadIdx.x; i < DIG_CP * DIG_HS; i += NT) hist[i] = 0u;
}
__device__ __forceinline__ void dig_add(uint32_t* hist, bool m, uint32_t digit) {
  const uint32_t base = (uint32_t)(lane_id() & (DIG_CP - 1)) * DIG_HS;
  atomicAdd(&hist[base + (m ? digit : (uint32_t)(DIG_HS - 1))], 1u);
}
// copies summed into red[0..NB); call after a barrier that follows the adds
template <int NT, int NB>
__device__ __forceinline__ void dig_reduce(const uint32_t* hist, uint32_t* red) {
  const int t = (int)threadIdx.x;
  if (t < NB) {
    uint32_t s = 0;
#pragma unroll
    for (int c = 0; c < DIG_CP; ++c) s += hist[c * DIG_HS + t];
    red[t] = s;
  }
}

// After the barrier that follows exchange A's every workgroup has read the
// exchange A words of its parity: each clears a slice of them.
__device__ __forceinline__ void grp_clear_a(const GrpMem& g, uint32_t par, uint32_t P, uint32_t part) {
  const uint32_t n1 = HIST_BINS, n2 = FINE_SLOTS * FINE_N;
  uint32_t* h1 = g.hist1(par);
  uint32_t* f1 = g.fine(par);
  for (uint32_t i = part * GRP_NT + threadIdx.x; i < n1 + n2; i += P * GRP_NT) st_agent(i < n1 ? h1 + i : f1 + (i - n1), 0u);
  if (part == 0 && threadIdx.x < 2) st_agent(&g.ctl()[32 + 2 * threadIdx.x + par], 0u);
}

// Exchange A's first histogram (bits 30..19 of every key) and the small
// counters of both exchanges, cleared before the workgroup's values arrive,
// so that the keys of each run can be counted as soon as that run's loads
// land.
template <int NT>
__device__ __forceinline__ void grp_hist_clear(GrpSelShared& sh, GrpSmall& sm) {
  zero_lds<NT>(sh.hist, HIST_BINS);
  const uint32_t t = threadIdx.x;
  static_assert(NT >= 2 * LAST_BINS + 2 * (int)RLE_SLOTS + (int)REC_W && NT >= 3 * (int)FINE_N, "one word per thread");
  if (t < 3 * FINE_N) sm.fwin[t] = 0u;
  if (t < (uint32_t)LAST_BINS) sm.h7a[t] = 0u;
  else if (t < 2u * LAST_BINS) sm.h7b[t - LAST_BINS] = 0u;
  else if (t < 2u * LAST_BINS + RLE_SLOTS) sm.hk[t - 2u * LAST_BINS] = 0u;
  else if (t < 2u * LAST_BINS + 2u * RLE_SLOTS) sm.hc[t - 2u * LAST_BINS - RLE_SLOTS] = 0u;
  else if (t < 2u * LAST_BINS + 2u * RLE_SLOTS + REC_W) sm.rec[t - 2u * LAST_BINS - 2u * RLE_SLOTS] = 0u;
  if (t == 0) sm.misc[4] = 0u;
  __syncthreads();
}
// One key into it; exact zeros (common after a ReLU, and the padding) are
// counted in the thread's zc and added once per wave by exchange A, off one
// hot bin.
__device__ __forceinline__ void grp_hist_add(GrpSelShared& sh, uint32_t kk, uint32_t& zc) {
  const uint32_t z = eq31(kk, 0u);
  zc += z;
  atomicAdd(&sh.hist[pick(z, HIST_BINS + (uint32_t)lane_id(), kk >> 19)], 1u);
}

// The bin of the merged first histogram that holds the k-th largest key:
// found[0] (left alone when the counts do not reach k) and the keys in larger
// bins found[1].  A thread that passes an address `word` loads it in the same
// round trip into *to.
template <int NT>
__device__ __forceinline__ void grp_find_merged(const uint32_t* gh, uint32_t k, const uint32_t* word, uint32_t* to,
                                                uint32_t* scratch, uint32_t* found) {
  constexpr int BPT = HIST_BINS / NT;
  static_assert(BPT >= 2 && BPT % 2 == 0, "two bins per 8-byte load");
  uint32_t loc[BPT];
  const uint64_t* p = reinterpret_cast<const uint64_t*>(gh + threadIdx.x * BPT);
#pragma unroll
  for (int i = 0; i < BPT / 2; ++i) {
    const uint64_t w = ld_agent64(p + i);
    loc[2 * i] = (uint32_t)w;
    loc[2 * i + 1] = (uint32_t)(w >> 32);
  }
  if (word) *to = ld_agent(word);
  find_bin_loc<NT, BPT>(loc, k, scratch, found);
}

// Exchange A for one segment held by the P workgroups of a group (this
// one is `part`, with n_loc >= 1 elements of the segment), k >= 1; every key
// of the workgroup is in the first histogram (grp_hist_clear, then
// grp_hist_add per key; zc: this thread's exact zeros).  v[j][i] is element i
// of this thread's run j.  Elements past the segment's end hold +0: they
// have the smallest key and the highest indices, so with k <= L they rank
// after every real element and are never kept; the counts need no bounds
// checks.  The guess scales k by the elements the chunk really holds: a last
// chunk that is only partly filled guesses as well as the others (scaled by
// the whole chunk it missed, and every segment whose length is not a multiple
// of the chunk took the digit passes: 5 x 100,003 binary16, TopK 30 %, sender
// 25.4 us).
template <int NT, int R, int E, bool LOOP>
__device__ __forceinline__ SelA grp_exchange_a(float (&v)[R][E], uint32_t zc, uint32_t k, uint32_t n_loc, uint64_t L,
                                               uint32_t P, uint32_t part, const GrpMem& g,
                                               GrpSelShared& sh, GrpSmall& sm, GrpState& gs) {
  const uint32_t t = grp_thread<LOOP>();
  auto key = [&](int j, int i) { return mag_key(v[j][i]); };
  const uint32_t par = gs.iter & 1u;
  SelA A;

  // ---- the exact zeros into the first histogram, once per wave
  const uint32_t zs = wave_sum(zc);
  if (lane_id() == 0 && zs) atomicAdd(&sh.hist[0], zs);
  __syncthreads();

  // this workgroup's guess: its own bin at the same rank fraction
  const uint32_t need_loc = (uint32_t)min<uint64_t>(max<uint64_t>(((uint64_t)k * n_loc + L - 1) / L, 1), n_loc);
  find_bin<NT, HIST_BINS>(sh.hist, need_loc, sm.scratch, sm.found);
  const uint32_t bh = sm.found[0];
  // the window: three bins in every workgroup, whatever it guesses (none lies
  // above the last bin), which is what the test of b1 below takes for granted
  const uint32_t lo = bh > 0u ? bh - 1u : 0u;
  const uint32_t hi = min(lo + 2u, (uint32_t)HIST_BINS - 1u);
  // bits 18..14 of the keys in bins lo..hi (the exact zeros, whose bits
  // 18..14 are 0, once per wave)
  refresh(v);
#pragma unroll
  for (int j = 0; j < R; ++j)
#pragma unroll
    for (int i = 0; i < E; ++i) {
      const uint32_t kk = key(j, i), b = kk >> 19;
      // in the window lo..hi (b - lo < 3, unsigned) and not an exact zero
      const uint32_t in = gt31(3u, b - lo) & (eq31(kk, 0u) ^ 1u) & (gt31(lo, b) ^ 1u);
      atomicAdd(&sm.fwin[pick(in, (b - lo) * FINE_N + ((kk >> LOW_BITS) & (FINE_N - 1u)), 3u * FINE_N + (uint32_t)lane_id())], 1u);
    }
  if (lo == 0u && lane_id() == 0 && zs) atomicAdd(&sm.fwin[0], zs);
  __syncthreads();
  // merge into the group's counts
  uint32_t* h1 = g.hist1(par);
  uint32_t* gmax = g.ctl() + 32 + par;
  uint32_t* gmin = g.ctl() + 34 + par;
  const uint32_t first = sat_sub(lo, A_MARGIN);
  for (uint32_t b = (first & ~(uint32_t)(NT - 1)) + t; b < (uint32_t)HIST_BINS; b += NT)
    if (b >= first && sh.hist[b]) add_agent(&h1[b], sh.hist[b]);
  const uint32_t* word = nullptr;   // the word this thread reads back with the histogram
  if (t < 3 * FINE_N) {
    const uint32_t b = lo + t / FINE_N;
    uint32_t* f = &g.fine(par)[(b & (FINE_SLOTS - 1)) * FINE_N + t % FINE_N];
    if (b <= hi && sm.fwin[t]) add_agent(f, sm.fwin[t]);
    word = f;
  } else if (t == 3 * FINE_N) {
    __hip_atomic_fetch_max(gmax, lo + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    word = gmax;
  } else if (t == 3 * FINE_N + 1) {
    __hip_atomic_fetch_max(gmin, (uint32_t)HIST_BINS - lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    word = gmin;
  }
  if (t == 0) sm.found[0] = ~0u;
  group_sync(g.ctl(), P * ++gs.nbar);
  // one round trip: the merged histogram, this window's fine counts, the
  // smallest and largest window
  grp_find_merged<NT>(h1, k, word, &sm.fmrg[t], sm.scratch, sm.found);
  uint32_t b1 = sm.found[0];
  const uint32_t lo_max = sm.fmrg[3 * FINE_N] - 1u, lo_min = (uint32_t)HIST_BINS - sm.fmrg[3 * FINE_N + 1];
  // every window covers b1 (this one's too): bits 18..14 of T from the
  // merged fine counts of b1, by every wavefront alike
  A.fine = b1 != ~0u && lo_max <= b1 && b1 <= lo_min + 2u && b1 - lo <= 2u;
  if (A.fine) {
    const uint32_t need = k - sm.found[1], lane = (uint32_t)lane_id();
    const uint32_t c = (lane < FINE_N) ? sm.fmrg[(b1 - lo) * FINE_N + (FINE_N - 1u - lane)] : 0u;
    const uint32_t incl = wave_incl_scan(c);
    const uint64_t hit = __ballot(lane < FINE_N && incl >= need);
    if (hit == 0 && t == 0) raise_error(KERR_INTERNAL);   // (the counts are complete: a hit is certain)
    const int l = hit ? __builtin_ctzll(hit) : 0;
    A.prefix = (b1 << FINE_BITS) | (FINE_N - 1u - (uint32_t)l);
    A.pbits = 12 + FINE_BITS;
    A.need = need - (uint32_t)__builtin_amdgcn_readlane((int)(incl - c), l);
    __syncthreads();
    return A;
  }
  if (b1 == ~0u || b1 < sat_sub(lo_max, A_MARGIN)) {
    // some workgroup left out bins at or above b1: the rest of the counts,
    // then the search again
    __syncthreads();   // (everybody has read found[])
    for (uint32_t b = t; b < first; b += NT)
      if (sh.hist[b]) add_agent(&h1[b], sh.hist[b]);
    if (t == 0) sm.found[0] = 0u;
    group_sync(g.ctl(), P * ++gs.nbar);
    grp_find_merged<NT>(h1, k, nullptr, nullptr, sm.scratch, sm.found);
    b1 = sm.found[0];
  }
  A.prefix = b1;
  A.pbits = 12;
  A.need = k - sm.found[1];
  __syncthreads();
  return A;
}

// One digit pass (pass p of the segment): the next w <= 8 bits of the keys
// that share the known prefix, counted by every workgroup and merged through
// hist2(p).
template <int NT, int R, int E>
__device__ __forceinline__ void grp_pass(float (&v)[R][E], uint32_t w, uint32_t p, uint32_t P, const GrpMem& g, GrpSelShared& sh,
                                         GrpSmall& sm, GrpState& gs, SelA& A) {
  const int t = (int)threadIdx.x;
  const uint32_t left = 31u - A.pbits, shift = left - w;
  dig_zero<NT>(sh.hist);
  __syncthreads();
  refresh(v);
#pragma unroll
  for (int j = 0; j < R; ++j)
#pragma unroll
    for (int i = 0; i < E; ++i) {
      const uint32_t kk = mag_key(v[j][i]);
      dig_add(sh.hist, (kk >> left) == A.prefix, (kk >> shift) & ((1u << w) - 1u));
    }
  __syncthreads();
  dig_reduce<NT, 256>(sh.hist, sm.red);
  __syncthreads();
  uint32_t* h2 = g.hist2(p);
  if (t < (int)DIG_BINS && sm.red[t]) add_agent(&h2[t], sm.red[t]);
  group_sync(g.ctl(), P * ++gs.nbar);
  if (t < (int)DIG_BINS) sm.red[t] = ld_agent(&h2[t]);
  __syncthreads();
  find_bin_wave<256>(sm.red, A.need, sm.found);
  A.prefix = (A.prefix << w) | sm.found[0];
  A.pbits += w;
  A.need -= sm.found[1];
  __syncthreads();
}
// after a later barrier everybody has read pass p's counts: each workgroup
// clears a slice of them
__device__ __forceinline__ void grp_clear_pass(const GrpMem& g, uint32_t p, uint32_t P, uint32_t part) {
  uint32_t* h2 = g.hist2(p);
  for (uint32_t b = part * GRP_NT + threadIdx.x; b < DIG_BINS; b += P * GRP_NT) st_agent(&h2[b], 0u);
}

// One of this workgroup's keys on the prefix (its low bits), c times, into
// the table of distinct keys.  A table too full to place it raises misc[4]:
// the record is then marked as overflowed.  False once that is so: what else
// is on the prefix need not enter (up to 12,288 distinct keys, each of which
// would try its eight places: 16 x 200,000 binary32 within 2^-9 of 1, TopK 10 %,
// 131 us without this test and with one exchange more in the fallback, now 91).
__device__ __forceinline__ bool grp_rle_add(GrpSmall& sm, uint32_t low, uint32_t c) {
  if (__hip_atomic_load(&sm.misc[4], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != 0u) return false;
  uint32_t h = ((low * 0x9E5u) >> 4) & (RLE_SLOTS - 1u);
  for (uint32_t p = 0; p < RLE_PROBES; ++p) {
    const uint32_t old = atomicCAS(&sm.hk[h], 0u, low + 1u);
    if (old == 0u || old == low + 1u) {
      atomicAdd(&sm.hc[h], c);
      return true;
    }
    h = (h + 1u) & (RLE_SLOTS - 1u);
  }
  sm.misc[4] = 1u;
  return false;
}

// Exchange B (fine mode), first half.  A record is a header (the keys above
// the prefix, below 2^16, and REC_OVF << 16 when its keys did not fit) and
// entries: a key's low bits and its multiplicity << LOW_BITS (at most 12,288;
// an unused entry is 0).  Before calling, this workgroup has either put one
// entry per key on the prefix into sm.rec (direct) or its keys into the table
// of distinct keys.  The first wavefront stores the record with one
// instruction and arrives at the group's barrier; nobody waits here.
template <int NT>
__device__ __forceinline__ void grp_publish_b(uint32_t part, const GrpMem& g, GrpSmall& sm, GrpState& gs,
                                              uint32_t abv_wg, bool direct) {
  __syncthreads();   // the entries or the table are complete
  ++gs.nbar;
  if (threadIdx.x >= WAVE) return;
  const uint32_t lane = threadIdx.x;
  uint32_t hdr = abv_wg;
  if (!direct) {
    const uint32_t kx = sm.hk[lane], c = sm.hc[lane];
    const uint64_t in = __ballot(kx != 0u);
    const uint32_t q = lanes_below(in);
    if (kx != 0u && q < REC_KEYS) sm.rec[1 + q] = (kx - 1u) | (c << LOW_BITS);
    if ((uint32_t)__popcll(in) > REC_KEYS || sm.misc[4] != 0u) hdr |= REC_OVF << 16;
  }
  // (a wavefront's LDS accesses complete in program order)
  __builtin_amdgcn_wave_barrier();
  if (lane < REC_W) st_agent(&g.rec()[(uint64_t)part * REC_W + lane], lane == 0 ? hdr : sm.rec[lane]);
  __builtin_amdgcn_s_waitcnt(0);
  if (lane == 0) __hip_atomic_fetch_add(g.ctl(), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// the bin d of a 128-bin histogram in LDS with  sum_{c > d} h[c] < need <=
// sum_{c >= d} h[c], and that first sum; every wavefront finds it alike
__device__ __forceinline__ void wave_find128(const uint32_t* h, uint32_t need, uint32_t& d, uint32_t& above) {
  const uint32_t lane = (uint32_t)lane_id();
  const uint32_t c0 = h[2 * lane], c1 = h[2 * lane + 1], sum = c0 + c1;
  const uint32_t incl = wave_incl_scan(sum);
  const uint32_t acc = (uint32_t)__builtin_amdgcn_readlane((int)incl, WAVE - 1) - incl;   // bins of higher lanes
  const uint64_t hit = __ballot(acc < need && need <= acc + sum);
  const uint32_t dd = (acc + c1 >= need) ? 2 * lane + 1 : 2 * lane;
  const uint32_t aa = (acc + c1 >= need) ? acc : acc + c1;
  const int l = hit ? __builtin_ctzll(hit) : 0;   // (a hit is certain: the counts cover need)
  d = (uint32_t)__builtin_amdgcn_readlane((int)dd, l);
  above = (uint32_t)__builtin_amdgcn_readlane((int)aa, l);
}

// Exchange B, second half: waits for the group, reads all records in one
// round trip (SPT words per thread, two per access: up to 16 * SPT workgroups)
// and finds T, the tie quota and the larger keys and ties of lower workgroups
// (the last after one more barrier, by grp_finish_b_lower).  Returns false (nothing
// decided) when some record could not hold its keys; the words of exchange A
// (fine) or of the digit pass after it are cleared either way.
template <int NT, int SPT, bool LOOP>
__device__ __forceinline__ bool grp_finish_b(uint32_t P, uint32_t part, const GrpMem& g, GrpSmall& sm, GrpState& gs,
                                             const SelA& A, SelResult& res) {
  constexpr int NW = NT / WAVE;
  constexpr int LP = SPT / 2;                     // 8-byte loads per thread
  constexpr uint32_t PERW = WAVE * 2 / REC_W;     // records per wavefront read
  static_assert(WAVE * 2 % REC_W == 0, "whole records per wavefront read");
  const uint32_t t = grp_thread<LOOP>(), wv = t / WAVE, lane = t % WAVE;
  const uint32_t sub = lane / (REC_W / 2), wi = lane % (REC_W / 2);
  group_wait(g.ctl(), P * gs.nbar);
  // lane i of wavefront wv reads words 2 (i % 16) and + 1 of record
  // 4 * (u*NW + wv) + i / 16 (the last record again in place of one past it)
  const uint64_t* rec = reinterpret_cast<const uint64_t*>(g.rec());
  uint32_t wd[SPT];
#pragma unroll
  for (int u = 0; u < LP; ++u) {
    const uint32_t w = PERW * (uint32_t)(u * NW + wv) + sub;
    const uint64_t x = ld_agent64(&rec[min(w, P - 1u) * (REC_W / 2) + wi]);
    wd[2 * u] = (uint32_t)x;
    wd[2 * u + 1] = (uint32_t)(x >> 32);
  }
  if (A.fine) grp_clear_a(g, gs.iter & 1u, P, part);
  else grp_clear_pass(g, 0, P, part);
  // headers (the first word of a record) give the keys above the prefix before
  // this workgroup; entries count into the histogram of their bits 13..7
  uint32_t abv = 0, bad = 0;
#pragma unroll
  for (int u = 0; u < LP; ++u) {
    const uint32_t w = PERW * (uint32_t)(u * NW + wv) + sub;
    const bool head = wi == 0u;
    abv += (head && w < part) ? wd[2 * u] & 0xFFFFu : 0u;
    bad |= head ? wd[2 * u] >> 16 : 0u;
    wd[2 * u] = (head || w >= P) ? 0u : wd[2 * u];
    wd[2 * u + 1] = (w >= P) ? 0u : wd[2 * u + 1];
  }
#pragma unroll
  for (int u = 0; u < SPT; ++u) {
    const uint32_t c = wd[u] >> LOW_BITS;
    atomicAdd(&sm.h7a[c ? (wd[u] >> 7) & 0x7Fu : (uint32_t)LAST_BINS + lane], c);
  }
  abv = wave_sum(abv);
  const bool wbad = __ballot(bad != 0u) != 0u;
  uint32_t* tsc = sm.scratch + 5 * NW;   // clear of the sums below
  if (lane == 0) { tsc[wv] = abv; tsc[NW + wv] = wbad ? 1u : 0u; }
  __syncthreads();
  uint32_t abv_bef = 0;
  bad = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) { abv_bef += tsc[i]; bad |= tsc[NW + i]; }
  if (bad != 0) return false;
  uint32_t da, db, above;
  wave_find128(sm.h7a, A.need, da, above);
  const uint32_t need_c = A.need - above;
#pragma unroll
  for (int u = 0; u < SPT; ++u) {
    const uint32_t c = (((wd[u] >> 7) & 0x7Fu) == da) ? wd[u] >> LOW_BITS : 0u;
    atomicAdd(&sm.h7b[c ? wd[u] & 0x7Fu : (uint32_t)LAST_BINS + lane], c);
  }
  __syncthreads();
  wave_find128(sm.h7b, need_c, db, above);
  const uint32_t low = (da << 7) | db;
  res.T = (A.prefix << (31u - A.pbits)) | low;
  res.r = need_c - above;
  // larger keys and ties in lower workgroups' records, summed per wavefront
  // into sm.scratch: grp_finish_b_lower adds them up after the caller's next
  // barrier
  uint32_t gt = 0, eq = 0;
#pragma unroll
  for (int u = 0; u < SPT; ++u) {
    const uint32_t w = PERW * (uint32_t)((u / 2) * NW + wv) + sub;
    const uint32_t c = (w < part) ? wd[u] >> LOW_BITS : 0u, kl = wd[u] & ((1u << LOW_BITS) - 1u);
    gt += (kl > low) ? c : 0u;
    eq += (kl == low) ? c : 0u;
  }
  gt = wave_sum(gt);
  eq = wave_sum(eq);
  if (lane == 0) { sm.scratch[wv] = gt; sm.scratch[NW + wv] = eq; }
  res.gt_before = abv_bef;
  res.eq_before = 0;
  return true;
}

template <int NT>
__device__ __forceinline__ void grp_finish_b_lower(const GrpSmall& sm, SelResult& res) {
  constexpr int NW = NT / WAVE;
#pragma unroll
  for (int i = 0; i < NW; ++i) { res.gt_before += sm.scratch[i]; res.eq_before += sm.scratch[NW + i]; }
}

// The exact passes once a record overflowed: a digit pass of 8 bits merged
// through device memory, then the last bits (at most 6) counted per workgroup,
// which also gives what precedes this workgroup.  `pass`: digit passes already
// done for this segment.
template <int NT, int R, int E, bool LOOP>
__device__ __forceinline__ SelResult grp_fallback(float (&v)[R][E], uint32_t P, uint32_t part, const GrpMem& g,
                                                  GrpSelShared& sh, GrpSmall& sm, GrpState& gs,
                                                  SelA A, uint32_t pass) {
  constexpr uint32_t NW = NT / WAVE;
  const uint32_t t = grp_thread<LOOP>(), wv = t / WAVE, lane = t % WAVE;
  grp_pass<NT, R, E>(v, 8u, pass, P, g, sh, sm, gs, A);
  // ---- the last digit: this workgroup's counts, and its keys above the prefix
  const uint32_t left = 31u - A.pbits;
  dig_zero<NT>(sh.hist);
  __syncthreads();
  refresh(v);
  uint32_t gt = 0;
#pragma unroll
  for (int j = 0; j < R; ++j)
#pragma unroll
    for (int i = 0; i < E; ++i) {
      const uint32_t kk = mag_key(v[j][i]), hi = kk >> left;
      dig_add(sh.hist, hi == A.prefix, kk & ((1u << left) - 1u));
      gt += gt31(hi, A.prefix);
    }
  const uint32_t gt_wg = block_sum<NT>(gt, sm.scratch);   // (contains barriers)
  dig_reduce<NT, CNT_BINS>(sh.hist, sm.red);
  uint32_t* cnt = g.cnt();
  gs.used_cnt = true;
  if (t < CNT_BINS) st_agent(&cnt[part * CNT_W + t], sm.red[t]);
  else if (t == CNT_BINS) st_agent(&cnt[part * CNT_W + t], gt_wg);
  group_sync(g.ctl(), P * ++gs.nbar);
  grp_clear_pass(g, pass, P, part);
  // lane b of a wavefront adds up bin b of every eighth workgroup
  static_assert(CNT_BINS == (uint32_t)WAVE, "a bin per lane");
  uint32_t all = 0, bef = 0;
#pragma unroll 4
  for (uint32_t w = wv; w < P; w += NW) {
    const uint32_t c = ld_agent(&cnt[w * CNT_W + lane]);
    all += c;
    bef += (w < part) ? c : 0u;
  }
  uint32_t gtb = 0;
  for (uint32_t w = t; w < part; w += NT) gtb += ld_agent(&cnt[w * CNT_W + CNT_BINS]);
  sh.hist[(wv * 2u) * WAVE + lane] = all;
  sh.hist[(wv * 2u + 1u) * WAVE + lane] = bef;
  SelResult res;
  res.gt_before = block_sum<NT>(gtb, sm.scratch);         // (contains barriers)
  all = 0;
  bef = 0;
#pragma unroll
  for (uint32_t w = 0; w < NW; ++w) {
    // (bins from the top: lane l takes bin 63 - l)
    all += sh.hist[(w * 2u) * WAVE + (WAVE - 1u - lane)];
    bef += sh.hist[(w * 2u + 1u) * WAVE + (WAVE - 1u - lane)];
  }
  const uint32_t incl = wave_incl_scan(all), bincl = wave_incl_scan(bef);
  const uint64_t hit = __ballot(incl - all < A.need && A.need <= incl);
  if (hit == 0 && t == 0) raise_error(KERR_INTERNAL);   // (the counts cover need: a hit is certain)
  const int l = hit ? __builtin_ctzll(hit) : 0;
  res.T = (A.prefix << left) | (WAVE - 1u - (uint32_t)l);
  res.r = A.need - (uint32_t)__builtin_amdgcn_readlane((int)(incl - all), l);
  res.gt_before += (uint32_t)__builtin_amdgcn_readlane((int)(bincl - bef), l);
  res.eq_before = (uint32_t)__builtin_amdgcn_readlane((int)bef, l);
  __syncthreads();
  return res;
}

// Leave the group's workspace zero.  Every workgroup takes an exit ticket
// once it has read the last exchange words (grp_exit_ticket: the atomic is
// issued, nobody waits for it); at its very end, the workgroup that drew the
// last ticket (all others have finished reading) clears the barrier words,
// the records and, if the fallback ran, the workgroups' counts; everything
// else is cleared in flight.
__device__ __forceinline__ uint32_t grp_exit_ticket(const GrpMem& g) {
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  uint32_t prev = 0;
  if (threadIdx.x == 0) prev = __hip_atomic_fetch_add(g.ctl() + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return prev;   // thread 0's ticket; other threads' values are meaningless
}

template <int NT>
__device__ __forceinline__ void grp_exit_finish(const GrpMem& g, uint32_t P, const GrpState& gs, uint32_t ticket,
                                                uint32_t* flag) {
  if (threadIdx.x == 0) *flag = (ticket == P - 1) ? 1u : 0u;
  __syncthreads();
  if (!*flag) return;
  // the records and the counts lie back to back
  const uint32_t n = P * (REC_W + (gs.used_cnt ? CNT_W : 0u));
  uint32_t* rec = g.rec();
  for (uint32_t i = threadIdx.x; i < n; i += NT) st_agent(&rec[i], 0u);
  if (threadIdx.x == 0) {
    st_agent(g.ctl(), 0u);
    st_agent(g.ctl() + 1, 0u);
  }
}

}  // namespace tc
