// Variable-length partitioner (section 3.2.2) on the GPU.
//
// Split: the greedy of the paper, which includes the next value in the
// current partition while the approximate cost of doing so,
//   C = (len + 1) * D~new - len * D~old,  D~ = bitlen(max d - min d)
// over the partition's first differences d, stays within tau * S_M, and
// the partition holds fewer than max_len values.  The column is cut into
// 2^11-value sub-chunks that are first split speculatively in parallel, as
// if a partition began at each one's start, and then again from the state
// that its left neighbour ended in, until this run starts a partition where
// the first one did (from there on the two runs are the same), rewriting the
// starts it passes.  Where a sub-chunk holds no such place, one wavefront per
// 2^20-value segment walks the next ones on from its end; a last wavefront
// does the same across segments, from the end state of each segment to the
// next.  The wavefront walks 64 candidates at a
// time (see greedy_walk).  This reproduces the sequential greedy exactly.
// Optionally the split also honours starting partitions (section 3.2.2,
// selecting good starting positions): runs of smallest second-order delta,
// whose first value begins a partition and whose other values join it
// without the cost test.
//
// Merge: the paper's scan.  The current partition merges with its right
// neighbour when the union (sized with the encoder's own fit: 32-byte
// record, 8-byte start, residual words) is strictly smaller than the two
// apart and fits max_len, and then tries the next neighbour; passes repeat
// until one merges nothing.  The scan's state is the current partition
// (its first index and size), and it is reset by every refused merge, so
// the same speculation applies: chunks of the partition list are scanned
// in parallel as if a partition began at each chunk's start; then, in
// rounds of alternating parity, every chunk whose left neighbour's end
// state changed is walked again from it until it keeps a boundary its
// recorded run also kept.  A run of merges spanning c chunks takes about c
// rounds.  Within a run, 256 steps are sized at once (one per thread of a
// workgroup), and a long current partition is represented by the convex hulls
// of its points, so a step costs neither the union's values nor those it adds.
//
// What bounds a column whose runs are long (a noisy polyline of 1e7 values:
// partitions of two values merged into partitions of up to 370,000) is the
// latency of the batches along its longest run, one chunk per round: a walker
// takes 20 to 33 us for 256 steps and 50 to 60 where every second CU has one,
// and a round lasts as long as its slowest (58 rounds, 28 ms).  With
// one wavefront, 64 steps a batch, every added value broadcast to all lanes
// and the hulls kept by a serial chain it was 60 us for 64, and short chunks
// re-walked most of the column in every round: 512 -> 48 ms (in order: hulls
// by parallel peeling, unions sized by bounds of two hulls, 4096-boundary
// chunks and a workgroup per walker; then the split's look-ahead), sorted
// normal samples 30 -> 7 ms.
#include <math.h>

#include <utility>
#include <vector>

#include "fit.hpp"
#include "internal.hpp"
#include "leco_dev.hpp"
#include "minimax.hpp"

namespace leco {

constexpr uint32_t kSegLog2 = 20;
constexpr uint32_t kSubLog2 = 11;  // speculative split sub-chunks of a segment
constexpr uint32_t kSplitWindow = 1024;  // values staged in LDS per window
constexpr uint32_t kSplitAhead = 16;      // values one lane tries in a row (split_ahead)
constexpr uint32_t kScanBlock = 256;
constexpr uint32_t kItemsPerBlock = 1024;  // bitmap words or flags per scan block
constexpr uint64_t kNoMerge = ~uint64_t(0);

// A first difference d = v_j - v_{j-1} of (up to) 64-bit values as the
// 65-bit unsigned number d + 2^64 = (hi, lo), which orders like d.
struct DKey {
  uint32_t hi;
  uint64_t lo;
};

__device__ inline bool key_less(const DKey& a, const DKey& b) {
  return a.hi != b.hi ? a.hi < b.hi : a.lo < b.lo;
}

__device__ inline DKey key_shfl_up(const DKey& k, int delta) {
  DKey r;
  r.hi = uint32_t(__shfl_up(int(k.hi), delta, 64));
  r.lo = uint64_t(__shfl_up(static_cast<unsigned long long>(k.lo), delta, 64));
  return r;
}

__device__ inline DKey key_readlane(const DKey& k, int lane) {
  DKey r;
  r.hi = uint32_t(__shfl(int(k.hi), lane, 64));
  r.lo = uint64_t(__shfl(static_cast<unsigned long long>(k.lo), lane, 64));
  return r;
}

// bitlen(max - min) of two keys (at most 65).
__device__ inline uint32_t key_span_bits(const DKey& mn, const DKey& mx) {
  const uint64_t lo = mx.lo - mn.lo;
  const uint32_t hi = mx.hi - mn.hi - (mx.lo < mn.lo ? 1u : 0u);
  return hi ? 65u : bitlen64(lo);
}

// For 32-bit columns a first difference fits 33 bits: the key d + 2^32 is
// one 64-bit word (two 32-bit shuffles instead of three).
__device__ inline bool key_less(uint64_t a, uint64_t b) { return a < b; }
__device__ inline uint64_t key_shfl_up(uint64_t k, int delta) {
  return uint64_t(__shfl_up(static_cast<unsigned long long>(k), delta, 64));
}
__device__ inline uint64_t key_readlane(uint64_t k, int lane) {
  return uint64_t(__shfl(static_cast<unsigned long long>(k), lane, 64));
}
__device__ inline uint32_t key_span_bits(uint64_t mn, uint64_t mx) { return bitlen64(mx - mn); }

// Key of the first difference v_j - v_{j-1}, and the state's stored form.
__device__ inline DKey make_key(DKey*, uint64_t vj, uint64_t vp) {
  return DKey{vj >= vp ? 1u : 0u, vj - vp};
}
__device__ inline uint64_t make_key(uint64_t*, uint64_t vj, uint64_t vp) {
  return vj - vp + (uint64_t(1) << 32);  // v < 2^32
}
__device__ inline DKey key_from(DKey*, uint32_t hi, uint64_t lo) { return DKey{hi, lo}; }
__device__ inline uint64_t key_from(uint64_t*, uint32_t, uint64_t lo) { return lo; }
__device__ inline uint32_t key_hi(const DKey& k) { return k.hi; }
__device__ inline uint32_t key_hi(uint64_t) { return 0; }
__device__ inline uint64_t key_lo(const DKey& k) { return k.lo; }
__device__ inline uint64_t key_lo(uint64_t k) { return k; }

__device__ inline void mark(unsigned long long* bitmap, uint64_t j) {
  atomicOr(bitmap + (j >> 6), 1ull << (j & 63));
}

// The greedy's state: the current partition's first value i, and whether
// it has first differences yet with their min / max keys and D~.
struct SplitState {
  uint64_t i;
  uint64_t kmin_lo, kmax_lo;
  uint32_t kmin_hi, kmax_hi;
  uint32_t w_old, have;
};

// Clears bits [x, y) of the bitmap (y - x <= 128, so at most three words).
__device__ inline void clear_bits(unsigned long long* bitmap, uint64_t x, uint64_t y) {
  while (x < y) {
    const uint64_t w = x >> 6;
    const uint64_t hi = (y - (w << 6)) < 64 ? y - (w << 6) : 64;  // bit bound in word w
    const uint64_t lo = x & 63;
    const uint64_t mask = (hi == 64 ? ~0ull : ((1ull << hi) - 1)) & ~((1ull << lo) - 1);
    atomicAnd(bitmap + w, ~mask);
    x = (w + 1) << 6;
  }
}

__device__ inline bool bit_set(unsigned long long* bitmap, uint64_t j) {
  const unsigned long long word =
      __hip_atomic_load(bitmap + (j >> 6), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return (word >> (j & 63)) & 1ull;
}

// The greedy from 64 partition starts at once: lane l takes v[p - 1 + l] as a
// partition's first value and tries up to kSplitAhead values after it, so
// that each knows where the next partition would begin, if it is that near
// (0: not known).  win[0] is v[p - 1]; candidates end before b.
template <class K>
__device__ inline uint32_t split_ahead(const uint64_t* win, uint64_t p, uint64_t b, double thr,
                                       uint64_t max_len) {
  const uint32_t lane = threadIdx.x & 63;
  // tries 1 .. reach stay before b; of a partition of max_len values the
  // next one begins without the cost test
  const uint64_t after = b - (p - 1);
  const uint32_t reach = after <= lane + 1 ? 0 : uint32_t(after - lane - 1 < kSplitAhead ? after - lane - 1 : kSplitAhead);
  const uint32_t cap = uint32_t(max_len < kSplitAhead + 1 ? max_len : kSplitAhead + 1);
  uint32_t next = 0;
  int32_t w_old = 0;
  uint64_t prev = win[reach ? lane : 0];  // lanes past b read nothing past it
  K mn = make_key(static_cast<K*>(nullptr), 0, 0), mx = mn;
  for (uint32_t k = 1; k <= kSplitAhead; ++k) {
    const bool on = next == 0 && k <= reach;
    if (__ballot(on) == 0) break;
    const uint64_t v = win[on ? lane + k : 0];
    const K d = make_key(static_cast<K*>(nullptr), v, prev);
    prev = v;
    if (k == 1 || key_less(d, mn)) mn = d;
    if (k == 1 || key_less(mx, d)) mx = d;
    const int32_t w_new = int32_t(key_span_bits(mn, mx));
    const int32_t cost = int32_t(k + 1) * w_new - int32_t(k) * w_old;
    w_old = w_new;
    if (on && !(k < cap && double(cost) <= thr)) next = k;
  }
  return next;
}

// Runs the greedy over candidates [p, b) from state st, 64 candidates per
// step: lane l assumes the values before its own are all included, takes
// the inclusive prefix min / max of the first differences over the lanes
// below it and evaluates C; the first lane that fails starts the next
// partition and the lanes after it are retried from there.
//
// kFix = false: sets the bit of every start.  kFix = true: the bits in
// [p, b) are a speculative run's, made from a different state; the walk
// rewrites them until it starts a partition where the speculative run also
// did (from there on both runs are the same), returning true at that point.
//
// Where partitions are short that is a step of about 1 us for each, the
// latency of its scans.  So after a partition of at most kSplitAhead values,
// and at the walk's start, the lanes run the greedy from 64 starts in a row
// (split_ahead) and the partitions are read off as a chain of them, as far as
// it is known: a 2^14-value sub-chunk of normal samples, in partitions of two
// or three, took 5.8 ms and takes 0.78, one of 2^11 0.10.
//
// forced and inside (both null, or both bitmaps over the column): bit j of
// forced set means a partition begins at j (the first value of a starting
// partition), whatever the cost; bit j of inside set means v[j] joins the
// current partition without the cost test (a later value of a starting
// partition).  The length cap applies to both.
//
// K: the key type, DKey for 64-bit columns, one 64-bit word for 32-bit ones.
template <bool kFix, class K>
__device__ bool greedy_walk(const uint8_t* __restrict__ col, uint32_t dtype, uint64_t p,
                            uint64_t b, double thr, uint64_t max_len, SplitState& st,
                            uint64_t* win, unsigned long long* __restrict__ bitmap,
                            const uint64_t* __restrict__ forced,
                            const uint64_t* __restrict__ inside) {
  const uint32_t lane = threadIdx.x & 63;
  K kmin = key_from(static_cast<K*>(nullptr), st.kmin_hi, st.kmin_lo);
  K kmax = key_from(static_cast<K*>(nullptr), st.kmax_hi, st.kmax_lo);
  uint64_t i = st.i;
  bool have = st.have != 0;
  uint32_t w_old = st.w_old;
  uint64_t base = 0, wend = 0;  // the window holds v[base - 1, wend)
  bool synced = false;
  bool ahead = forced == nullptr;
  while (p < b) {
    const uint64_t need = p + 64 + kSplitAhead < b ? p + 64 + kSplitAhead : b;
    if (wend < need) {
      __syncthreads();  // every lane is done with the old window
      base = p;
      wend = b - p < kSplitWindow ? b : p + kSplitWindow;
      for (uint64_t k = lane; k <= wend - base; k += 64)
        win[k] = load_value(col, dtype, base - 1 + k);
      __syncthreads();
    }
    if (ahead && !have) {  // v[i] = v[p - 1] is the partition's only value yet
      const uint32_t next = split_ahead<K>(win + (p - base), p, b, thr, max_len);
      // bit x of (found1, found0): a partition begins at p + x
      uint64_t found0 = 0, found1 = 0;
      uint32_t at = 0;  // of the last one found: p - 1 + at
      while (at < 64) {
        const uint32_t k = uint32_t(__builtin_amdgcn_readlane(int(next), int(at)));
        if (k == 0) break;
        at += k;
        if (at <= 64)
          found0 |= 1ull << (at - 1);
        else
          found1 |= 1ull << (at - 65);
      }
      ahead = at >= 64;
      if (at != 0) {
        // words of the bitmap that hold bits p .. p + at - 1: three at most
        const uint32_t sh = uint32_t(p & 63);
        const auto word_of = [&](uint64_t m0, uint64_t m1) {
          return lane == 0   ? m0 << sh
                 : lane == 1 ? (sh ? m0 >> (64 - sh) : 0) | m1 << sh
                             : (sh ? m1 >> (64 - sh) : 0);
        };
        unsigned long long* word = bitmap + (p >> 6) + lane;
        uint64_t range0 = at >= 64 ? ~0ull : (1ull << at) - 1;
        uint64_t range1 = at > 64 ? (1ull << (at - 64)) - 1 : 0;
        if (kFix) {
          // the first start of both runs, if any, ends the walk
          uint64_t both = 0;
          if (lane < 3 && word_of(range0, range1) != 0)
            both = word_of(found0, found1) &
                   __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          const uint64_t hit = __ballot(both != 0);
          if (hit != 0) {
            const int w = __ffsll(static_cast<long long>(hit)) - 1;
            const uint64_t bits = uint64_t(__shfl(static_cast<unsigned long long>(both), w, 64));
            const uint64_t js = (((p >> 6) + uint64_t(w)) << 6) + uint64_t(__ffsll(static_cast<long long>(bits)) - 1);
            at = uint32_t(js - p) + 1;
            // up to js, whose bit is set
            range0 = at > 64 ? ~0ull : (1ull << (at - 1)) - 1;
            range1 = at > 64 ? (1ull << (at - 65)) - 1 : 0;
            found0 &= range0;
            found1 &= range1;
            synced = true;
          }
          if (lane < 3) {
            const uint64_t gone = word_of(range0 & ~found0, range1 & ~found1);
            if (gone) atomicAnd(word, ~gone);
          }
        }
        if (lane < 3) {
          const uint64_t put = word_of(found0, found1);
          if (put) atomicOr(word, put);
        }
        i = p - 1 + at;
        w_old = 0;
        p += at;
        if (synced) break;
        continue;
      }
    }
    const uint64_t j = p + lane;
    const bool valid = j < b;
    K d = make_key(static_cast<K*>(nullptr), 0, 0);
    if (valid) d = make_key(static_cast<K*>(nullptr), win[j - base + 1], win[j - base]);
    // inclusive prefix min / max over the lanes up to this one; the invalid
    // lanes are the last ones and never feed a valid lane
    K mn = d, mx = d;
#pragma unroll
    for (int delta = 1; delta < 64; delta <<= 1) {
      const K lo = key_shfl_up(mn, delta), hi = key_shfl_up(mx, delta);
      if (int(lane) >= delta) {
        if (key_less(lo, mn)) mn = lo;
        if (key_less(mx, hi)) mx = hi;
      }
    }
    if (have) {
      if (key_less(kmin, mn)) mn = kmin;
      if (key_less(mx, kmax)) mx = kmax;
    }
    const uint32_t w_new = key_span_bits(mn, mx);
    uint32_t w_prev = uint32_t(__shfl_up(int(w_new), 1, 64));
    if (lane == 0) w_prev = w_old;
    const uint64_t len = j - i;
    const int64_t cost = int64_t((len + 1) * w_new) - int64_t(len * w_prev);
    const bool start_here = forced && valid && ((forced[j >> 6] >> (j & 63)) & 1ull);
    const bool in_start = forced && valid && ((inside[j >> 6] >> (j & 63)) & 1ull);
    const bool include = len < max_len && !start_here && (in_start || double(cost) <= thr);
    const uint64_t split = __ballot(valid && !include);
    if (split == 0) {
      const int last = int(b - p - 1 < 63 ? b - p - 1 : 63);
      if (kFix && lane == 0) clear_bits(bitmap, p, p + uint64_t(last) + 1);
      kmin = key_readlane(mn, last);
      kmax = key_readlane(mx, last);
      w_old = uint32_t(__shfl(int(w_new), last, 64));
      have = true;
      p += uint64_t(last) + 1;
      // Differences within the partition's own leave D~ alone, so that each
      // of their values costs D~: whole steps without a scan where that is
      // allowed, none of them must begin a partition and all have room.  One
      // partition of 2e5 u64 values took 4.8 ms (in order, 64 values per 1.4
      // us) and takes 1.9.
      if (double(w_old) <= thr) {
        for (; p + 64 <= wend && p + 63 - i < max_len; p += 64) {
          const uint64_t x = p + lane;
          const K e = make_key(static_cast<K*>(nullptr), win[x - base + 1], win[x - base]);
          bool apart = key_less(e, kmin) || key_less(kmax, e);
          if (forced) apart = apart || ((forced[x >> 6] >> (x & 63)) & 1ull);
          if (__ballot(apart) != 0) break;
          if (kFix && lane == 0) clear_bits(bitmap, p, p + 64);
        }
      }
    } else {
      const uint64_t js = p + uint64_t(__ffsll(static_cast<long long>(split)) - 1);
      if (kFix) {
        bool hit = false;
        if (lane == 0) {
          clear_bits(bitmap, p, js);
          hit = bit_set(bitmap, js);
          if (!hit) mark(bitmap, js);
        }
        synced = __ballot(hit) != 0;
      } else if (lane == 0) {
        mark(bitmap, js);
      }
      ahead = forced == nullptr && js - i <= kSplitAhead;
      i = js;
      have = false;
      w_old = 0;
      p = js + 1;
      if (synced) break;
    }
  }
  st.i = i;
  st.have = have ? 1u : 0u;
  st.kmin_hi = key_hi(kmin);
  st.kmin_lo = key_lo(kmin);
  st.kmax_hi = key_hi(kmax);
  st.kmax_lo = key_lo(kmax);
  st.w_old = w_old;
  return synced;
}

// Speculative split: one 64-lane workgroup per 2^kSubLog2-value sub-chunk.
// Sub-chunk 0 of the column begins where a partition really begins; the
// others begin a partition at their own start, which the fix-up passes
// correct.  Each records its final state.
__global__ __launch_bounds__(64) void k_split_spec(const uint8_t* __restrict__ col,
                                                   uint32_t dtype, uint64_t n, double thr,
                                                   uint64_t max_len,
                                                   unsigned long long* __restrict__ bitmap,
                                                   SplitState* __restrict__ states,
                                                   const uint64_t* __restrict__ forced,
                                                   const uint64_t* __restrict__ inside) {
  __shared__ uint64_t win[kSplitWindow + 1];  // win[k] = v[base - 1 + k]
  const uint64_t a = uint64_t(blockIdx.x) << kSubLog2;
  if (a >= n) return;
  const uint64_t b = n - a < (uint64_t(1) << kSubLog2) ? n : a + (uint64_t(1) << kSubLog2);
  if (threadIdx.x == 0) mark(bitmap, a);
  SplitState st{a, 0, 0, 0, 0, 0, 0};
  if (dtype == 4)
    greedy_walk<false, uint64_t>(col, dtype, a + 1, b, thr, max_len, st, win, bitmap, forced,
                                 inside);
  else
    greedy_walk<false, DKey>(col, dtype, a + 1, b, thr, max_len, st, win, bitmap, forced, inside);
  if (threadIdx.x == 0) states[blockIdx.x] = st;
}

// Walks sub-chunks [q, q_end) of the column in order from state st (fix
// mode), each from the state the previous one ends in; returns at the
// first sub-chunk where the walk meets the starts already there (st is
// then that meeting's state, and the caller continues from the run already
// recorded), or after the last one with st its end state.
__device__ bool walk_subchunks(const uint8_t* col, uint32_t dtype, uint64_t n, double thr,
                               uint64_t max_len, uint64_t q, uint64_t q_end, SplitState& st,
                               uint64_t* win, unsigned long long* bitmap, const uint64_t* forced,
                               const uint64_t* inside) {
  for (; q < q_end; ++q) {
    const uint64_t aq = q << kSubLog2;
    if (aq >= n) break;
    const uint64_t bq = n - aq < (uint64_t(1) << kSubLog2) ? n : aq + (uint64_t(1) << kSubLog2);
    const bool synced =
        dtype == 4
            ? greedy_walk<true, uint64_t>(col, dtype, aq, bq, thr, max_len, st, win, bitmap, forced,
                                          inside)
            : greedy_walk<true, DKey>(col, dtype, aq, bq, thr, max_len, st, win, bitmap, forced,
                                      inside);
    if (synced) return true;
  }
  return false;
}

// Every sub-chunk but a segment's first again, from the speculative end
// state of the one before it, until it meets its own speculative starts.
// met[q]: it did, so that it ends as the speculative run does (if the one
// before it did too); else ends[q] is its end state.  Partitions are short
// enough to meet in nearly all columns, and one wavefront that walked a
// segment's sub-chunks in order took 6 us for each.
__global__ __launch_bounds__(64) void k_split_meet(const uint8_t* __restrict__ col,
                                                   uint32_t dtype, uint64_t n, double thr,
                                                   uint64_t max_len,
                                                   unsigned long long* __restrict__ bitmap,
                                                   const SplitState* __restrict__ states,
                                                   SplitState* __restrict__ ends,
                                                   uint8_t* __restrict__ met,
                                                   const uint64_t* __restrict__ forced,
                                                   const uint64_t* __restrict__ inside) {
  __shared__ uint64_t win[kSplitWindow + 1];
  constexpr uint64_t kSubs = uint64_t(1) << (kSegLog2 - kSubLog2);
  const uint64_t q = blockIdx.x;
  if (q << kSubLog2 >= n) return;
  bool same = true;
  if (q % kSubs != 0) {
    SplitState st = states[q - 1];
    same = walk_subchunks(col, dtype, n, thr, max_len, q, q + 1, st, win, bitmap, forced, inside);
    if (!same && threadIdx.x == 0) ends[q] = st;
  }
  if (threadIdx.x == 0) met[q] = same ? 1 : 0;
}

// Fix-up within segments: one workgroup per 2^20-value segment walks on from
// each sub-chunk that did not meet its speculative starts, until a later one
// does; the segment's end state (as if a partition began at the segment
// start) goes to seg_states.
__global__ __launch_bounds__(64) void k_split_fix(const uint8_t* __restrict__ col,
                                                  uint32_t dtype, uint64_t n, double thr,
                                                  uint64_t max_len,
                                                  unsigned long long* __restrict__ bitmap,
                                                  const SplitState* __restrict__ states,
                                                  const SplitState* __restrict__ ends,
                                                  const uint8_t* __restrict__ met,
                                                  SplitState* __restrict__ seg_states,
                                                  const uint64_t* __restrict__ forced,
                                                  const uint64_t* __restrict__ inside) {
  __shared__ uint64_t win[kSplitWindow + 1];
  constexpr uint64_t kSubs = uint64_t(1) << (kSegLog2 - kSubLog2);
  const uint64_t a = uint64_t(blockIdx.x) << kSegLog2;
  if (a >= n) return;
  const uint64_t q0 = uint64_t(blockIdx.x) * kSubs;
  const uint64_t nsub = (n + (uint64_t(1) << kSubLog2) - 1) >> kSubLog2;
  const uint64_t q_end = q0 + kSubs < nsub ? q0 + kSubs : nsub;
  SplitState st = states[q_end - 1];
  for (uint64_t q = q0 + 1; q < q_end;) {
    const uint64_t at = q + threadIdx.x;
    const uint64_t apart = __ballot(at < q_end && met[at < q_end ? at : q] == 0);
    if (apart == 0) {
      q += 64;
      continue;
    }
    q += uint64_t(__ffsll(static_cast<long long>(apart)) - 1);
    st = ends[q++];
    while (q < q_end) {
      // meeting the starts there, the rest of q is the run recorded for it:
      // the speculative one if that met, else the one that ends[q] ends
      if (walk_subchunks(col, dtype, n, thr, max_len, q, q + 1, st, win, bitmap, forced, inside)) {
        st = met[q] ? states[q_end - 1] : ends[q];
        if (met[q++]) break;
      } else {
        ++q;
      }
    }
  }
  if (threadIdx.x == 0) seg_states[blockIdx.x] = st;
}

// Fix-up across segments: one wavefront walks each segment from the true
// state the previous segment ends in, until it meets the starts already
// there (from then on the segment's run, and its end state, are right).
__global__ __launch_bounds__(64) void k_split_join(const uint8_t* __restrict__ col,
                                                   uint32_t dtype, uint64_t n, double thr,
                                                   uint64_t max_len,
                                                   unsigned long long* __restrict__ bitmap,
                                                   const SplitState* __restrict__ seg_states,
                                                   uint64_t nseg, const uint64_t* __restrict__ forced,
                                                   const uint64_t* __restrict__ inside) {
  __shared__ uint64_t win[kSplitWindow + 1];
  constexpr uint64_t kSubs = uint64_t(1) << (kSegLog2 - kSubLog2);
  const uint64_t nsub = (n + (uint64_t(1) << kSubLog2) - 1) >> kSubLog2;
  SplitState st = seg_states[0];
  for (uint64_t g = 1; g < nseg; ++g) {
    const uint64_t q0 = g * kSubs, q_end = q0 + kSubs < nsub ? q0 + kSubs : nsub;
    if (walk_subchunks(col, dtype, n, thr, max_len, q0, q_end, st, win, bitmap, forced, inside))
      st = seg_states[g];
  }
}

// ---- starting partitions ---------------------------------------------------------
//
// Second-order deltas dd_k = v_k - 2 v_{k-1} + v_{k-2} (k >= 2, exact in
// 128 bits, |dd| < 2^66).  Positions whose |dd| is the column's smallest
// are good; a maximal run k..k' of them is the starting partition
// v[k-2, k'+1), and of two that would share a value the later keeps it
// (section 3.2.2, selecting good starting positions, for a degree-1 model).

typedef unsigned __int128 u128_t;

__device__ inline u128_t dd_magnitude(const uint8_t* col, uint32_t dtype, uint64_t k) {
  const __int128 a = __int128(load_value(col, dtype, k));
  const __int128 b = __int128(load_value(col, dtype, k - 1));
  const __int128 c = __int128(load_value(col, dtype, k - 2));
  const __int128 dd = a - 2 * b + c;
  return dd < 0 ? u128_t(-dd) : u128_t(dd);
}

__device__ inline u128_t wave_min_u128(u128_t x) {
  for (int off = 32; off > 0; off >>= 1) {
    const uint64_t lo = uint64_t(__shfl_xor(static_cast<unsigned long long>(uint64_t(x)), off, 64));
    const uint64_t hi =
        uint64_t(__shfl_xor(static_cast<unsigned long long>(uint64_t(x >> 64)), off, 64));
    const u128_t y = (u128_t(hi) << 64) | lo;
    x = y < x ? y : x;
  }
  return x;
}

// partial[block] = the smallest |dd_k| over the block's grid-stride share of
// k = 2 .. n-1 (all ones when it has none), as (low, high) words.
__global__ __launch_bounds__(kScanBlock) void k_dd_min(const uint8_t* __restrict__ col,
                                                      uint32_t dtype, uint64_t n,
                                                      uint64_t* __restrict__ partial) {
  __shared__ uint64_t red[kScanBlock / 64][2];
  u128_t best = ~u128_t(0);
  for (uint64_t k = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x + 2; k < n;
       k += uint64_t(gridDim.x) * blockDim.x) {
    const u128_t x = dd_magnitude(col, dtype, k);
    best = x < best ? x : best;
  }
  best = wave_min_u128(best);
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
    red[wave][0] = uint64_t(best);
    red[wave][1] = uint64_t(best >> 64);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (uint32_t w = 1; w < kScanBlock / 64; ++w) {
      const u128_t y = (u128_t(red[w][1]) << 64) | red[w][0];
      best = y < best ? y : best;
    }
    partial[2 * blockIdx.x] = uint64_t(best);
    partial[2 * blockIdx.x + 1] = uint64_t(best >> 64);
  }
}

// out[0..1] = the smallest of `count` partial minima (one wavefront).
__global__ __launch_bounds__(64) void k_dd_min_final(const uint64_t* __restrict__ partial,
                                                    uint64_t count, uint64_t* __restrict__ out) {
  u128_t best = ~u128_t(0);
  for (uint64_t i = threadIdx.x; i < count; i += 64) {
    const u128_t y = (u128_t(partial[2 * i + 1]) << 64) | partial[2 * i];
    best = y < best ? y : best;
  }
  best = wave_min_u128(best);
  if (threadIdx.x == 0) {
    out[0] = uint64_t(best);
    out[1] = uint64_t(best >> 64);
  }
}

// good(k): k >= 2 and |dd_k| is the smallest.
__device__ inline bool dd_good(const uint8_t* col, uint32_t dtype, uint64_t n, uint64_t k,
                               u128_t best) {
  return k >= 2 && k < n && dd_magnitude(col, dtype, k) == best;
}

// first[w] bit l: value p = 64 w + l begins a starting partition (p + 2 is
// good, p + 1 is not); inside[w] bit l: p is a later value of one (p or
// p + 1 is good, and p does not begin one).  One lane per value; the
// wavefront's ballots are the words.
__global__ __launch_bounds__(kScanBlock) void k_mark_starting(const uint8_t* __restrict__ col,
                                                             uint32_t dtype, uint64_t n,
                                                             const uint64_t* __restrict__ best_dd,
                                                             uint64_t* __restrict__ first,
                                                             uint64_t* __restrict__ inside) {
  const u128_t best = (u128_t(best_dd[1]) << 64) | best_dd[0];
  const uint64_t nwords = (n + 63) / 64;
  for (uint64_t p0 = (uint64_t(blockIdx.x) * blockDim.x + (threadIdx.x & ~63u));
       p0 < nwords * 64; p0 += uint64_t(gridDim.x) * blockDim.x) {
    const uint64_t p = p0 + (threadIdx.x & 63);
    bool begins = false, in = false;
    if (p < n) {
      const bool g0 = dd_good(col, dtype, n, p, best);
      const bool g1 = dd_good(col, dtype, n, p + 1, best);
      const bool g2 = dd_good(col, dtype, n, p + 2, best);
      begins = g2 && !g1;
      in = !begins && (g0 || g1);
    }
    const uint64_t wb = __ballot(begins), wi = __ballot(in);
    if ((threadIdx.x & 63) == 0) {
      first[p0 >> 6] = wb;
      inside[p0 >> 6] = wi;
    }
  }
}

// ---- block-wide scan of counts -------------------------------------------------

// Exclusive prefix sum of x over the workgroup's threads; *total receives
// the workgroup sum.
__device__ inline uint32_t block_exclusive_scan(uint32_t x, uint32_t* total) {
  __shared__ uint32_t wsum[kScanBlock / 64];
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t inc = x;
#pragma unroll
  for (int delta = 1; delta < 64; delta <<= 1) {
    const uint32_t y = uint32_t(__shfl_up(int(inc), delta, 64));
    if (int(lane) >= delta) inc += y;
  }
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (uint32_t w = 0; w < kScanBlock / 64; ++w) {
    if (w < wave) before += wsum[w];
    all += wsum[w];
  }
  __syncthreads();
  *total = all;
  return before + inc - x;
}

// Set bits of bitmap words [blockIdx * 1024, +1024).
__global__ __launch_bounds__(kScanBlock) void k_bitmap_count(const uint64_t* __restrict__ bitmap,
                                                             uint64_t nwords,
                                                             uint64_t* __restrict__ counts) {
  const uint64_t w0 = uint64_t(blockIdx.x) * kItemsPerBlock + threadIdx.x * 4;
  uint32_t c = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (w0 + k < nwords) c += uint32_t(__popcll(bitmap[w0 + k]));
  uint32_t total;
  block_exclusive_scan(c, &total);
  if (threadIdx.x == 0) counts[blockIdx.x] = total;
}

// Writes the positions of the set bits, in order, from starts[offsets[block]].
__global__ __launch_bounds__(kScanBlock) void k_bitmap_emit(const uint64_t* __restrict__ bitmap,
                                                            uint64_t nwords,
                                                            const uint64_t* __restrict__ offsets,
                                                            uint64_t* __restrict__ starts) {
  const uint64_t w0 = uint64_t(blockIdx.x) * kItemsPerBlock + threadIdx.x * 4;
  uint64_t words[4];
  uint32_t c = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    words[k] = w0 + k < nwords ? bitmap[w0 + k] : 0;
    c += uint32_t(__popcll(words[k]));
  }
  uint32_t total;
  uint64_t out = offsets[blockIdx.x] + block_exclusive_scan(c, &total);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    uint64_t w = words[k];
    while (w) {
      const int bit = __ffsll(static_cast<long long>(w)) - 1;
      starts[out++] = (w0 + k) * 64 + uint64_t(bit);
      w &= w - 1;
    }
  }
}

// ---- sizes -----------------------------------------------------------------------

struct FitShared {
  uint64_t red[kEncWaves][4];
  double theta1;
};

// Value summary of a range of the column: smallest and largest value, and
// the sums of v and of t * v (t counted from the range's first position)
// modulo 2^128: the least-squares slope needs no more (N is the same for
// shifted values, and exact because |N| < 2^121).
struct RangeSum {
  uint64_t vmin, vmax;
  U128 sy, sty;
};

// Bytes that the partition v[s, e) costs in a variable-length blob: its
// 32-byte record, its 8-byte start and its residual words, with the model
// the encoder would choose; sum receives its summary.  Called by every
// thread of the workgroup.  Each pass issues the loads of kLongLoads values
// per thread together (a loop of one load per step waited for memory every
// 256 values).
constexpr uint32_t kLongLoads = 8;

__device__ uint64_t range_cost(FitShared& sh, const uint8_t* col, uint32_t dtype, uint64_t s,
                               uint64_t e, RangeSum& sum) {
  const uint64_t len = e - s;
  const uint8_t* src = col + s * dtype;
  uint64_t vmin = ~uint64_t(0), vmax = 0;
  U128 sv{0, 0}, stv{0, 0};
  for (uint64_t t0 = threadIdx.x; t0 < len; t0 += kEncBlock * kLongLoads) {
    uint64_t x[kLongLoads];
#pragma unroll
    for (uint32_t k = 0; k < kLongLoads; ++k) {
      const uint64_t t = t0 + k * kEncBlock;
      x[k] = load_value(src, dtype, t < len ? t : len - 1);
    }
#pragma unroll
    for (uint32_t k = 0; k < kLongLoads; ++k) {
      const uint64_t t = t0 + k * kEncBlock;
      if (t < len) {
        vmin = x[k] < vmin ? x[k] : vmin;
        vmax = x[k] > vmax ? x[k] : vmax;
        sv = add128(sv, U128{x[k], 0});
        stv = add128(stv, mul64x64(t, x[k]));
      }
    }
  }
  block_minmax_u64(sh, vmin, vmax);
  block_sum_u128x2(sh, sv, stv);
  sum = RangeSum{vmin, vmax, sv, stv};
  const uint64_t range = vmax - vmin;
  Model md{vmin, vmin, 0.0, bitlen64(range), false, 0, range};
  if (len > 1 && range < (uint64_t(1) << 61)) {
    const double th = block_slope(sh, len, sv, stv);
    int64_t rmin = INT64_MAX, rmax = INT64_MIN;
    for (uint64_t t0 = threadIdx.x; t0 < len; t0 += kEncBlock * kLongLoads) {
      uint64_t x[kLongLoads];
#pragma unroll
      for (uint32_t k = 0; k < kLongLoads; ++k) {
        const uint64_t t = t0 + k * kEncBlock;
        x[k] = load_value(src, dtype, t < len ? t : len - 1);
      }
#pragma unroll
      for (uint32_t k = 0; k < kLongLoads; ++k) {
        const uint64_t t = t0 + k * kEncBlock;
        if (t < len) {
          const int64_t rr = int64_t(x[k] - vmin) - predict(th, uint32_t(t));
          rmin = rr < rmin ? rr : rmin;
          rmax = rr > rmax ? rr : rmax;
        }
      }
    }
    block_minmax_i64(sh, rmin, rmax);
    choose_model(md, th, rmin, rmax);
  }
  return kRecordBytes + 8 + 8 * ((len * md.bits + 63) >> 6);
}

// Ranges up to kLaneRangeMax values are sized by one lane, up to
// kWaveRangeMax by one wavefront, longer ones by a whole workgroup.
constexpr uint64_t kLaneRangeMax = 32;
constexpr uint64_t kWaveRangeMax = 8192;

// range_cost computed by one lane alone.
__device__ uint64_t range_cost_lane(const uint8_t* col, uint32_t dtype, uint64_t s, uint64_t e,
                                    RangeSum& sum) {
  const uint64_t len = e - s;
  const uint8_t* src = col + s * dtype;
  uint64_t vmin = ~uint64_t(0), vmax = 0;
  U128 sv{0, 0}, stv{0, 0};
  for (uint64_t t = 0; t < len; ++t) {
    const uint64_t x = load_value(src, dtype, t);
    vmin = x < vmin ? x : vmin;
    vmax = x > vmax ? x : vmax;
    sv = add128(sv, U128{x, 0});
    stv = add128(stv, mul64x64(t, x));
  }
  sum = RangeSum{vmin, vmax, sv, stv};
  const uint64_t range = vmax - vmin;
  Model md{vmin, vmin, 0.0, bitlen64(range), false, 0, range};
  if (len > 1 && range < (uint64_t(1) << 61)) {
    const double th = ls_slope(len, sv, stv);
    int64_t rmin = INT64_MAX, rmax = INT64_MIN;
    for (uint64_t t = 0; t < len; ++t) {
      const int64_t rr = int64_t(load_value(src, dtype, t) - vmin) - predict(th, uint32_t(t));
      rmin = rr < rmin ? rr : rmin;
      rmax = rr > rmax ? rr : rmax;
    }
    choose_model(md, th, rmin, rmax);
  }
  return kRecordBytes + 8 + 8 * ((len * md.bits + 63) >> 6);
}

// The ranges of at most kLaneRangeMax values (and the ones too long to
// merge): one lane each.
__global__ __launch_bounds__(kEncBlock) void k_costs_short(const uint8_t* __restrict__ col,
                                                           uint32_t dtype,
                                                           const uint64_t* __restrict__ starts,
                                                           uint64_t count, uint32_t span,
                                                           uint64_t max_len,
                                                           const uint8_t* __restrict__ dirty,
                                                           uint64_t* __restrict__ out,
                                                           RangeSum* __restrict__ sums) {
  const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
  for (uint64_t j = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; j < count; j += stride) {
    if (dirty && !dirty[j]) continue;
    const uint64_t s = starts[j], e = starts[j + span];
    if (e - s > max_len) {
      out[j] = kNoMerge;
    } else if (e - s <= kLaneRangeMax) {
      RangeSum sum;
      out[j] = range_cost_lane(col, dtype, s, e, sum);
      if (sums) sums[j] = sum;
    }
  }
}

// range_cost computed by one wavefront alone (no workgroup barrier), the
// same arithmetic in the same order of operations where it matters: the
// sums are exact and the slope is one function of them.
//
// Ranges of at most 64 kCostRegs values are held in registers: every load
// is issued before any is used and the residual pass reads the registers
// (a loop of dependent loads per pass made the wavefront wait once per 64
// values, twice).  The sums are exact, so their order does not matter.
constexpr int kCostRegs = 8;

template <class T>
__device__ uint64_t range_cost_wave_regs(const T* src, uint64_t len, RangeSum& sum) {
  const uint32_t lane = threadIdx.x & 63;
  const auto g = global_ptr(src);
  uint64_t x[kCostRegs];
#pragma unroll
  for (int k = 0; k < kCostRegs; ++k) {
    const uint32_t t = lane + 64u * k;
    x[k] = uint64_t(g[t < len ? t : len - 1]);
  }
  uint64_t vmin = ~uint64_t(0), vmax = 0;
  U128 sv{0, 0}, stv{0, 0};
#pragma unroll
  for (int k = 0; k < kCostRegs; ++k) {
    const uint32_t t = lane + 64u * k;
    if (t < len) {
      vmin = x[k] < vmin ? x[k] : vmin;
      vmax = x[k] > vmax ? x[k] : vmax;
      sv = add128(sv, U128{x[k], 0});
      stv = add128(stv, mul64x64(t, x[k]));
    }
  }
  wave_minmax_u64(vmin, vmax);
  wave_sum_u128x2(sv, stv);
  sum = RangeSum{vmin, vmax, sv, stv};
  const uint64_t range = vmax - vmin;
  Model md{vmin, vmin, 0.0, bitlen64(range), false, 0, range};
  if (len > 1 && range < (uint64_t(1) << 61)) {
    const double th = ls_slope(len, sv, stv);
    int64_t rmin = INT64_MAX, rmax = INT64_MIN;
#pragma unroll
    for (int k = 0; k < kCostRegs; ++k) {
      const uint32_t t = lane + 64u * k;
      if (t < len) {
        const int64_t rr = int64_t(x[k] - vmin) - predict(th, t);
        rmin = rr < rmin ? rr : rmin;
        rmax = rr > rmax ? rr : rmax;
      }
    }
    wave_minmax_i64(rmin, rmax);
    choose_model(md, th, rmin, rmax);
  }
  return kRecordBytes + 8 + 8 * ((len * md.bits + 63) >> 6);
}

__device__ uint64_t range_cost_wave(const uint8_t* col, uint32_t dtype, uint64_t s, uint64_t e,
                                    RangeSum& sum) {
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t len = e - s;
  const uint8_t* src = col + s * dtype;
  if (len <= 64u * kCostRegs)
    return dtype == 8 ? range_cost_wave_regs(reinterpret_cast<const uint64_t*>(src), len, sum)
                      : range_cost_wave_regs(reinterpret_cast<const uint32_t*>(src), len, sum);
  // longer ranges in blocks of 64 kCostRegs values, each block's loads
  // issued together (indices clamped, the extra lanes masked)
  uint64_t vmin = ~uint64_t(0), vmax = 0;
  U128 sv{0, 0}, stv{0, 0};
  for (uint64_t t0 = 0; t0 < len; t0 += 64u * kCostRegs) {
    uint64_t x[kCostRegs];
#pragma unroll
    for (int k = 0; k < kCostRegs; ++k) {
      const uint64_t t = t0 + lane + 64u * k;
      x[k] = load_value(src, dtype, t < len ? t : len - 1);
    }
#pragma unroll
    for (int k = 0; k < kCostRegs; ++k) {
      const uint64_t t = t0 + lane + 64u * k;
      if (t < len) {
        vmin = x[k] < vmin ? x[k] : vmin;
        vmax = x[k] > vmax ? x[k] : vmax;
        sv = add128(sv, U128{x[k], 0});
        stv = add128(stv, mul64x64(t, x[k]));
      }
    }
  }
  wave_minmax_u64(vmin, vmax);
  wave_sum_u128x2(sv, stv);
  sum = RangeSum{vmin, vmax, sv, stv};
  const uint64_t range = vmax - vmin;
  Model md{vmin, vmin, 0.0, bitlen64(range), false, 0, range};
  if (len > 1 && range < (uint64_t(1) << 61)) {
    const double th = ls_slope(len, sv, stv);
    int64_t rmin = INT64_MAX, rmax = INT64_MIN;
    for (uint64_t t0 = 0; t0 < len; t0 += 64u * kCostRegs) {
      uint64_t x[kCostRegs];
#pragma unroll
      for (int k = 0; k < kCostRegs; ++k) {
        const uint64_t t = t0 + lane + 64u * k;
        x[k] = load_value(src, dtype, t < len ? t : len - 1);
      }
#pragma unroll
      for (int k = 0; k < kCostRegs; ++k) {
        const uint64_t t = t0 + lane + 64u * k;
        if (t < len) {
          const int64_t rr = int64_t(x[k] - vmin) - predict(th, uint32_t(t));
          rmin = rr < rmin ? rr : rmin;
          rmax = rr > rmax ? rr : rmax;
        }
      }
    }
    wave_minmax_i64(rmin, rmax);
    choose_model(md, th, rmin, rmax);
  }
  return kRecordBytes + 8 + 8 * ((len * md.bits + 63) >> 6);
}

// Ranges are screened `chunk` (at most kCostChunk) at a time: the chunk's
// lanes read their dirty flag and bounds together (one round trip), and the
// wavefront or workgroup then sizes the chunk's ranges of its class one
// after another.  (Walking one range per iteration made every idle launch
// cost a chain of dependent loads per range.)  The host picks the chunk so
// that there are at least as many chunks as resident wavefronts or
// workgroups: few, long ranges still get one each.
constexpr uint32_t kCostChunk = 64;

// Bounds of range j0 + lane for lanes below kCostChunk; true if it needs
// sizing by the caller's class [lo_len, hi_len] (and is within max_len).
__device__ inline bool cost_candidate(const uint64_t* starts, uint64_t count, uint32_t span,
                                      uint64_t max_len, const uint8_t* dirty, uint64_t j,
                                      uint64_t lo_len, uint64_t hi_len) {
  if (j >= count) return false;
  // the flag and both bounds in one round trip
  const bool d = !dirty || dirty[j];
  const uint64_t len = starts[j + span] - starts[j];
  return d && len <= max_len && len > lo_len && len <= hi_len;
}

// out[j] = cost of v[starts[j], starts[j + span]) for j < count (only
// where dirty[j], if dirty is given), or kNoMerge when that is longer than
// max_len, and sums[j] (if given) its summary: one wavefront per range of more than kLaneRangeMax and at most
// kWaveRangeMax values; the others are left to k_costs_short and
// k_costs_long.
__global__ __launch_bounds__(kEncBlock) void k_costs(const uint8_t* __restrict__ col,
                                                     uint32_t dtype,
                                                     const uint64_t* __restrict__ starts,
                                                     uint64_t count, uint32_t span,
                                                     uint64_t max_len,
                                                     const uint8_t* __restrict__ dirty,
                                                     uint64_t* __restrict__ out,
                                                     RangeSum* __restrict__ sums, uint32_t chunk) {
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t waves = uint64_t(gridDim.x) * kEncWaves;
  for (uint64_t j0 = (uint64_t(blockIdx.x) * kEncWaves + (threadIdx.x >> 6)) * chunk;
       j0 < count; j0 += waves * chunk) {
    const bool mine = lane < chunk &&
                      cost_candidate(starts, count, span, max_len, dirty, j0 + lane,
                                     kLaneRangeMax, kWaveRangeMax);
    uint64_t todo = __ballot(mine);
    while (todo) {
      const uint64_t j = j0 + uint64_t(__ffsll(static_cast<long long>(todo)) - 1);
      todo &= todo - 1;
      RangeSum sum;
      const uint64_t c = range_cost_wave(col, dtype, starts[j], starts[j + span], sum);
      if (lane == 0) {
        out[j] = c;
        if (sums) sums[j] = sum;
      }
    }
  }
}

// The ranges k_costs left: one workgroup each.
__global__ __launch_bounds__(kEncBlock) void k_costs_long(const uint8_t* __restrict__ col,
                                                          uint32_t dtype,
                                                          const uint64_t* __restrict__ starts,
                                                          uint64_t count, uint32_t span,
                                                          uint64_t max_len,
                                                          const uint8_t* __restrict__ dirty,
                                                          uint64_t* __restrict__ out,
                                                          RangeSum* __restrict__ sums,
                                                          uint32_t chunk) {
  __shared__ FitShared sh;
  __shared__ uint64_t todo_sh;
  for (uint64_t j0 = uint64_t(blockIdx.x) * chunk; j0 < count;
       j0 += uint64_t(gridDim.x) * chunk) {
    if (threadIdx.x < 64) {
      const bool mine =
          threadIdx.x < chunk && cost_candidate(starts, count, span, max_len, dirty,
                                                     j0 + threadIdx.x, kWaveRangeMax, max_len);
      const uint64_t b = __ballot(mine);
      if (threadIdx.x == 0) todo_sh = b;
    }
    __syncthreads();
    uint64_t todo = todo_sh;
    while (todo) {
      const uint64_t j = j0 + uint64_t(__ffsll(static_cast<long long>(todo)) - 1);
      todo &= todo - 1;
      RangeSum sum;
      const uint64_t c = range_cost(sh, col, dtype, starts[j], starts[j + span], sum);
      if (threadIdx.x == 0) {
        out[j] = c;
        if (sums) sums[j] = sum;
      }
    }
    __syncthreads();  // todo_sh is rewritten by the next chunk
  }
}

// ---- merge scan -------------------------------------------------------------------
//
// Boundary k (1 <= k < m) is the start of partition k.  Step k of a pass
// tries to merge the current partition, which begins at boundary a (a < k)
// and costs cc bytes, with partition k:
//   union = pair[k - 1] when a = k - 1 (two unmerged partitions, sized in
//           advance), else the size of v[s[a], s[k+1]) fitted now; none
//           when longer than max_len;
//   merge when union < cc + cost[k]: the current partition grows (cc =
//   union); else boundary k is kept, and partition k is the current one
//   (a = k, cc = cost[k]).
// The pass keeps a bitmap of kept boundaries (bit 0 always set); the
// partitions that absorbed others are sized once the pass is done.

__device__ inline uint64_t shfl_up64(uint64_t x, int d) {
  return uint64_t(__shfl_up(static_cast<unsigned long long>(x), d, 64));
}

// The summary of [x, z) from those of [x, y) and [y, z).
__device__ inline RangeSum join(const RangeSum& a, const RangeSum& b, uint64_t a_len) {
  RangeSum r;
  r.vmin = a.vmin < b.vmin ? a.vmin : b.vmin;
  r.vmax = a.vmax > b.vmax ? a.vmax : b.vmax;
  r.sy = add128(a.sy, b.sy);
  r.sty = add128(add128(a.sty, b.sty), mul128x64(b.sy, a_len));
  return r;
}

struct MergeState {
  uint64_t a;   // boundary where the current partition begins
  uint64_t cc;  // its size in bytes
  RangeSum sum; // its values' summary
};

// Convex hulls of the current partition's points (t, v_t), t counted from
// its first value: the upper hull (left to right, right turns only) and the
// lower one.  Over any set of points, v_t - theta1 * t is largest at an
// upper-hull vertex and smallest at a lower-hull vertex, whatever theta1;
// so is the exact residual v_t - floor(theta1 * t), the ceiling of that real
// number.  The encoder's residual takes the binary64 product, whose floor
// exceeds the exact one by 1 exactly when the product rounds up onto an
// integer (hull_ranges checks for that).  A long run of merges then sizes
// each union from the hulls, not from its values.
//
// Vertices per hull: sorted normal samples, one partition of 500,000 of which
// merges with 900 short ones behind it, have 65 to 128.  Without hulls each of
// those merges scans the whole of it: 89 ms at 64, 24 now.
constexpr uint32_t kHullMax = 128;
constexpr uint64_t kHullBuildMin = 128;        // shorter partitions are scanned whole
constexpr uint64_t kHullBuildNow = 2048;       // longer ones get hulls after kSoloMerges merges
constexpr uint32_t kSoloMerges = 8;            // (a build costs about what 16 whole scans do)
constexpr uint64_t kBatchNew = 1024;           // values a batch may add
constexpr uint64_t kReachMin = 64, kReachMax = 512;  // and without hulls, at least (reach)
constexpr uint64_t kSoloMin = 256;             // longer neighbours: sized alone without hulls
constexpr uint64_t kHullAppendMax = 8192;      // and longer than this with them
constexpr uint64_t kDeadScanMax = 16384;       // longest partition a batch scans whole without hulls
constexpr uint64_t kWide = uint64_t(1) << 61;  // value spread beyond which no line is fitted
enum : uint32_t { kHullNone = 0, kHullValid = 1, kHullDead = 2 };

struct ChainHull {  // side 0: upper, side 1: lower
  uint32_t n[2], state, pad;
  uint32_t t[2][kHullMax + 1];  // one entry of padding for the searches
  uint64_t x[2][kHullMax + 1];
};

constexpr uint32_t kWalk = 256;                // threads of a walker, steps of a batch
constexpr uint32_t kWalkWaves = kWalk / 64;
constexpr uint32_t kPeelCap = 640;             // points of a hull under construction
static_assert(kHullMax + kWalk <= kPeelCap, "a block fits behind a hull");
constexpr uint32_t kStageVals = 1024;          // values staged with a window, when no more
static_assert(kWalk == uint32_t(kEncBlock), "workgroup reductions");

// A walker's LDS (one workgroup): the current partition's hulls and those of
// the batch's longest union, the point lists they are built from, and the
// sizes, summaries and values of the next kWalk partitions, loaded together
// so that a batch waits for memory once per window.
struct WalkLds {
  ChainHull h[2];
  uint32_t lt[2][2][kPeelCap];
  uint64_t lx[2][2][kPeelCap];
  uint64_t s[kWalk + 1], cost[kWalk], size[kWalk];
  RangeSum psum[kWalk];
  uint64_t vals[kStageVals];
  double scan[kWalk];
  RangeSum wave_sum[kWalkWaves];
  uint64_t mask[3][kWalkWaves];
  uint32_t count[2][kWalkWaves];  // survivors of each wavefront's block, per side
  uint32_t n[2], cur[2];
  StripShared strip;
  uint64_t red[kEncWaves][4];     // workgroup reductions of fit.hpp
};

// The hulls' counts and state, identical in every thread of the walker.
struct HullRegs {
  uint32_t n[2], state;
};

__device__ inline void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ inline uint32_t lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi(uint32_t(mask >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(mask), 0));
}

// Sign of (b - a) x (c - a) for points with ta < tb < tc whose values lie
// within 2^61 of each other.  kW = 64: within 2^42, so that with t <= 2^20
// each product fits in 64 bits; kW = 32: within 2^31, so that each factor
// fits in 32 bits as well (one 32 x 32 -> 64 multiply).
template <int kW = 128>
__device__ inline int turn(uint32_t ta, uint64_t xa, uint32_t tb, uint64_t xb, uint32_t tc,
                           uint64_t xc) {
  if (kW == 32) {
    const int64_t l = int64_t(int32_t(tb - ta)) * int64_t(int32_t(uint32_t(xc - xa)));
    const int64_t r = int64_t(int32_t(uint32_t(xb - xa))) * int64_t(int32_t(tc - ta));
    return l > r ? 1 : (l < r ? -1 : 0);
  }
  if (kW == 64) {
    const int64_t l = int64_t(tb - ta) * int64_t(xc - xa);
    const int64_t r = int64_t(xb - xa) * int64_t(tc - ta);
    return l > r ? 1 : (l < r ? -1 : 0);
  }
  const __int128 l = __int128(int64_t(tb - ta)) * __int128(int64_t(xc - xa));
  const __int128 r = __int128(int64_t(xb - xa)) * __int128(int64_t(tc - ta));
  return l > r ? 1 : (l < r ? -1 : 0);
}

// Drops points from the list of `side` (n points in buffer cur) until it is
// a convex chain, by one wavefront.  A point on or below (upper hull; on or
// above, lower) the chord of two others of the list on either side of it is
// no vertex; a round tests every point against its neighbours 1, 2 and 4
// places away at once, and a list that a round leaves alone has only strict
// turns: it is the hull.  About five rounds on noise.
template <int kW>
__device__ __attribute__((always_inline)) inline void peel(WalkLds& w, uint32_t side, uint32_t& n,
                                                           uint32_t& cur) {
  const uint32_t lane = threadIdx.x & 63;
  while (n > 2) {
    const uint32_t* T = w.lt[side][cur];
    const uint64_t* X = w.lx[side][cur];
    uint32_t* T2 = w.lt[side][cur ^ 1];
    uint64_t* X2 = w.lx[side][cur ^ 1];
    uint32_t out = 0;
    for (uint32_t i0 = 0; i0 < n; i0 += 64) {
      const uint32_t i = i0 + lane;
      bool stays = i < n;
      const uint32_t ic = stays ? i : n - 1;
      // every neighbour loaded at once, out of range ones as the point itself
      uint32_t ta[3], tc[3];
      uint64_t xa[3], xc[3];
      const uint32_t t = T[ic];
      const uint64_t x = X[ic];
#pragma unroll
      for (uint32_t q = 0; q < 3; ++q) {
        const uint32_t d = 1u << q;
        const bool in = ic >= d && ic + d < n;
        const uint32_t ia = in ? ic - d : ic, io = in ? ic + d : ic;
        ta[q] = T[ia];
        xa[q] = X[ia];
        tc[q] = T[io];
        xc[q] = X[io];
      }
#pragma unroll
      for (uint32_t q = 0; q < 3; ++q) {
        const int tr = turn<kW>(ta[q], xa[q], t, x, tc[q], xc[q]);
        if (ta[q] != t && (side ? tr <= 0 : tr >= 0)) stays = false;
      }
      const uint64_t mask = __ballot(stays);
      if (stays) {
        const uint32_t o = out + lanes_below(mask);
        T2[o] = t;
        X2[o] = x;
      }
      out += uint32_t(__popcll(mask));
    }
    wave_lds_order();
    cur ^= 1;
    if (out == n) break;
    n = out;
  }
}

// Hull h[to] = hull h[from] (counts in hr; empty when hr is not valid) with
// the points [u0, u1) of the partition beginning at column position sa
// added, all later than its own.  read(t) is the value at position t < u1.
// Each wavefront takes a block of 64 points and tests them against chords of
// points at equal distances 1, 2 .. 16 on either side (about a quarter
// stay); wavefronts 0 and 1 peel the upper and the lower list.  Returns the
// counts; kHullDead when a hull has over kHullMax vertices.  Called by the
// whole workgroup.
template <int kW, class Read>
__device__ __attribute__((always_inline)) inline HullRegs hull_extend_t(WalkLds& w, uint32_t from,
                                                                        uint32_t to,
                                                                        const HullRegs& hr,
                                                                        uint64_t u0, uint64_t u1,
                                                                        const Read& read) {
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t n[2] = {0, 0}, cur[2] = {0, 0};
  if (hr.state == kHullValid) {
#pragma unroll
    for (uint32_t side = 0; side < 2; ++side) {
      n[side] = hr.n[side];
      if (threadIdx.x < n[side]) {
        w.lt[side][0][threadIdx.x] = w.h[from].t[side][threadIdx.x];
        w.lx[side][0][threadIdx.x] = w.h[from].x[side][threadIdx.x];
      }
    }
  }
  bool dead = false;
  for (uint64_t b0 = u0; b0 < u1; b0 += kWalk) {
    const uint64_t t = b0 + threadIdx.x;
    const bool in = t < u1;
    const uint64_t tc = in ? t : u1 - 1;
    const uint64_t x = read(tc);
    // all chord ends loaded at once, out of range ones as the point itself
    uint64_t xa[5], xb[5];
#pragma unroll
    for (uint32_t q = 0; q < 5; ++q) {
      const uint32_t d = 1u << q;
      const bool both = tc >= d && tc + d < u1;
      xa[q] = read(both ? tc - d : tc);
      xb[q] = read(both ? tc + d : tc);
    }
    bool up = in, low = in;
#pragma unroll
    for (uint32_t q = 0; q < 5; ++q) {
      const uint32_t d = 1u << q;
      const int tr = turn<kW>(0, xa[q], d, x, 2 * d, xb[q]);
      const bool both = tc >= d && tc + d < u1;
      if (both && tr >= 0) up = false;
      if (both && tr <= 0) low = false;
    }
    const uint64_t mu = __ballot(up), ml = __ballot(low);
    if (lane == 0) {
      w.count[0][wave] = uint32_t(__popcll(mu));
      w.count[1][wave] = uint32_t(__popcll(ml));
    }
    __syncthreads();
    uint32_t before[2] = {0, 0}, total[2] = {0, 0};
#pragma unroll
    for (uint32_t v = 0; v < kWalkWaves; ++v) {
#pragma unroll
      for (uint32_t side = 0; side < 2; ++side) {
        const uint32_t c = w.count[side][v];
        if (v < wave) before[side] += c;
        total[side] += c;
      }
    }
    if (up) {
      const uint32_t o = n[0] + before[0] + lanes_below(mu);
      w.lt[0][cur[0]][o] = uint32_t(t);
      w.lx[0][cur[0]][o] = x;
    }
    if (low) {
      const uint32_t o = n[1] + before[1] + lanes_below(ml);
      w.lt[1][cur[1]][o] = uint32_t(t);
      w.lx[1][cur[1]][o] = x;
    }
    n[0] += total[0];
    n[1] += total[1];
    __syncthreads();
    // peeled at the end, and whenever the next blocks might not fit
    if (b0 + kWalk >= u1 || n[0] > kPeelCap - kWalk || n[1] > kPeelCap - kWalk) {
      if (wave < 2) {
        uint32_t c = wave ? n[1] : n[0], buf = wave ? cur[1] : cur[0];
        peel<kW>(w, wave, c, buf);
        if (lane == 0) {
          w.n[wave] = c;
          w.cur[wave] = buf;
        }
      }
      __syncthreads();
#pragma unroll
      for (uint32_t side = 0; side < 2; ++side) {
        n[side] = w.n[side];
        cur[side] = w.cur[side];
      }
      dead = n[0] > kPeelCap - kWalk || n[1] > kPeelCap - kWalk;
      if (dead) break;
    }
  }
  __syncthreads();  // every thread has read w.n
  if (dead || n[0] > kHullMax || n[1] > kHullMax) return HullRegs{{0, 0}, kHullDead};
#pragma unroll
  for (uint32_t side = 0; side < 2; ++side) {
    if (threadIdx.x < n[side]) {
      w.h[to].t[side][threadIdx.x] = w.lt[side][cur[side]][threadIdx.x];
      w.h[to].x[side][threadIdx.x] = w.lx[side][cur[side]][threadIdx.x];
    }
  }
  __syncthreads();  // the vertices are read by every thread next
  return HullRegs{{n[0], n[1]}, kHullValid};
}

// Values spread below 2^31 take the 32-bit turn test, below 2^42 the 64-bit one.
template <class Read>
__device__ __attribute__((always_inline)) inline HullRegs hull_extend(
    WalkLds& w, uint32_t from, uint32_t to, const HullRegs& hr, uint64_t u0, uint64_t u1,
    uint64_t spread, const Read& read) {
  if (spread < (uint64_t(1) << 31)) return hull_extend_t<32>(w, from, to, hr, u0, u1, read);
  if (spread < (uint64_t(1) << 42)) return hull_extend_t<64>(w, from, to, hr, u0, u1, read);
  return hull_extend_t<128>(w, from, to, hr, u0, u1, read);
}

__device__ inline void hull_store(ChainHull* __restrict__ g, const ChainHull& h, const HullRegs& hr) {
  const uint32_t i = threadIdx.x;
  if (hr.state == kHullValid) {
#pragma unroll
    for (uint32_t side = 0; side < 2; ++side) {
      if (i < hr.n[side]) {
        g->t[side][i] = h.t[side][i];
        g->x[side][i] = h.x[side][i];
      }
    }
  }
  if (i == 0) {
    g->n[0] = hr.n[0];
    g->n[1] = hr.n[1];
    g->state = hr.state;
  }
}

__device__ inline HullRegs hull_load(const ChainHull* __restrict__ g, ChainHull& h) {
  const uint32_t i = threadIdx.x;
  const HullRegs hr{{g->n[0], g->n[1]}, g->state};
  if (hr.state == kHullValid) {
#pragma unroll
    for (uint32_t side = 0; side < 2; ++side) {
      if (i < hr.n[side]) {
        h.t[side][i] = g->t[side][i];
        h.x[side][i] = g->x[side][i];
      }
    }
  }
  __syncthreads();
  return hr;
}

// The encoder's residual v - vmin - floor(fl(theta1 * t)) at a hull vertex,
// plus 1 when the binary64 product rounded up onto an integer (then the
// exact residual is one more; `up` says so).  `gap` is 1 - frac(theta1 * t)
// of the exact product, to within 2^-50, when up is false.
__device__ inline int64_t vertex_residual(double th, uint32_t t, uint64_t x, uint64_t vmin,
                                          bool& up, double& gap) {
  const double p = __dmul_rn(th, double(t));
  const double fp = floor(p);
  const double e = __fma_rn(th, double(t), -p);  // exact: theta1 * t - p
  up = fp == p && e < 0.0;
  gap = ((fp + 1.0) - p) - e;
  return int64_t(x - vmin) - int64_t(fp) + (up ? 1 : 0);
}

// Bounds of the largest and of the smallest residual the encoder would have
// over the points of a hull, for this thread's slope.
struct HullRange {
  int64_t max_lo, max_hi, min_lo, min_hi;
  __device__ uint32_t bits_lo() const {
    return max_lo > min_hi ? bitlen64(uint64_t(max_lo) - uint64_t(min_hi)) : 0;
  }
  __device__ uint32_t bits_hi() const { return bitlen64(uint64_t(max_hi) - uint64_t(min_lo)); }
  __device__ bool exact() const { return max_lo == max_hi && min_lo == min_hi; }
};

// The vertex of largest v - th t of an upper hull is the first whose next
// edge is no steeper than th (a lower hull's smallest: no flatter), found by
// binary search, the four searches side by side.  An edge (dt, dx) is
// compared with th exactly: th dt = p + e with e the product's rounding
// error, and dx - p is exact wherever it is as small as e.  Hulls 0 and 1 of
// w.h have n0 and n1 vertices; pmax bounds every |product|, below 2^31.
__device__ __attribute__((always_inline)) inline void hull_ranges(
    const WalkLds& w, const uint32_t (&n0)[2], const uint32_t (&n1)[2], double th, double pmax,
    uint64_t vmin, HullRange (&out)[2]) {
  uint32_t lo[4] = {0, 0, 0, 0};
  uint32_t hi[4] = {n0[0] - 1, n0[1] - 1, n1[0] - 1, n1[1] - 1};
  const uint32_t most = max(max(hi[0], hi[1]), max(hi[2], hi[3]));
  for (uint32_t span = most; span > 0; span >>= 1) {  // uniform: ends with every search done
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
      const ChainHull& h = w.h[q >> 1];
      const uint32_t side = q & 1, mid = (lo[q] + hi[q]) >> 1;
      const uint32_t dt = h.t[side][mid + 1] - h.t[side][mid];
      const int64_t dx = int64_t(h.x[side][mid + 1] - h.x[side][mid]);
      const double p = __dmul_rn(th, double(dt));
      const double e = __fma_rn(th, double(dt), -p);
      const double d = double(dx) - p;
      const bool right = side ? d < e : d > e;
      if (lo[q] < hi[q]) {
        if (right)
          lo[q] = mid + 1;
        else
          hi[q] = mid;
      }
    }
  }
  // The exact residuals' largest, R, is the upper vertex's and the smallest,
  // Q, the lower vertex's.  The encoder's largest is R when that product
  // does not round up, else R or R - 1.  Its smallest is Q - 1 when the lower
  // vertex's product rounds up; else Q unless another value reaching Q rounds
  // up, which needs a product within half an ulp of pmax under an integer,
  // where the vertex's own gap is at least as small (margin: two ulps of
  // pmax, at least 2^-48 against the gap's own rounding).
  const double margin = pmax >= 0x1p-3 ? fmax(ldexp(1.0, ilogb(pmax) - 51), 0x1p-48) : 0x1p-48;
#pragma unroll
  for (uint32_t b = 0; b < 2; ++b) {
    const ChainHull& h = w.h[b];
    const uint32_t iu = lo[2 * b], il = lo[2 * b + 1];
    bool up, q_up;
    double gap, q_gap;
    const int64_t R = vertex_residual(th, h.t[0][iu], h.x[0][iu], vmin, up, gap);
    const int64_t Q = vertex_residual(th, h.t[1][il], h.x[1][il], vmin, q_up, q_gap);
    out[b].max_hi = R;
    out[b].max_lo = up ? R - 1 : R;
    out[b].min_hi = q_up ? Q - 1 : Q;
    out[b].min_lo = q_up || q_gap < margin ? Q - 1 : Q;
  }
}

// Sets (clears) bits [k, k + f) of a bitmap, f <= kWalk: thread i takes the
// i-th word that the run touches.
__device__ inline void set_run(unsigned long long* bits, uint64_t k, uint64_t f) {
  const uint64_t w = (k >> 6) + threadIdx.x;
  if (f == 0 || w > (k + f - 1) >> 6) return;
  const uint64_t lo = w << 6 < k ? k & 63 : 0;
  const uint64_t end = k + f - (w << 6);
  const uint64_t mask = (end >= 64 ? ~0ull : (1ull << end) - 1) & ~((1ull << lo) - 1);
  atomicOr(bits + w, static_cast<unsigned long long>(mask));
}

__device__ inline void clear_run(unsigned long long* bits, uint64_t k, uint64_t f) {
  const uint64_t w = (k >> 6) + threadIdx.x;
  if (f == 0 || w > (k + f - 1) >> 6) return;
  const uint64_t lo = w << 6 < k ? k & 63 : 0;
  const uint64_t end = k + f - (w << 6);
  const uint64_t mask = (end >= 64 ? ~0ull : (1ull << end) - 1) & ~((1ull << lo) - 1);
  atomicAnd(bits + w, ~static_cast<unsigned long long>(mask));
}

// Residual range of v[0, len) of `src` for one slope, by the workgroup.
__device__ __attribute__((always_inline)) inline void range_scan(
    WalkLds& w, StripGroup<kEncBlock>& g, const uint8_t* src, uint32_t dtype, uint64_t len,
    uint64_t vmin, uint64_t range, double th, int64_t& rmin, int64_t& rmax) {
  constexpr uint32_t kR = 8;
  rmin = INT64_MAX;
  rmax = INT64_MIN;
  // offsets and predictions below 2^50: differences exact in binary64
  if (range < (uint64_t(1) << 32) && __dmul_rn(fabs(th), double(len)) < 0x1p50) {
    double mx = -__builtin_inf(), mn = __builtin_inf();
    for (uint64_t t0 = threadIdx.x; t0 < len; t0 += kWalk * kR) {
      uint64_t x[kR];
#pragma unroll
      for (uint32_t k = 0; k < kR; ++k) {
        const uint64_t t = t0 + kWalk * k;
        x[k] = load_value(src, dtype, t < len ? t : len - 1);
      }
#pragma unroll
      for (uint32_t k = 0; k < kR; ++k) {
        const uint64_t t = t0 + kWalk * k;
        const double tt = double(uint32_t(t < len ? t : len - 1));
        const double r = double(uint32_t(x[k] - vmin)) - floor(__dmul_rn(th, tt));
        mx = fmax(mx, r);
        mn = fmin(mn, r);
      }
    }
    g.maxmin(mx, mn);
    rmin = int64_t(mn);
    rmax = int64_t(mx);
    return;
  }
  for (uint64_t t = threadIdx.x; t < len; t += kWalk) {
    const int64_t rr = int64_t(load_value(src, dtype, t) - vmin) - predict(th, uint32_t(t));
    rmin = rr < rmin ? rr : rmin;
    rmax = rr > rmax ? rr : rmax;
  }
  block_minmax_i64(w, rmin, rmax);
}

__device__ inline uint64_t merged_size(uint64_t len, uint32_t bits) {
  return kRecordBytes + 8 + 8 * ((len * bits + 63) >> 6);
}

// First thread whose flag is set, or kWalk; which = the mask slot (a slot is
// used again only behind another slot's barrier).
__device__ inline uint32_t first_of(WalkLds& w, uint32_t which, bool flag) {
  const uint64_t mask = __ballot(flag);
  if ((threadIdx.x & 63) == 0) w.mask[which][threadIdx.x >> 6] = mask;
  __syncthreads();
  uint32_t first = kWalk;
#pragma unroll
  for (int v = int(kWalkWaves) - 1; v >= 0; --v) {
    const uint64_t m = w.mask[which][v];
    if (m) first = uint32_t(v) * 64 + uint32_t(__ffsll(static_cast<long long>(m)) - 1);
  }
  return uint32_t(__builtin_amdgcn_readfirstlane(int(first)));
}

// Runs steps [kb, ke) from state st.  kFix = false: the bitmap holds zeros
// there and the walk sets the kept bits.  kFix = true: the bits are another
// run's, made from a different state; the walk rewrites them until it keeps
// a boundary that run also kept (from there on both runs are the same) and
// returns true at that point.  w.h[cur] / hr: the current partition's hulls,
// valid when hr.state is kHullValid and a merge is pending.  Called by a
// whole workgroup; state and decisions are the same in every thread.  The
// walk only reads bits from step k on and only writes those before it.
template <bool kFix>
__device__ __attribute__((always_inline)) inline bool merge_walk(
    const uint8_t* __restrict__ col, uint32_t dtype, const uint64_t* __restrict__ s,
    const uint64_t* __restrict__ cost, const uint64_t* __restrict__ pair,
    const RangeSum* __restrict__ psum, uint64_t max_len, uint64_t kb, uint64_t ke, MergeState& st,
    unsigned long long* __restrict__ keep, WalkLds& w, HullRegs& hr, uint32_t& cur) {
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  StripGroup<kEncBlock> group{&w.strip};
  uint64_t k = kb;
  uint64_t w0 = 0, w1 = 0;  // partitions staged
  uint64_t vb = 0, ve = 0;  // values staged (column positions)
  uint64_t sa = s[st.a];
  uint32_t solo = 0;        // merges sized one at a time since the last refusal
  // Values a batch without hulls may add at least: twice as many as the longer
  // of the last two merged partitions got to hold.  Where chains end after a
  // merge or two, scans of 512 more values were most of a batch: 2e5 values in
  // clusters of 40, split around starting partitions, 6.8 ms and now 3.6.  (64
  // everywhere: merges of long lines 11% slower.)
  uint64_t reach = kReachMax, held = kReachMax / 2;
  while (k < ke) {
    if (st.a + 1 == k) {
      // No merge pending: the next kWalk steps are decided from the sizes
      // known in advance, each as if the steps before it kept their
      // boundary; the first merge (or meeting) ends the batch.
      const uint64_t kk = k + tid;
      const bool valid = kk < ke;
      bool merge = false, met = false;
      if (valid) {
        const uint64_t u = pair[kk - 1];
        merge = u != kNoMerge && u < cost[kk - 1] + cost[kk];
        if (kFix && !merge) met = bit_set(keep, kk);
      }
      const uint32_t steps = uint32_t(ke - k < kWalk ? ke - k : kWalk);
      const uint32_t fm = first_of(w, 0, merge);
      const uint32_t fs = kFix ? first_of(w, 1, met) : kWalk;
      const uint32_t stop = min(min(fm, fs), steps);
      set_run(keep, k, stop);
      __syncthreads();               // the masks are read
      if (fs < fm) return true;      // kFix: both runs keep boundary k + fs
      if (fm == kWalk) {             // every valid step kept its boundary
        st.a = k + steps - 1;
        st.cc = cost[st.a];
        st.sum = psum[st.a];
        sa = s[st.a];
        k += steps;
        continue;
      }
      const uint64_t km = k + fm;
      if (kFix) clear_run(keep, km, 1);
      st.a = km - 1;
      st.cc = pair[km - 1];
      sa = s[km - 1];
      st.sum = join(psum[km - 1], psum[km], s[km] - sa);
      hr = HullRegs{{0, 0}, kHullNone};
      solo = 0;
      k = km + 1;
      continue;
    }
    // The current partition absorbed others.
    if (k < w0 || k >= w1) {
      w0 = k;
      w1 = ke - k < kWalk ? ke : k + kWalk;
      __syncthreads();  // every read of the old window is done
      if (tid < w1 - w0) {
        w.s[tid] = s[w0 + tid];
        w.cost[tid] = cost[w0 + tid];
        w.psum[tid] = psum[w0 + tid];
      }
      if (tid == 0) w.s[w1 - w0] = s[w1];
      vb = s[w0];
      ve = s[w1];
      if (ve - vb <= kStageVals) {
        for (uint64_t i = tid; i < ve - vb; i += kWalk) w.vals[i] = load_value(col, dtype, vb + i);
      } else {
        ve = vb;
      }
      __syncthreads();
    }
    // the value at position t of the current partition
    const auto read = [&](uint64_t t) {
      const uint64_t p = sa + t;
      return p >= vb && p < ve ? w.vals[p - vb] : load_value(col, dtype, p);
    };
    const uint64_t lold = w.s[k - w0] - sa;
    const uint64_t l0 = w.s[k - w0 + 1] - w.s[k - w0];
    uint32_t f = 0;  // steps k .. k+f-1 merge
    bool on = false;  // and the chain goes on
    if (lold + l0 > max_len) {
      // refused
    } else if (l0 > kHullAppendMax ||
               (hr.state == kHullNone && solo < kSoloMerges &&
                (l0 > kSoloMin || lold > kHullBuildNow)) ||
               (hr.state == kHullDead && (l0 > kSoloMin || lold > kDeadScanMax))) {
      // One step, its union's residuals scanned by all threads, when the
      // neighbour is long, or a long current partition has no hulls (yet).
      const RangeSum u = join(st.sum, w.psum[k - w0], lold);
      const uint64_t len = lold + l0, range = u.vmax - u.vmin;
      uint32_t bits = bitlen64(range);
      if (range < kWide) {
        const double th = ls_slope(len, u.sy, u.sty);
        int64_t rmin, rmax;
        range_scan(w, group, col + sa * dtype, dtype, len, u.vmin, range, th, rmin, rmax);
        bits = min(bits, bitlen64(uint64_t(rmax) - uint64_t(rmin)));
      }
      const uint64_t size = merged_size(len, bits);
      if (size < st.cc + w.cost[k - w0]) {
        f = 1;
        on = true;
        st.cc = size;
        st.sum = u;
        hr.state = kHullNone;  // built again when short neighbours follow
        ++solo;
      }
    } else {
      // Thread i sizes the union with partitions k .. k+i: the union's sums
      // and extremes from the partitions' summaries (a prefix across
      // threads), its slope from them, and its width from hulls: the union's
      // points lie between the current partition's and those of the batch's
      // longest union, so where the two hulls' residual ranges need the same
      // number of bits, so does the union.  Otherwise (or without hulls) the
      // added (or all) values are broadcast one by one to all threads, each
      // predicting with its own slope; without hulls the unions taken are at
      // most about twice the current length, so a run that stops early
      // wastes little.
      if (hr.state == kHullNone && lold >= kHullBuildMin) {
        if (st.sum.vmax - st.sum.vmin < kWide) {
          hr = hull_extend(w, cur, cur ^ 1, hr, 0, lold, st.sum.vmax - st.sum.vmin, read);
          cur ^= 1;
        } else {
          hr.state = kHullDead;
        }
      }
      const bool via_hull = hr.state == kHullValid;
      const uint64_t j = k + tid;
      const uint64_t len0 = lold + l0;
      uint64_t lcap = via_hull ? lold + kBatchNew : len0 + (len0 > reach ? len0 : reach);
      if (lcap > max_len) lcap = max_len;
      const uint64_t e_l = j < w1 ? w.s[j - w0 + 1] : 0;
      const bool act = j < w1 && (tid == 0 || e_l - sa <= lcap);
      RangeSum u{~uint64_t(0), 0, U128{0, 0}, U128{0, 0}};
      if (act) {
        u = w.psum[j - w0];
        u.sty = add128(u.sty, mul128x64(u.sy, w.s[j - w0] - sa));
      }
      // inclusive prefix over the threads (the inactive ones, the last, add
      // nothing), from the current partition's own summary on
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const uint64_t mn = shfl_up64(u.vmin, d), mx = shfl_up64(u.vmax, d);
        const U128 y{shfl_up64(u.sy.lo, d), shfl_up64(u.sy.hi, d)};
        const U128 ty{shfl_up64(u.sty.lo, d), shfl_up64(u.sty.hi, d)};
        if (int(lane) >= d) {
          u.vmin = mn < u.vmin ? mn : u.vmin;
          u.vmax = mx > u.vmax ? mx : u.vmax;
          u.sy = add128(u.sy, y);
          u.sty = add128(u.sty, ty);
        }
      }
      if (lane == 63) w.wave_sum[wave] = u;
      const uint32_t nact = first_of(w, 0, !act);  // also orders wave_sum
      RangeSum all = st.sum;  // summary of the longest union
#pragma unroll
      for (uint32_t v = 0; v < kWalkWaves; ++v) {
        if (v == wave) u = join(all, u, 0);
        all = join(all, w.wave_sum[v], 0);
      }
      const uint64_t len_l = act ? e_l - sa : 0;
      const uint64_t lmax = w.s[k - w0 + nact] - sa;
      const uint64_t spread = all.vmax - all.vmin;
      const uint64_t vmin = u.vmin, range = u.vmax - u.vmin;
      const bool lin = act && range < kWide;
      double th = 0.0;
      if (lin) th = ls_slope(len_l, u.sy, u.sty);
      const double pmax = __dmul_rn(fabs(th), double(len_l));  // bounds every |product|
      int64_t rmin = INT64_MAX, rmax = INT64_MIN;
      uint32_t bits = bitlen64(range);
      // the unions that a line is fitted to are the first ones; only their
      // values need a scan (1e5 values in clusters of 40, far apart: 3.2 ms
      // and now 2.7)
      const uint32_t nlin = spread < kWide ? nact : first_of(w, 2, !lin);
      const uint64_t lscan = nlin ? w.s[k - w0 + nlin] - sa : 0;
      // the values of [tb, lscan) staged in LDS, each read by every thread at
      // once, every thread predicting with its own slope; with narrow64 (in
      // every thread) offsets and predictions below 2^50, exact in binary64
      const auto scan = [&](uint64_t tb, bool narrow64) {
        double mx = -__builtin_inf(), mn = __builtin_inf();
        const double own = lin ? double(uint32_t(len_l)) : 0.0;
        for (uint64_t t0 = tb; t0 < lscan; t0 += kWalk) {
          const uint64_t t = t0 + tid;
          const uint32_t cnt = lscan - t0 < kWalk ? uint32_t(lscan - t0) : kWalk;
          __syncthreads();  // every read of the block before is done
          const uint64_t x = t < lscan ? read(t) - all.vmin : 0;
          // past the end: NaN, which maximum and minimum pass over
          if (narrow64)
            w.scan[tid] = t < lscan ? double(x) : __builtin_nan("");
          else
            w.scan[tid] = __longlong_as_double(static_cast<long long>(x));
          __syncthreads();
          if (narrow64) {
            for (uint32_t q0 = 0; q0 < cnt; q0 += 8) {
#pragma unroll
              for (uint32_t q = 0; q < 8; ++q) {
                const double tq = double(uint32_t(t0) + q0 + q);
                const double r = w.scan[q0 + q] - floor(__dmul_rn(th, tq));
                const double rr = tq < own ? r : __builtin_nan("");
                mx = fmax(mx, rr);
                mn = fmin(mn, rr);
              }
            }
          } else {
            for (uint32_t q = 0; q < cnt; ++q) {
              const uint64_t tq = t0 + q;
              if (lin && tq < len_l) {
                // counted from the thread's own smallest value: below kWide
                // for the values of its union, wherever the batch's others lie
                const uint64_t y = uint64_t(__double_as_longlong(w.scan[q])) - (vmin - all.vmin);
                const int64_t rr = int64_t(y) - predict(th, uint32_t(tq));
                rmin = rr < rmin ? rr : rmin;
                rmax = rr > rmax ? rr : rmax;
              }
            }
          }
        }
        // likewise (the batch's spread is below 2^50 there)
        if (narrow64 && mn <= mx) {
          rmin = int64_t(mn) - int64_t(vmin - all.vmin);
          rmax = int64_t(mx) - int64_t(vmin - all.vmin);
        }
      };
      // a batch of one: its slope (thread 0's) and a scan by all threads
      const auto alone = [&](double own_th) {
        if (tid == 0) w.scan[0] = own_th;
        __syncthreads();
        range_scan(w, group, col + sa * dtype, dtype, lmax, all.vmin, spread, w.scan[0], rmin, rmax);
        __syncthreads();
      };
      HullRegs grown{{0, 0}, kHullDead};
      if (via_hull) {
        if (spread < kWide) grown = hull_extend(w, cur, cur ^ 1, hr, lold, lmax, spread, read);
        const bool two = grown.state == kHullValid;
        HullRange r[2];
        if (cur == 0)
          hull_ranges(w, hr.n, two ? grown.n : hr.n, th, pmax, vmin, r);
        else
          hull_ranges(w, two ? grown.n : hr.n, hr.n, th, pmax, vmin, r);
        const HullRange own = cur == 0 ? r[0] : r[1], most = cur == 0 ? r[1] : r[0];
        const bool small = pmax < 2147483648.0;
        const uint32_t b_own = own.bits_lo();
        const bool decided = small && (b_own >= bits || (two && b_own == most.bits_hi()));
        if (first_of(w, 1, lin && !decided) == kWalk) {
          if (lin && b_own < bits) bits = b_own;
        } else {
          const bool whole =
              nact == 1 || first_of(w, 2, lin && !(small && own.exact())) != kWalk;
          const bool narrow64 =
              spread < (uint64_t(1) << 50) && first_of(w, 0, lin && !(pmax < 0x1p50)) == kWalk;
          if (nact == 1)  // one slope: thread 0's
            alone(th);
          else
            scan(whole ? 0 : lold, narrow64);
          if (!whole && lin) {
            rmin = own.min_lo < rmin ? own.min_lo : rmin;
            rmax = own.max_hi > rmax ? own.max_hi : rmax;
          }
          if (lin) bits = min(bits, bitlen64(uint64_t(rmax) - uint64_t(rmin)));
        }
      } else {
        const bool narrow64 =
            spread < (uint64_t(1) << 50) && first_of(w, 1, lin && !(pmax < 0x1p50)) == kWalk;
        scan(0, narrow64);
        if (lin) bits = min(bits, bitlen64(uint64_t(rmax) - uint64_t(rmin)));
      }
      const uint64_t size = act ? merged_size(len_l, bits) : kNoMerge;
      w.size[tid] = size;
      __syncthreads();
      const uint64_t prev = tid == 0 ? st.cc : w.size[tid - 1];
      const bool merge = act && size < prev + (act ? w.cost[j - w0] : 0);
      f = min(first_of(w, 2, act && !merge), nact);
      on = f == nact;
      if (on) {  // the chain goes on past the batch
        st.cc = w.size[f - 1];
        st.sum = all;
        if (via_hull) {
          hr = grown;  // dead when it outgrew kHullMax vertices
          cur ^= 1;
        }
      }
      __syncthreads();  // sizes and masks are read
    }
    if (kFix) clear_run(keep, k, f);
    if (on) {
      k += f;
      continue;
    }
    // step k+f refuses: boundary k+f is kept and partition k+f is current
    const uint64_t kk = k + f, lnow = w.s[kk - w0] - sa;
    reach = 2 * (held > lnow ? held : lnow);
    reach = reach < kReachMin ? kReachMin : (reach > kReachMax ? kReachMax : reach);
    held = lnow;
    // (one thread reads the bit: another's read might follow the write below)
    bool met = false;
    if (kFix) {
      met = first_of(w, 1, tid == 0 && bit_set(keep, kk)) == 0;
      __syncthreads();  // the mask is read
    }
    if (!met) set_run(keep, kk, 1);
    st.a = kk;
    st.cc = w.cost[kk - w0];
    st.sum = w.psum[kk - w0];
    sa = w.s[kk - w0];
    hr = HullRegs{{0, 0}, kHullNone};
    solo = 0;
    k = kk + 1;
    if (met) return true;
  }
  return false;
}

// Speculative pass: one workgroup per chunk of 2^chunk_log2 boundaries,
// scanned as if its first boundary were kept (chunk 0 from the true start);
// each chunk's end state and hulls go to out and hulls, and seen[q] records
// the entry state the chunk was walked from.
__global__ __launch_bounds__(kWalk) void k_merge_spec(
    const uint8_t* __restrict__ col, uint32_t dtype, const uint64_t* __restrict__ s,
    const uint64_t* __restrict__ cost, const uint64_t* __restrict__ pair,
    const RangeSum* __restrict__ psum, uint64_t m, uint64_t max_len, uint32_t chunk_log2,
    unsigned long long* __restrict__ keep, MergeState* __restrict__ out,
    ChainHull* __restrict__ hulls, uint64_t* __restrict__ seen) {
  __shared__ WalkLds lds;
  const uint64_t q = blockIdx.x;
  const uint64_t k0 = q << chunk_log2, chunk = uint64_t(1) << chunk_log2;
  if (k0 >= m) return;
  const uint64_t ke = m - k0 < chunk ? m : k0 + chunk;
  MergeState st;
  uint64_t kb = k0;
  if (q == 0) {
    set_run(keep, 0, 1);
    st = MergeState{0, cost[0], psum[0]};
    kb = 1;
  } else {
    st = MergeState{k0 - 1, cost[k0 - 1], psum[k0 - 1]};
    if (threadIdx.x == 0) seen[q] = k0 - 1;
  }
  HullRegs hr{{0, 0}, kHullNone};
  uint32_t cur = 0;
  merge_walk<false>(col, dtype, s, cost, pair, psum, max_len, kb, ke, st, keep, lds, hr, cur);
  if (threadIdx.x == 0) out[q] = st;
  hull_store(hulls + q, lds.h[cur], hr);
}

// Fix-up rounds.  out[q] is the end state (hulls[q] its hulls) of the run
// recorded in chunk q's bits, and seen[q] the state that run began in.  A
// round walks the chunks of one parity whose left neighbour's end state
// differs from seen: from that state, rewriting the chunk's bits until it
// keeps a boundary the recorded run also kept (from there on that run is
// right, and so is its end state) or reaches the chunk's end (its end state
// is the new out[q], and chunk q + 1, of the other parity, is looked at in
// the next round).  The neighbours, of the other parity, do not run in the
// same round.  Rounds 0 and 1 look at every odd and every even chunk, the
// later ones at the list the round before them left in lists[r & 1], of
// todo[0] entries; todo[1] counts the next round's.  Chunk 0 begins where
// the column does, so after round r at least chunks 0..r+1 are right; rounds
// end when one leaves an empty list.
__global__ __launch_bounds__(kWalk) void k_merge_round(
    const uint8_t* __restrict__ col, uint32_t dtype, const uint64_t* __restrict__ s,
    const uint64_t* __restrict__ cost, const uint64_t* __restrict__ pair,
    const RangeSum* __restrict__ psum, uint64_t m, uint64_t max_len, uint32_t chunk_log2,
    unsigned long long* __restrict__ keep, MergeState* __restrict__ out,
    ChainHull* __restrict__ hulls, uint64_t* __restrict__ seen, uint64_t nchunks, uint64_t round,
    uint32_t* __restrict__ lists, uint32_t* __restrict__ todo) {
  __shared__ WalkLds lds;
  const uint32_t* list = lists + (round & 1) * nchunks;
  uint32_t* next = lists + ((round + 1) & 1) * nchunks;
  const uint64_t count = round < 2 ? (nchunks + 1) / 2 : todo[0];
  for (uint64_t i = blockIdx.x; i < count; i += gridDim.x) {
    const uint64_t q = round < 2 ? 2 * i + (round == 0 ? 1 : 0) : list[i];
    if (q == 0 || q >= nchunks) continue;
    MergeState st = out[q - 1];
    const uint64_t from = st.a;
    if (from == seen[q]) continue;
    __syncthreads();  // seen[q] is read by every thread before it is written
    const uint64_t kb = q << chunk_log2, chunk = uint64_t(1) << chunk_log2;
    const uint64_t ke = m - kb < chunk ? m : kb + chunk;
    HullRegs hr{{0, 0}, kHullNone};
    uint32_t cur = 0;
    if (from + 1 < kb) hr = hull_load(hulls + (q - 1), lds.h[0]);
    const bool met = merge_walk<true>(col, dtype, s, cost, pair, psum, max_len, kb, ke, st, keep,
                                      lds, hr, cur);
    if (threadIdx.x == 0) {
      seen[q] = from;
      if (!met) {
        out[q] = st;
        if (q + 1 < nchunks) next[atomicAdd(todo + 1, 1u)] = uint32_t(q + 1);
      }
    }
    if (!met) hull_store(hulls + q, lds.h[cur], hr);
    __syncthreads();  // the walker's LDS is free
  }
}

// ---- compaction after a pass --------------------------------------------------------

constexpr uint32_t kKeepWords = 64;  // bitmap words per workgroup

// Word w of the bitmap of kept boundaries, bits from m on clear.
__device__ inline uint64_t kept_word(const unsigned long long* keep, uint64_t w, uint64_t m) {
  if (w * 64 >= m) return 0;
  const uint64_t x = keep[w];
  return m - w * 64 < 64 ? x & ((1ull << (m - w * 64)) - 1) : x;
}

// Kept boundaries in the workgroup's words.
__global__ __launch_bounds__(64) void k_keep_count(const unsigned long long* __restrict__ keep,
                                                   uint64_t m, uint64_t* __restrict__ counts) {
  uint32_t c = uint32_t(__popcll(kept_word(keep, uint64_t(blockIdx.x) * kKeepWords + threadIdx.x, m)));
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) c += uint32_t(__shfl_xor(int(c), d, 64));
  if (threadIdx.x == 0) counts[blockIdx.x] = c;
}

// Copies the kept starts to their new places with their sizes and summaries
// (a partition that absorbed others is sized afterwards), whether it
// absorbed others, and its old index.  A lane per boundary, so that a
// word's partitions are read and written side by side.
__global__ __launch_bounds__(kScanBlock) void k_keep_emit(
    const unsigned long long* __restrict__ keep, uint64_t m, const uint64_t* __restrict__ offsets,
    const uint64_t* __restrict__ starts, const uint64_t* __restrict__ cost,
    const RangeSum* __restrict__ psum, uint64_t* __restrict__ starts_out,
    uint64_t* __restrict__ cost_out, RangeSum* __restrict__ psum_out,
    uint8_t* __restrict__ changed_out, uint64_t* __restrict__ old_out) {
  constexpr uint32_t kPer = kKeepWords / (kScanBlock / 64);  // words per wavefront
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t w0 = uint64_t(blockIdx.x) * kKeepWords;
  // kept boundaries before this wavefront's words
  uint32_t c = lane < wave * kPer ? uint32_t(__popcll(kept_word(keep, w0 + lane, m))) : 0;
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) c += uint32_t(__shfl_xor(int(c), d, 64));
  uint64_t out = offsets[blockIdx.x] + c;
  for (uint32_t q = 0; q < kPer; ++q) {
    const uint64_t w = w0 + wave * kPer + q;
    const uint64_t x = kept_word(keep, w, m);
    const uint64_t k = w * 64 + lane;
    if ((x >> lane) & 1) {
      const uint64_t o = out + uint64_t(__popcll(x & ((1ull << lane) - 1)));
      const uint64_t after = lane < 63 ? x >> (lane + 1) : kept_word(keep, w + 1, m);
      const bool absorbed = k + 1 < m && !(after & 1);
      starts_out[o] = starts[k];
      cost_out[o] = cost[k];
      if (!absorbed) psum_out[o] = psum[k];
      changed_out[o] = absorbed ? 1 : 0;
      old_out[o] = k;
    }
    out += uint64_t(__popcll(x));
  }
}

// After a pass: the pair (k, k+1) of the new partitions keeps its union
// size when neither absorbed a neighbour (they were adjacent before, as old
// partitions old[k] and old[k] + 1); the others are marked for sizing.
__global__ void k_pair_reuse(uint64_t m, const uint8_t* __restrict__ changed,
                             const uint64_t* __restrict__ old, const uint64_t* __restrict__ pair,
                             uint64_t* __restrict__ pair_out, uint8_t* __restrict__ dirty) {
  const uint64_t k = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (k + 1 >= m) return;
  const bool fresh = changed[k] || changed[k + 1];
  if (!fresh) pair_out[k] = pair[old[k]];
  dirty[k] = fresh ? 1 : 0;
}

}  // namespace leco

// ---- host side ------------------------------------------------------------------

namespace {

// Device arrays of one call, one allocation for each commit, freed on every
// exit path.
struct Buffers {
  std::vector<std::pair<void**, size_t>> wanted;
  std::vector<void*> ptrs;
  ~Buffers() {
    for (void* p : ptrs) (void)hipFree(p);
  }
  template <class T>
  void add(T** p, uint64_t count) {
    static_assert(alignof(T) <= 256, "arrays begin at multiples of 256 bytes");
    wanted.emplace_back(reinterpret_cast<void**>(p), ((count ? count : 1) * sizeof(T) + 255) / 256 * 256);
  }
  bool commit() {
    size_t total = 0;
    for (const auto& w : wanted) total += w.second;
    void* q = nullptr;
    if (hipMalloc(&q, total) != hipSuccess) return false;
    ptrs.push_back(q);
    char* at = static_cast<char*>(q);
    for (const auto& w : wanted) {
      *w.first = at;
      at += w.second;
    }
    wanted.clear();
    return true;
  }
};

constexpr uint64_t kRoundGroup = 16;  // fix-up rounds launched between checks
constexpr uint64_t kRoundGrid = 1024;  // workgroups of a round that works off a list

// Boundaries per speculative chunk of a merge pass over m partitions of n
// values.  A run of merges crosses one chunk per round and every chunk is
// walked again in each round until its run is the right one, so long chunks
// save work (256 boundaries made a thousand walkers re-walk 20,000 chunks 93
// times each), as long as there is a walker for every CU: about a thousand
// chunks of 1024 (four batches, 130 us by itself) to 4096 boundaries.  Partitions that are sized one at a time (kSoloMin) take
// as long each as a batch of short ones: 16 per chunk.
uint32_t chunk_log2(uint64_t m, uint64_t n) {
  if (n / m > leco::kSoloMin) return 4;
  uint32_t c = 10;
  while (c < 12 && (m >> c) > 1024) ++c;
  return c;
}

// The most chunks a pass over at most m partitions of n values has.
uint64_t chunks_bound(uint64_t m, uint64_t n) {
  const uint64_t few = n / leco::kSoloMin;  // partitions longer than kSoloMin on average
  return ((m < few ? m : few) >> 4) + (m >> 10) + 2;
}

leco_status pfail(leco_ctx* ctx, leco_status st, const char* msg) {
  ctx->last_error = msg;
  return st;
}

// Exclusive scan of per-block counts on the host (a few thousand entries).
hipError_t scan_counts(uint64_t* counts_dev, uint64_t nblocks, uint64_t* total,
                       hipStream_t stream) {
  std::vector<uint64_t> c(nblocks);
  hipError_t e = hipMemcpyAsync(c.data(), counts_dev, 8 * nblocks, hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) return e;
  uint64_t run = 0;
  for (uint64_t i = 0; i < nblocks; ++i) {
    const uint64_t x = c[i];
    c[i] = run;
    run += x;
  }
  *total = run;
  e = hipMemcpyAsync(counts_dev, c.data(), 8 * nblocks, hipMemcpyHostToDevice, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);  // c is freed on return
  return e;
}

}  // namespace

#define P_TRY(call)                                                  \
  do {                                                               \
    const hipError_t e_ = (call);                                    \
    if (e_ != hipSuccess) return pfail(ctx, LECO_EDEVICE, hipGetErrorString(e_)); \
  } while (0)

extern "C" {

leco_status leco_partition(leco_ctx* ctx, const void* col_dev, uint64_t n, leco_dtype dtype,
                           const leco_partition_params* prm, uint64_t* starts_host,
                           uint64_t starts_cap, uint64_t* m_out, hipStream_t stream) {
  if (!ctx) return LECO_EINVAL;
  if (!prm || !m_out || (dtype != LECO_U32 && dtype != LECO_U64))
    return pfail(ctx, LECO_EINVAL, "partition: null argument or bad dtype");
  if (prm->max_len == 0 || prm->max_len > leco::kMaxPartLen || !(prm->tau == prm->tau))
    return pfail(ctx, LECO_EINVAL, "partition: max_len outside 1..2^20 or tau NaN");
  if ((prm->start_positions != 0 && prm->start_positions != 1) || prm->reserved != 0)
    return pfail(ctx, LECO_EINVAL, "partition: start_positions not 0 or 1, or reserved not 0");
  if (n && (!col_dev || (reinterpret_cast<uintptr_t>(col_dev) & (uint64_t(dtype) - 1))))
    return pfail(ctx, LECO_EINVAL, "partition: null or misaligned column");
  if (starts_cap && !starts_host) return pfail(ctx, LECO_EINVAL, "partition: null starts buffer");
  *m_out = 0;
  if (n == 0) {
    if (starts_cap < 1) return pfail(ctx, LECO_ENOSPC, "partition: starts buffer too small");
    starts_host[0] = 0;
    return LECO_OK;
  }
  P_TRY(hipSetDevice(ctx->device));
  const uint8_t* col = static_cast<const uint8_t*>(col_dev);
  const uint32_t w = uint32_t(dtype);
  const double thr = prm->tau * double(prm->sm_bits);
  Buffers buf;

  // split: bitmap of partition starts
  const uint64_t nwords = (n + 63) / 64;
  const uint64_t nseg = (n + (uint64_t(1) << leco::kSegLog2) - 1) >> leco::kSegLog2;
  const uint64_t nsub = (n + (uint64_t(1) << leco::kSubLog2) - 1) >> leco::kSubLog2;
  const uint64_t nb = (nwords + leco::kItemsPerBlock - 1) / leco::kItemsPerBlock;
  unsigned long long* bitmap = nullptr;
  leco::SplitState *states = nullptr, *ends = nullptr, *seg_states = nullptr;
  uint8_t* met = nullptr;
  uint64_t* counts = nullptr;
  buf.add(&bitmap, nwords);
  buf.add(&states, nsub);
  buf.add(&ends, nsub);
  buf.add(&met, nsub);
  buf.add(&seg_states, nseg);
  buf.add(&counts, nb);
  // starting partitions: bitmaps of their first and later values
  uint64_t *first = nullptr, *inside = nullptr, *partial = nullptr, *best = nullptr;
  const uint64_t gd_cap = uint64_t(ctx->num_cus) * 8;
  const uint64_t gd0 = (n + leco::kScanBlock - 1) / leco::kScanBlock;
  const uint64_t gd = gd0 < gd_cap ? gd0 : gd_cap;
  if (prm->start_positions) {
    buf.add(&first, nwords);
    buf.add(&inside, nwords);
    buf.add(&partial, 2 * gd);
    buf.add(&best, 2);
  }
  if (!buf.commit()) return pfail(ctx, LECO_ENOMEM, "partition: split arrays");
  P_TRY(hipMemsetAsync(bitmap, 0, 8 * nwords, stream));
  if (prm->start_positions) {
    hipLaunchKernelGGL(leco::k_dd_min, dim3(uint32_t(gd)), dim3(leco::kScanBlock), 0, stream, col,
                       w, n, partial);
    P_TRY(hipGetLastError());
    hipLaunchKernelGGL(leco::k_dd_min_final, dim3(1), dim3(64), 0, stream, partial, gd, best);
    P_TRY(hipGetLastError());
    hipLaunchKernelGGL(leco::k_mark_starting, dim3(uint32_t(gd)), dim3(leco::kScanBlock), 0, stream,
                       col, w, n, best, first, inside);
    P_TRY(hipGetLastError());
  }
  hipLaunchKernelGGL(leco::k_split_spec, dim3(uint32_t(nsub)), dim3(64), 0, stream, col, w, n,
                     thr, prm->max_len, bitmap, states, first, inside);
  P_TRY(hipGetLastError());
  hipLaunchKernelGGL(leco::k_split_meet, dim3(uint32_t(nsub)), dim3(64), 0, stream, col, w, n, thr,
                     prm->max_len, bitmap, states, ends, met, first, inside);
  P_TRY(hipGetLastError());
  hipLaunchKernelGGL(leco::k_split_fix, dim3(uint32_t(nseg)), dim3(64), 0, stream, col, w, n, thr,
                     prm->max_len, bitmap, states, ends, met, seg_states, first, inside);
  P_TRY(hipGetLastError());
  if (nseg > 1) {
    hipLaunchKernelGGL(leco::k_split_join, dim3(1), dim3(64), 0, stream, col, w, n, thr,
                       prm->max_len, bitmap, seg_states, nseg, first, inside);
    P_TRY(hipGetLastError());
  }

  // starts from the bitmap
  hipLaunchKernelGGL(leco::k_bitmap_count, dim3(uint32_t(nb)), dim3(leco::kScanBlock), 0, stream,
                     reinterpret_cast<const uint64_t*>(bitmap), nwords, counts);
  P_TRY(hipGetLastError());
  uint64_t m = 0;
  P_TRY(scan_counts(counts, nb, &m, stream));
  uint64_t *starts = nullptr, *starts2 = nullptr, *cost = nullptr, *cost2 = nullptr,
           *pair = nullptr, *pair2 = nullptr, *old = nullptr, *keep_counts = nullptr;
  uint8_t *changed = nullptr, *dirty = nullptr;
  unsigned long long* keep = nullptr;
  uint32_t *todo = nullptr, *lists = nullptr;
  leco::MergeState* mout = nullptr;
  leco::ChainHull* hulls = nullptr;
  leco::RangeSum *psum = nullptr, *psum2 = nullptr;
  uint64_t* seen = nullptr;
  const uint64_t kwords = (m + 63) / 64;
  const uint64_t nbk = (kwords + leco::kKeepWords - 1) / leco::kKeepWords;
  const uint64_t nchunks0 = chunks_bound(m, n);
  buf.add(&starts, m + 1);
  buf.add(&starts2, m + 1);
  for (uint64_t** p : {&cost, &cost2, &pair, &pair2, &old}) buf.add(p, m);
  buf.add(&changed, m);
  buf.add(&dirty, m);
  buf.add(&keep, kwords);
  buf.add(&keep_counts, nbk);
  buf.add(&mout, nchunks0);
  buf.add(&hulls, nchunks0);
  buf.add(&psum, m);
  buf.add(&psum2, m);
  buf.add(&seen, nchunks0);
  buf.add(&lists, 2 * nchunks0);
  buf.add(&todo, kRoundGroup + 1);
  if (!buf.commit()) return pfail(ctx, LECO_ENOMEM, "partition: partition arrays");
  hipLaunchKernelGGL(leco::k_bitmap_emit, dim3(uint32_t(nb)), dim3(leco::kScanBlock), 0, stream,
                     reinterpret_cast<const uint64_t*>(bitmap), nwords, counts, starts);
  P_TRY(hipGetLastError());
  P_TRY(hipMemcpyAsync(starts + m, &n, 8, hipMemcpyHostToDevice, stream));

  // merge passes
  const uint64_t grid_cap = uint64_t(ctx->num_cus) * 16;
  auto costs = [&](const uint64_t* s, uint64_t count, uint32_t span, const uint8_t* dirty,
                   uint64_t* out, leco::RangeSum* sums) {
    if (count == 0) return hipSuccess;
    const uint64_t gs = (count + leco::kEncBlock - 1) / leco::kEncBlock;
    hipLaunchKernelGGL(leco::k_costs_short, dim3(uint32_t(gs < grid_cap ? gs : grid_cap)),
                       dim3(leco::kEncBlock), 0, stream, col, w, s, count, span, prm->max_len,
                       dirty, out, sums);
    hipError_t e0 = hipGetLastError();
    if (e0 != hipSuccess) return e0;
    // chunks of ranges: at least one per resident wavefront (k_costs) or
    // workgroup (k_costs_long), at most kCostChunk ranges each
    auto chunk_for = [&](uint64_t units) {
      const uint64_t c = count / units;
      return uint32_t(c < 1 ? 1 : (c > leco::kCostChunk ? leco::kCostChunk : c));
    };
    const uint32_t cw = chunk_for(grid_cap * leco::kEncWaves);
    const uint64_t chunks_w = (count + cw - 1) / cw;
    const uint64_t gw = (chunks_w + leco::kEncWaves - 1) / leco::kEncWaves;
    hipLaunchKernelGGL(leco::k_costs, dim3(uint32_t(gw < grid_cap ? gw : grid_cap)),
                       dim3(leco::kEncBlock), 0, stream, col, w, s, count, span, prm->max_len,
                       dirty, out, sums, cw);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const uint32_t cl = chunk_for(grid_cap);
    const uint64_t chunks_l = (count + cl - 1) / cl;
    const uint64_t gl = chunks_l < grid_cap ? chunks_l : grid_cap;
    hipLaunchKernelGGL(leco::k_costs_long, dim3(uint32_t(gl)), dim3(leco::kEncBlock), 0, stream,
                       col, w, s, count, span, prm->max_len, dirty, out, sums, cl);
    return hipGetLastError();
  };
  P_TRY(costs(starts, m, 1, nullptr, cost, psum));
  if (m >= 2) P_TRY(costs(starts, m - 1, 2, nullptr, pair, nullptr));
  for (uint64_t pass = 0; prm->max_passes == 0 || pass < prm->max_passes; ++pass) {
    if (m < 2) break;
    const uint64_t words = (m + 63) / 64;
    const uint32_t clog2 = chunk_log2(m, n);
    const uint64_t nchunks = ((m - 1) >> clog2) + 1;
    P_TRY(hipMemsetAsync(keep, 0, 8 * words, stream));
    hipLaunchKernelGGL(leco::k_merge_spec, dim3(uint32_t(nchunks)), dim3(leco::kWalk), 0, stream, col, w,
                       starts, cost, pair, psum, m, prm->max_len, clog2, keep, mout, hulls, seen);
    P_TRY(hipGetLastError());
    // fix-up rounds until one leaves an empty list: chunk r is right after
    // round r, so nchunks rounds always suffice
    uint32_t left = 1;
    for (uint64_t r0 = 0; nchunks > 1 && left && r0 < nchunks + 2; r0 += kRoundGroup) {
      // todo[i] counts the entries of round r0 + i; the last one carries over
      if (r0) P_TRY(hipMemcpyAsync(todo, todo + kRoundGroup, 4, hipMemcpyDeviceToDevice, stream));
      P_TRY(hipMemsetAsync(todo + (r0 ? 1 : 0), 0, 4 * (kRoundGroup + (r0 ? 0 : 1)), stream));
      for (uint64_t i = 0; i < kRoundGroup; ++i) {
        const uint64_t r = r0 + i, all = (nchunks + 1) / 2;
        const uint64_t g = r < 2 ? all : all < kRoundGrid ? all : kRoundGrid;
        hipLaunchKernelGGL(leco::k_merge_round, dim3(uint32_t(g)), dim3(leco::kWalk), 0, stream, col, w,
                           starts, cost, pair, psum, m, prm->max_len, clog2, keep, mout, hulls,
                           seen, nchunks, r, lists, todo + i);
        P_TRY(hipGetLastError());
      }
      P_TRY(hipMemcpyAsync(&left, todo + kRoundGroup, 4, hipMemcpyDeviceToHost, stream));
      P_TRY(hipStreamSynchronize(stream));
    }
    const uint64_t blocks = (words + leco::kKeepWords - 1) / leco::kKeepWords;
    hipLaunchKernelGGL(leco::k_keep_count, dim3(uint32_t(blocks)), dim3(64), 0, stream, keep, m,
                       keep_counts);
    P_TRY(hipGetLastError());
    uint64_t m2 = 0;
    P_TRY(scan_counts(keep_counts, blocks, &m2, stream));
    if (m2 == m) break;  // the pass merged nothing
    hipLaunchKernelGGL(leco::k_keep_emit, dim3(uint32_t(blocks)), dim3(leco::kScanBlock), 0,
                       stream, keep, m, keep_counts, starts, cost, psum, starts2, cost2, psum2,
                       changed, old);
    P_TRY(hipGetLastError());
    P_TRY(hipMemcpyAsync(starts2 + m2, &n, 8, hipMemcpyHostToDevice, stream));
    // sizes and summaries of the partitions that absorbed others
    P_TRY(costs(starts2, m2, 1, changed, cost2, psum2));
    if (m2 >= 2) {
      // pair sizes for the next pass: reused, or sized where a merge happened
      hipLaunchKernelGGL(leco::k_pair_reuse, dim3(uint32_t((m2 - 1 + 255) / 256)), dim3(256), 0,
                         stream, m2, changed, old, pair, pair2, dirty);
      P_TRY(hipGetLastError());
      P_TRY(costs(starts2, m2 - 1, 2, dirty, pair2, nullptr));
    }
    P_TRY(hipStreamSynchronize(stream));  // &n stays valid until the copy is done
    std::swap(starts, starts2);
    std::swap(cost, cost2);
    std::swap(pair, pair2);
    std::swap(psum, psum2);
    m = m2;
  }
  *m_out = m;
  if (starts_cap < m + 1) return pfail(ctx, LECO_ENOSPC, "partition: starts buffer too small");
  P_TRY(hipMemcpyAsync(starts_host, starts, 8 * (m + 1), hipMemcpyDeviceToHost, stream));
  P_TRY(hipStreamSynchronize(stream));
  return LECO_OK;
}

}  // extern "C"
