// Work split of the attention call (stream-K): pure arithmetic on the page
// counts of a call, shared by the attention, merge and distortion kernels
// (pask_attn.hip) and callable on the host, where tests/native/plan_check.hip
// checks its invariants over many shapes.  The work of a call is counted in
// units: kUnit per page of a (sequence, KV head) segment.
#pragma once

#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>

namespace pask {

__host__ __device__ __forceinline__ int cdiv(int x, int y) { return (x + y - 1) / y; }

// a / b for 0 <= a, 0 < b: 32-bit division when both fit, as they do for any
// call below 2^32 units; the 64-bit expansion otherwise.
__host__ __device__ __forceinline__ long long udiv(long long a, long long b) {
  if ((((unsigned long long)a | (unsigned long long)b) >> 32) == 0) return (long long)((uint32_t)a / (uint32_t)b);
  return a / b;
}

// Pages of one sequence in a layer: the HIGH store, the recent window (HIGH
// layout, min(n_pos, W) slots), the LOW store and, when the call itself
// persists the step's entry, one page holding just that entry (n_x = 1), in
// that order.  Every page weighs kUnit work units (with the memory system
// saturated a page iteration costs about the same time whatever its size;
// weighting LOW pages by their bytes measured slower), so every page starts
// at a multiple of kUnit.
constexpr int kUnit = 32;
// The page of the step's own entry weighs eight pages in the ranges of calls
// with more than kAlignedSegments segments: the worker that writes and attends
// it does more than stream a page (its K / V rows are quantised, stored and
// attended from registers).  With weights of 1 / 2 / 4 / 8 pages, 64 sequences
// of 1,024-8,192 kept tokens and 64 generated took 200.1 / 198.6 / 196.1 /
// 192.5 us per call, 128 of 1,000-4,000 227.9 / 226.8 / 223.4 / 219.2, 64 with
// 88% LOW 113.3 / 112.9 / 111.9 / 111.3, 384 of 64-768 151.6 / 150.7 / 149.7 / 151.1.
#ifndef PASK_ENTRY_UNITS
#define PASK_ENTRY_UNITS 256
#endif
constexpr int kEntryUnits = PASK_ENTRY_UNITS;
struct SeqPages {
  int n_hi, n_win, n_lo;   // slots of the HIGH store, the window, the LOW store
  int np_hi, np_w, np_l;   // pages: HIGH store, + window (HIGH layout), + LOW store
  int np;                  // all pages: np_l + n_x
  int len;                 // units
};
__host__ __device__ __forceinline__ int len_of(int n_hi, int n_win, int n_lo, int n_x = 0) {
  return kUnit * (cdiv(n_hi, 16) + cdiv(n_win, 16) + cdiv(n_lo, 16)) + kEntryUnits * n_x;
}
__host__ __device__ __forceinline__ SeqPages make_pages(int n_hi, int n_win, int n_lo, int n_x = 0) {
  SeqPages s;
  s.n_hi = n_hi;
  s.n_win = n_win;
  s.n_lo = n_lo;
  s.np_hi = cdiv(n_hi, 16);
  s.np_w = s.np_hi + cdiv(n_win, 16);
  s.np_l = s.np_w + cdiv(n_lo, 16);
  s.np = s.np_l + n_x;
  s.len = len_of(n_hi, n_win, n_lo, n_x);
  return s;
}
// Units of a LOW store of n_lo slots.
__host__ __device__ __forceinline__ int low_len_of(int n_lo) { return kUnit * cdiv(n_lo, 16); }
// First page whose unit offset, kUnit per page, is >= u (s.np when there is none).
__host__ __device__ __forceinline__ int first_page_at(const SeqPages& s, int u) {
  const int j = cdiv(u, kUnit);
  return j < s.np ? j : s.np;
}

// Calls with many (sequence, KV head) segments.  The work list is the
// segments (sequence b, KV head g) in that nesting order, each the units of
// its pages.  Worker w (a wave) takes the pages that start in the w-th of equal
// contiguous ranges, [start_of(w), end_of(w)).  Every range is a multiple of
// half a page, at least min_pages pages and lo units, at least one page (pages
// start at multiples of kUnit), so each range between the first and the last of
// a segment holds a page of it, and no segment is cut into more than `splits`
// pieces (lo >= mx / (splits - 1)).  Workgroups are dealt to the 8 XCDs in
// turn; ranges 15/16 as long on the odd-numbered ones measured 4% slower at
// batch 64 with 512 workers streaming (195.0 against 188.0 us) and 5% slower
// with all 2,048 on an int4-heavy history (112.7 against 107.2 us).
struct StreamPlan {
  long long total;   // units
  int units;         // of a range
  __host__ __device__ __forceinline__ long long start_of(int w) const { return (long long)w * units; }
  __host__ __device__ __forceinline__ long long end_of(int w) const {
    const long long e = start_of(w) + units;
    return e < total ? e : total;
  }
  // Worker whose range holds unit u.
  __host__ __device__ __forceinline__ long long block_of(long long u) const { return udiv(u, units); }
};

// total: units of the call; mx: units of its longest segment; splits: pieces
// the workspace holds per segment (>= 2); min_pages: the fewest pages a range
// takes; n: workers.
__host__ __device__ __forceinline__ StreamPlan stream_plan_of(long long total, int mx, int splits, int min_pages,
                                                              int n) {
  const long long lo0 = (long long)kUnit * min_pages, lo1 = cdiv(mx, splits - 1);
  const long long least = ((lo0 > lo1 ? lo0 : lo1) + 15) / 16, even = udiv(total + 16LL * n - 1, 16LL * n);
  const long long halves = even > least ? even : least;
  return StreamPlan{total, 16 * (int)(halves < 0x7FFFFFFF / 16 ? halves : 0x7FFFFFFF / 16)};
}

// Workers such a call uses of the `limit` resident ones (`share` calls run on
// them at once).  Most of the history HIGH and long: 512 at head_dim 128, 1,024
// at 64, two per compute unit and one, with 8 MiB of pages in flight; more
// waves only lengthen the memory's queues (64 sequences, 8 KV heads, D 128,
// prompts of 1,024-8,192 tokens and 512 generated: 208.8 us with all 2,048,
// 203.5 with 1,024, 194.7 with 512, 209.8 with 768 and 242 with 384, which
// leave compute units unevenly loaded; prompts of 4,000: 175.9 -> 160.3; 8
// query heads per KV head, 96 of 16,384-32,000: 1,476 -> 1,443, 24 of
// 8,192-16,384: 204.0 -> 192.6; one query head, 24 of 16,384-32,000: 382.5 ->
// 367.8; at D 64, with 1,024 for all, 64 of 1,024-8,192: 108.6 -> 104.3, 128 of
// 4,096-16,384: 419.0 -> 413.2; as one of the distortion's two caches, 24 of
// 2,048-8,192 in both, 8 query heads per KV head: 191.2 -> 181.1 for the call).
// LOW pages are bound by the latency of their arithmetic and want every wave
// (61% LOW: 231 us with 512, 172 with all; 15%: 205.8 and 210.6; 19%: even),
// and so do calls of many short segments, a few of which each worker would
// take in turn (384 sequences, 26 pages a segment: 148 us with 512, 138 with all).
__host__ __device__ __forceinline__ int stream_workers(int total, int total_lo, int batch, int head_dim, int limit,
                                                       int share) {
  if (total_lo >= total / 6 || total / kUnit < 64 * batch) return limit;
  const int few = 512 * 128 / head_dim / share;
  return few < limit ? few : limit;
}

// Calls with at most kAlignedSegments segments: every segment is cut by itself
// into pieces of about small_units units, one worker each, so no worker
// crosses into another segment, where it would start its page stream anew
// (ranges over the whole list, one sequence of 4,064 entries, 8 KV heads, D 128:
// 33 pieces of 8 pages that happened to end at the segment's end 13.8 us per
// call, 37 of 7 pages 15.5, 26 of 10 16.8).  A piece is at least min_pages and
// 3/8 of the square root of the segment's pages (longer pieces leave fewer
// partials to merge), and the call has at most 512 pieces of HIGH pages or
// 1,536 of LOW pages at D 128, twice that at D 64 (see stream_workers).  Per
// call, ranges of at least 1/32 of the longest segment -> this: one sequence of
// 264 / 2,064 / 8,064 / 32,064 entries 11.6 / 13.2 / 18.7 / 42.0 -> 9.9 / 11.8 /
// 17.7 / 30.0 us, 8 of 1,064 18.3 -> 15.4; against ranges over the whole list
// with 2,048 workers: 9 of 4,064 43.3 -> 30.7, 16 of 512-2,112 31.8 -> 22.6.
__host__ __device__ constexpr int small_low_workers(int head_dim) { return 1536 * 128 / head_dim; }
// Units a piece of such a call should have.  total, mx (of stored pages),
// splits, min_pages: as for stream_plan_of; total_lo: the units of LOW pages
// among the total.
__host__ __device__ __forceinline__ int small_units(long long total, long long total_lo, int mx, int splits,
                                                    int min_pages, int head_dim) {
  int u = kUnit * min_pages;
  const int n = small_low_workers(head_dim);
  const int lo1 = cdiv(mx, splits > 2 ? splits - 2 : 1), lo2 = (int)udiv(3 * total - 2 * total_lo + n - 1, n);
  const int lo3 = (int)(12.0f * sqrtf((float)(mx / kUnit)));
  u = lo1 > u ? lo1 : u;
  u = lo2 > u ? lo2 : u;
  return lo3 > u ? lo3 : u;
}
// Pieces that len units of stored pages are cut into for pieces of about u
// units; the step's own entry is one piece more, the segment's last (beside
// stored pages it made its worker the call's slowest: one sequence of 2,048
// entries 12.4 us, 9.3 so).
__host__ __device__ __forceinline__ int small_pieces(int len, int u) { return (int)udiv(len + u - 1, u); }
// The pages [j0, j1) of piece p of a segment cut into n pieces of stored pages.
// None is empty: rounding a piece's units up moves the last one's start by less
// than n units, and a piece has at least 31 + n (small_units: 64 for n <= 33,
// else about 4.5 n by the square root).
__host__ __device__ __forceinline__ void small_piece(const SeqPages& s, int n, int p, int& j0, int& j1) {
  if (p == n) {
    j0 = s.np_l;
    j1 = s.np;
    return;
  }
  const int len = kUnit * s.np_l, units = (int)udiv((long long)len + n - 1, n);
  const long long u0 = (long long)p * units, u1 = u0 + units;
  const int a = first_page_at(s, (int)(u0 < len ? u0 : len)), b = first_page_at(s, (int)(u1 < len ? u1 : len));
  j0 = a < s.np_l ? a : s.np_l;
  j1 = b < s.np_l ? b : s.np_l;
}

}  // namespace pask
