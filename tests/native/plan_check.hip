// The attention's split of the whole work list (pask_plan.h), checked on the
// CPU over random calls: sequences with random HIGH / window / LOW page counts
// (empty ones included), 1-8 KV heads, head_dim 64 and 128, the workspace's
// piece bound of the C ABI for a hint at the longest sequence or one as low as
// two, and launches of 1 to 1,024 workgroups of four waves, for a decode call and for one of the
// distortion's two caches (which takes this split at any number of segments).
// The workers are as many as stream_workers says, numbered as the attention
// kernel numbers the first waves of every workgroup; each one's range is
// walked the way the kernel walks it, and:
//   - the ranges tile [0, total): every page is attended exactly once;
//   - the ranges tile [0, total) in worker order and block_of(u) is the
//     worker whose range holds u, for every page start u;
//   - every piece a worker writes has index w - block_of(seg0) in
//     [0, n_pieces) and n_pieces <= splits, and every index in [0, n_pieces)
//     of every segment is written once, the last by the worker that holds the
//     segment's last page (whose index + 1 is the merge's piece count).
// Both kinds of call, all workers and few, must have come up often.
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>
#include <vector>

#include "pask_plan.h"

using namespace pask;

namespace {
uint64_t g_s = 88172645463325252ull;
uint32_t rnd(uint32_t n) {
  g_s ^= g_s << 13;
  g_s ^= g_s >> 7;
  g_s ^= g_s << 17;
  return (uint32_t)(g_s % n);
}

int splits_for(int hint, long long segments) {   // as the C ABI sizes the workspace
  const int coarse = (hint + 127) / 128 + 2;
  if (segments > 64) return coarse;
  const int fine = (hint + 15) / 16 + 2;
  return std::max(coarse, std::min(fine, (int)(4096 / std::max<long long>(segments, 1))));
}

struct Call {
  int H;
  std::vector<SeqPages> seqs;
  std::vector<long long> excl;   // units of the sequences before b (one KV head)
  long long total;
  int mx;
};

// Pieces of the segment starting at unit seg0 with pages sp (sp.np > 0).
int n_pieces(const StreamPlan& plan, const SeqPages& sp, long long seg0) {
  return (int)(plan.block_of(seg0 + kUnit * (sp.np - 1)) - plan.block_of(seg0)) + 1;
}

int check(const Call& c, const StreamPlan& plan, const std::vector<int>& workers, int splits, const char* what) {
  // pieces[seg] -> which indices were written
  const int B = (int)c.seqs.size(), H = c.H;
  std::vector<std::vector<int>> written(B * H);
  std::vector<uint8_t> seen;   // per page of the call, in order
  long long pages_total = 0;
  for (auto& s : c.seqs) pages_total += (long long)s.np * H;
  seen.assign(pages_total, 0);
  std::vector<long long> page_base(B * H + 1, 0);
  for (int b = 0; b < B; ++b)
    for (int g = 0; g < H; ++g) page_base[b * H + g + 1] = page_base[b * H + g] + c.seqs[b].np;
  for (int w : workers) {
    const long long start = plan.start_of(w), end = plan.end_of(w);
    if (start >= end) continue;
    if (plan.block_of(start) != w) { printf("%s: block_of(start_of(%d)) = %lld\n", what, w, plan.block_of(start)); return 1; }
    // locate
    int b = (int)(std::upper_bound(c.excl.begin(), c.excl.end(), start / H) - c.excl.begin()) - 1;
    while (b < B && (c.seqs[b].len == 0 || (long long)(c.excl[b] + c.seqs[b].len) * H <= start)) ++b;
    if (b >= B) continue;
    long long excl = c.excl[b];
    SeqPages sp = c.seqs[b];
    const long long rel = start - excl * H;
    int g = (int)(rel / sp.len);
    int j0 = first_page_at(sp, (int)(rel - (long long)g * sp.len));
    while (true) {
      const long long seg0 = excl * H + (long long)g * sp.len;
      if (seg0 >= end) break;
      const int j1 = end - seg0 >= sp.len ? sp.np : first_page_at(sp, (int)(end - seg0));
      if (j0 < j1) {
        const long long slot = w - plan.block_of(seg0);
        const int np = n_pieces(plan, sp, seg0);
        if (np > splits || slot < 0 || slot >= np) {
          printf("%s: worker %d seg (%d,%d) slot %lld pieces %d splits %d\n", what, w, b, g, slot, np, splits);
          return 1;
        }
        written[b * H + g].push_back((int)slot);
        if (j1 == sp.np && slot != np - 1) { printf("%s: last page in piece %lld of %d\n", what, slot, np); return 1; }
        for (int j = j0; j < j1; ++j) {
          const long long pg = page_base[b * H + g] + j;
          if (seen[pg]++) { printf("%s: page attended twice\n", what); return 1; }
          if (plan.block_of(seg0 + kUnit * j) != w) { printf("%s: block_of(page) != worker\n", what); return 1; }
        }
      }
      if (j1 < sp.np) break;
      j0 = 0;
      if (++g == H) {
        g = 0;
        excl += sp.len;
        do {
          if (++b >= B) break;
          sp = c.seqs[b];
        } while (sp.len == 0);
        if (b >= B) break;
      }
    }
  }
  for (long long i = 0; i < pages_total; ++i)
    if (!seen[i]) { printf("%s: page %lld never attended\n", what, i); return 1; }
  for (int b = 0; b < B; ++b)
    for (int g = 0; g < H; ++g) {
      if (c.seqs[b].np == 0) continue;
      auto v = written[b * H + g];
      std::sort(v.begin(), v.end());
      const int np = n_pieces(plan, c.seqs[b], c.excl[b] * H + (long long)g * c.seqs[b].len);
      if ((int)v.size() != np) { printf("%s: segment (%d,%d) %zu pieces written, %d expected\n", what, b, g, v.size(), np); return 1; }
      for (int k = 0; k < np; ++k)
        if (v[k] != k) { printf("%s: piece index %d missing\n", what, k); return 1; }
    }
  return 0;
}
}  // namespace

int main(int argc, char** argv) {
  const int rounds = argc > 1 ? atoi(argv[1]) : 400;
  int bad = 0;
  long long calls = 0, few = 0;
  for (int r = 0; r < rounds && !bad; ++r) {
    Call c;
    const int kind = rnd(4);
    const int B = kind == 0 ? 1 + rnd(8) : (kind == 1 ? 1 + rnd(64) : 1 + rnd(300));
    c.H = 1 + rnd(8);
    int mx_tok = 0;
    const bool distortion = rnd(3) == 0;             // persists nothing
    long long acc = 0, acc_lo = 0;
    for (int b = 0; b < B; ++b) {
      const int shape = rnd(6);
      int hi = shape == 0 ? 0 : rnd(shape == 1 ? 40 : 9000), win = rnd(3) ? 0 : rnd(70), lo = rnd(2) ? rnd(3000) : 0;
      if (shape == 5) hi = 20000 + rnd(20000);
      SeqPages s = make_pages(hi, win, lo, !distortion && rnd(3) == 0 ? 1 : 0);   // with or without the step's own entry
      c.excl.push_back(acc);
      acc += s.len;
      acc_lo += low_len_of(lo);
      c.seqs.push_back(s);
      mx_tok = std::max(mx_tok, hi + win + lo + 1);
    }
    c.total = acc * c.H;
    c.mx = 0;
    for (auto& s : c.seqs) c.mx = std::max(c.mx, s.len);
    if (c.total == 0) continue;
    const long long segs = (long long)B * c.H;
    const int hint = std::max(1, mx_tok + (int)rnd(500));
    const int splits = rnd(4) ? splits_for(hint, segs) : 2 + rnd(6);   // or (a scratch limit) as few as two
    static const int groups[] = {1, 2, 16, 25, 64, 128, 250, 511, 512, 1024};
    const int limit = 4 * groups[rnd(sizeof(groups) / sizeof(groups[0]))], D = rnd(2) ? 64 : 128;
    const int n = stream_workers((int)acc, (int)acc_lo, B, D, limit, distortion ? 2 : 1);
    const int active = cdiv(n, limit / 4);
    std::vector<int> workers;
    for (int wg = 0; wg < limit / 4; ++wg)
      for (int wv = 0; wv < 4 && wv < active; ++wv) workers.push_back(wg * active + wv);
    ++calls;
    few += n < limit ? 1 : 0;
    bad |= check(c, stream_plan_of(c.total, c.mx, splits, 8, n), workers, splits, distortion ? "distortion" : "decode");
  }
  if (!bad && (few < calls / 20 || few > calls - calls / 20)) {
    printf("FAIL: few workers in %lld of %lld calls\n", few, calls);
    return 1;
  }
  printf("%s: %lld calls\n", bad ? "FAIL" : "ok", calls);
  return bad;
}
