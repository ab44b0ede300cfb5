// The work split of attention calls with few segments (pask_plan.h), checked
// on the CPU over random calls of up to 64 sequences and 128 segments (empty
// sequences, LOW and window pages, the step's own entry, one to eight KV
// heads, head_dim 64 and 128, the workspace's piece bound for any hint): the
// workers of the launch walk their pieces as the attention kernel does, every
// page is attended once, no segment has more pieces than the workspace holds,
// a segment's pieces that hold pages are 0..k-1 with the last page in piece
// k-1 (the step's own entry a piece of its own), and no piece has more than
// twice the pages of an equal cut.
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>
#include <vector>

#include "pask_plan.h"

using namespace pask;

static uint64_t g_s = 88172645463325252ull;
static uint32_t rnd(uint32_t n) {
  g_s ^= g_s << 13;
  g_s ^= g_s >> 7;
  g_s ^= g_s << 17;
  return (uint32_t)(g_s % n);
}

static int splits_for(int hint, long long segments) {   // as the C ABI sizes the workspace
  const int coarse = (hint + 127) / 128 + 2;
  if (segments > 64) return coarse;
  const int fine = (hint + 15) / 16 + 2;
  return std::max(coarse, std::min(fine, (int)(4096 / std::max<long long>(segments, 1))));
}

int main(int argc, char** argv) {
  const int rounds = argc > 1 ? atoi(argv[1]) : 400;
  for (int r = 0; r < rounds; ++r) {
    const int H = 1 + rnd(8), B = 1 + rnd(std::min(64, 128 / H)), D = rnd(2) ? 64 : 128;
    std::vector<SeqPages> s;
    long long total = 0, total_lo = 0;
    int mx = 0, mx_tok = 1;
    for (int b = 0; b < B; ++b) {
      const int shape = rnd(6);
      const int hi = shape == 0 ? 0 : rnd(shape == 1 ? 40 : (shape == 5 ? 40000 : 5000));
      const int win = rnd(3) ? 0 : rnd(70), lo = rnd(2) ? rnd(rnd(4) ? 3000 : 40000) : 0;
      s.push_back(make_pages(hi, win, lo, rnd(3) == 0 ? 1 : 0));
      total += (long long)kUnit * s[b].np_l * H;
      total_lo += (long long)low_len_of(lo) * H;
      mx = std::max(mx, kUnit * s[b].np_l);
      mx_tok = std::max(mx_tok, hi + win + lo + 1);
    }
    // the C ABI's bound for a hint at the longest sequence, or (a scratch limit) as few as two
    const int splits = rnd(4) ? splits_for(mx_tok, (long long)B * H) : 2 + rnd(6);
    const int u = small_units(total, total_lo, mx, splits, 4, D);
    std::vector<int> cuts(B), pieces(B), upto(B);
    int acc = 0;
    for (int b = 0; b < B; ++b) {
      cuts[b] = s[b].np_l > 0 ? small_pieces(kUnit * s[b].np_l, u) : 0;
      pieces[b] = cuts[b] + s[b].np - s[b].np_l;
      upto[b] = acc += pieces[b];
    }
    const int n_workers = small_low_workers(D) + 2 * B * H;
    if (acc * H > n_workers) { printf("FAIL: %d pieces, %d workers\n", acc * H, n_workers); return 1; }
    std::vector<std::vector<std::vector<int>>> seen(B, std::vector<std::vector<int>>(H));
    std::vector<std::vector<int>> last(B, std::vector<int>(H, -1)), held(B, std::vector<int>(H, 0));
    for (int b = 0; b < B; ++b)
      for (int g = 0; g < H; ++g) seen[b][g].assign(s[b].np, 0);
    for (int wg = 0; wg < n_workers; ++wg) {
      int b = 0;
      while (b < B && wg >= upto[b] * H) ++b;
      if (b == B) continue;
      const int q = wg - (upto[b] - pieces[b]) * H, p = q / H, g = q - p * H;
      int j0, j1;
      small_piece(s[b], cuts[b], p, j0, j1);
      if (j0 >= j1) continue;
      if (p >= splits) { printf("FAIL: piece %d of %d\n", p, splits); return 1; }
      if (p < cuts[b] && j1 - j0 > 2 * (s[b].np_l / cuts[b] + 1)) { printf("FAIL: %d pages in a piece\n", j1 - j0); return 1; }
      for (int j = j0; j < j1; ++j) ++seen[b][g][j];
      ++held[b][g];
      if (j1 == s[b].np) last[b][g] = p;
    }
    for (int b = 0; b < B; ++b)
      for (int g = 0; g < H; ++g) {
        for (int j = 0; j < s[b].np; ++j)
          if (seen[b][g][j] != 1) { printf("FAIL: page %d attended %d times\n", j, seen[b][g][j]); return 1; }
        if (s[b].np > 0 && last[b][g] + 1 != held[b][g]) { printf("FAIL: a gap in the pieces\n"); return 1; }
      }
  }
  printf("ok: %d calls\n", rounds);
  return 0;
}
