// Host build of the paged decode's split (kvs_decode_plan.h): for batches of
// many shapes, the units the sequences get
//  * are each sequence's tiles divided by the unit size, rounded up (at least
//    one), also with a reciprocal two units in the last place off;
//  * together fit the grid and workspace that were sized for them, and those
//    of one sequence the merge's list of 2,048;
//  * have rows of partial results to themselves, inside the workspace, where
//    a sequence is cut;
//  * have the smallest size that fits, or one at most an eighth and one above
//    it where the bisection stops at a sixteenth.
// Prints "ok" and exits 0, or names the first failure.
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "kvs_decode_plan.h"

static long long exact_units(const std::vector<int>& t, int c) {
  long long n = 0;
  for (int x : t) n += std::max(1, (x + c - 1) / c);
  return n;
}

static int check_count() {
  std::mt19937 rng(1);
  for (int it = 0; it < 2000000; ++it) {
    const int t = (int)(rng() % (kvs::kTileCap + 1)) >> (rng() % 20);
    const int C = std::max(kvs::kMinTiles, (int)(rng() % (kvs::kTileCap + 1)) >> (rng() % 20));
    float rc = 1.f / (float)C;
    for (int k = (int)(rng() % 5) - 2; k != 0; k += k > 0 ? -1 : 1) rc = std::nextafterf(rc, k > 0 ? 2.f : 0.f);
    const int want = std::max(1, (t + C - 1) / C), got = kvs::unit_count(t, C, rc);
    if (got != want) {
      std::printf("unit_count(%d, %d, %.9g) = %d, not %d\n", t, C, rc, got, want);
      return 1;
    }
  }
  return 0;
}

int main() {
  if (check_count()) return 1;
  std::mt19937 rng(2);
  const int sizes[] = {1, 2, 5, 63, 64, 65, 200, 255, 256, 257, 300, 600, 1024, 1025, 4097, 9000};
  const int heads[] = {1, 2, 3, 8, 16, 64, 300};
  long checked = 0, cut = 0;
  for (int S : sizes)
    for (int Hkv : heads)
      for (int D : {64, 128})
        for (int width : {1, 8, 64, 500, 9000, 33000000})
          for (int kind = 0; kind < 6; ++kind) {
            const int BS = 16, units = kvs::paged_units(S, Hkv, width, BS, D);
            if (units < S) {
              std::printf("S %d Hkv %d D %d width %d: %d units\n", S, Hkv, D, width, units);
              return 1;
            }
            ++checked;
            if (units == S) continue;   // one unit each: nothing to fit
            const int most = kvs::plan_tiles((int)std::min(width * (long long)BS, 0x7fffffffll));
            std::vector<int> t(S);
            for (int s = 0; s < S; ++s)
              t[s] = kind == 0   ? most
                     : kind == 1 ? 0
                     : kind == 2 ? (s == S / 2 ? most : 1)
                     : kind == 3 ? (int)(rng() % (most + 1ll))
                     : kind == 4 ? (int)(rng() % (most + 1ll)) >> (rng() % 24)
                                 : (s % 3 == 0 ? most : 0);
            long long total = 0;
            int top = 0;
            for (int x : t) total += x, top = std::max(top, x);
            auto units_at = [&](int c) {
              int n = 0;
              for (int x : t) n += kvs::unit_count(x, c, 1.f / (float)c);
              return n;
            };
            auto upper = [&]() { return (int)std::min<long long>(top, total / (units - S) + 1); };
            const int least = (int)((std::max(total, 1ll) - 1) / units) + 1;
            const int best = kvs::unit_size(least, units, 30, units_at, upper);
            const int C = kvs::unit_size(least, units, 4, units_at, upper);
            const long long n = exact_units(t, C);
            if (n > units || exact_units({top}, C) > 2048) {
              std::printf("S %d Hkv %d D %d width %d kind %d: size %d gives %lld units, %d sized for\n", S, Hkv, D,
                          width, kind, C, n, units);
              return 1;
            }
            cut += n > S;
            int first = 0, end = 0;   // first unit of the sequence; rows given out
            for (int s = 0; s < S; ++s) {
              const int m = kvs::unit_count(t[s], C, 1.f / (float)C), row = kvs::partial_row(S, units, s, first);
              if (m > 1 && (row < end || row + m > kvs::partial_units(S, units))) {
                std::printf("S %d Hkv %d D %d width %d kind %d: rows %d to %d of sequence %d\n", S, Hkv, D, width, kind,
                            row, row + m, s);
                return 1;
              }
              if (m > 1) end = row + m;
              first += m;
            }
            int lo = kvs::kMinTiles, hi = std::max(C, lo);   // smallest size that fits
            while (lo < hi) {
              const int c = lo + (hi - lo) / 2;
              if (exact_units(t, c) <= units) hi = c;
              else lo = c + 1;
            }
            if (best != lo || C > lo + lo / 8 + 1) {
              std::printf("S %d Hkv %d D %d width %d kind %d: sizes %d, %d where %d fits\n", S, Hkv, D, width, kind, best,
                          C, lo);
              return 1;
            }
          }
  std::printf("%ld batches checked, %ld with cut sequences\nok\n", checked, cut);
  return 0;
}
