// Host build of the sharing of slot runs (share_runs): every item of every run
// belongs to exactly one workgroup, found as the kernels find it (the last run
// that begins at or before it), no workgroup is without items, and there are no
// more of them than the runs' work asks for, however unequal the runs are.
// Prints "ok" and exits 0, or names the first failure.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "kvs_launch.h"

static int check(kvs::SlotRuns& runs, long long per_tok) {
  long long items = 0, all = 0, need = 0;
  const unsigned grid = kvs::share_runs(&runs, per_tok, &items);
  for (int i = 0; i < runs.n; ++i) {
    const long long work = std::abs((long long)runs.r[i].len) * per_tok;
    all += work;
    need += (work + items - 1) / items;
  }
  if (grid != need || grid > 65535u + runs.n || (all <= 256ll * 65535 && items != 256)) {
    std::printf("%d runs, %lld items: %u workgroups of %lld\n", runs.n, all, grid, items);
    return 1;
  }
  long long given = 0;
  int last = -1;
  for (unsigned wg = 0; wg < grid; ++wg) {
    int k = 0;
    for (int i = 0; i < runs.n; ++i) k += runs.first[i] <= (int)wg;
    --k;
    const long long work = std::abs((long long)runs.r[k].len) * per_tok, c0 = (wg - runs.first[k]) * items;
    if (k < last || c0 >= work) {
      std::printf("workgroup %u of %u: run %d, item %lld of %lld\n", wg, grid, k, c0, work);
      return 1;
    }
    last = k;
    given += std::min(items, work - c0);
  }
  if (given != all) {
    std::printf("%lld of %lld items given out\n", given, all);
    return 1;
  }
  return 0;
}

int main() {
  std::mt19937 rng(3);
  kvs::SlotRuns runs;
  for (int it = 0; it < 3000; ++it) {
    runs.n = 1 + (int)(rng() % kvs::kMaxRuns);
    for (int i = 0, tok = 0; i < runs.n; ++i) {
      const int len = 1 + (int)(rng() % (it % 3 == 0 ? 3 : it % 3 == 1 ? 700 : 20));
      runs.r[i] = {tok, 0, 0, rng() % 2 ? len : -len};
      tok += len;
    }
    if (it % 5 == 0) runs.r[rng() % runs.n].len = 20000;   // one long run beside the others
    if (it % 500 == 0) runs.r[0].len = 0x7fffffff;
    if (check(runs, it % 2 ? 1 : 8 * (1 + rng() % 16))) return 1;
  }
  std::printf("ok\n");
  return 0;
}
