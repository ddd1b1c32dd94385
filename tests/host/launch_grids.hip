// Host build of two launch grids.  Slot runs (run_grid): every item of every run
// belongs to exactly one workgroup, found as the kernels find it (blockIdx.y, or
// the last run that begins at or before it), and there are no more workgroups
// than the runs' work asks for and kIdleGroups, however unequal the runs are.  And the
// grid of the backward's preprocess: it takes every number of rows that fits a
// launch by itself, with the key-tile statistics only where they fit as well.
// Prints "ok" and exits 0, or names the first failure.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "kvs_launch.h"

static int check(kvs::SlotRuns& runs, long long per_tok) {
  kvs::RunList list;
  const dim3 g = kvs::run_grid(runs, per_tok, &list);
  auto work = [&](int i) { return std::abs((long long)runs.r[i].len) * per_tok; };
  long long all = 0, need = 0, given = 0;
  for (int i = 0; i < runs.n; ++i) {
    all += work(i);
    need += (work(i) + 255) / 256;
  }
  const long long grid = (long long)g.x * g.y;
  if (g.x < 1 || g.y < 1 || grid > need + kvs::kIdleGroups || (list.items && grid > 65535ll + runs.n)) {
    std::printf("%d runs, %lld items: %u x %u workgroups of %lld\n", runs.n, all, g.x, g.y, list.items);
    return 1;
  }
  if (list.items == 0) {   // strides of the grid: every run has its workgroups
    if (g.y != (unsigned)runs.n) {
      std::printf("%d runs, %u rows of workgroups\n", runs.n, g.y);
      return 1;
    }
    return 0;
  }
  int last = -1;
  for (unsigned wg = 0; wg < g.x; ++wg) {
    int k = 0;
    for (int i = 0; i < runs.n; ++i) k += list.first[i] <= (int)wg;
    --k;
    const long long c0 = (wg - list.first[k]) * list.items;
    if (k < last || c0 >= work(k)) {
      std::printf("workgroup %u of %u: run %d, item %lld of %lld\n", wg, g.x, k, c0, work(k));
      return 1;
    }
    last = k;
    given += std::min(list.items, work(k) - c0);
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
  const long long most = 0xffffffffll / 256;   // workgroups of a launch
  for (long long blocks : {1ll, 1000ll, most - 5, most - 1, most})
    for (long long ks : {1ll, 2ll, 4ll, 5ll, 6ll, 4096ll, most}) {
      const kvs::PreGrid g = kvs::bwd_pre_grid(16 * blocks, ks);
      if (g.with_kstats != (blocks + ks <= most) || g.blocks != blocks + (g.with_kstats ? ks : 0) || g.blocks > most) {
        std::printf("%lld row and %lld statistics workgroups: %u, %d\n", blocks, ks, g.blocks, g.with_kstats);
        return 1;
      }
    }
  std::printf("ok\n");
  return 0;
}
