// Block manager under failing allocations: an append whose k-th allocation
// fails, for every k it makes, gives kCapacity and leaves the free blocks, the
// tables and the live entries as they were; the same append then succeeds, and
// the entries it reserved are the ones that are evicted and released.
// Prints "ok" and exits 0, or names the first failure.
#include <cstdio>
#include <cstdlib>
#include <new>
#include <vector>

#include "kvs_cache.h"

static long g_left = -1;   // allocations until one fails; -1: none fails

void* operator new(std::size_t n) {
  if (g_left >= 0 && g_left-- == 0) throw std::bad_alloc();
  if (void* p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

int main() {
  constexpr int NB = 400, BS = 4, N = 1100;
  std::vector<int32_t> pos(N), slots(N), table(2 * NB), before(2 * NB), nblk(2), nbefore(2), far(1, 5);
  for (int i = 0; i < N; ++i) pos[i] = 200 + i;   // five pages of positions
  long failures = 0;
  for (long k = 0;; ++k) {
    kvs::BlockManager bm(NB, BS, 2, NB);
    std::string err;
    err.reserve(256);
    if (bm.append(0, far.data(), 1, slots.data(), &err) != kvs::BlockManager::kOk) return 1;
    bm.tables(before.data(), nbefore.data());
    const int free_before = bm.free_blocks();
    int code = -1;
    g_left = k;
    try {
      code = bm.append(0, pos.data(), N, slots.data(), &err);
    } catch (const std::bad_alloc&) {
      g_left = -1;
      std::printf("allocation %ld: the exception leaves append\n", k);
      return 1;
    }
    const bool failed = g_left < 0;   // the k-th allocation took place
    g_left = -1;
    if (failed) {
      ++failures;
      bm.tables(table.data(), nblk.data());
      if (code != kvs::BlockManager::kCapacity || bm.free_blocks() != free_before || bm.live(0) != 1 || table != before ||
          nblk != nbefore) {
        std::printf("allocation %ld: code %d, %d free blocks (%d before), %d live\n", k, code, bm.free_blocks(), free_before,
                    bm.live(0));
        return 1;
      }
      code = bm.append(0, pos.data(), N, slots.data(), &err);
    }
    if (code != kvs::BlockManager::kOk || bm.live(0) != N + 1) {
      std::printf("allocation %ld: append after it gives %d\n", k, code);
      return 1;
    }
    std::vector<int32_t> gone(N), rest(N + 1);
    int n = 0;
    if (bm.evict(0, pos.data(), N - 1, gone.data(), &err) != kvs::BlockManager::kOk) return 1;
    for (int i = 0; i < N - 1; ++i)
      if (gone[i] != slots[i]) return 1;
    if (bm.release(0, rest.data(), &n, &err) != kvs::BlockManager::kOk || n != 2 || bm.free_blocks() != NB) return 1;
    if (!failed) break;
  }
  if (failures < 6) {
    std::printf("only %ld allocations failed\n", failures);
    return 1;
  }
  std::printf("%ld failed allocations\nok\n", failures);
  return 0;
}
