// Host-side bookkeeping of the streamed paged KV cache (the inference side of
// KV-streams, Section 2 "KV-streams" and Section 4 "Inference engine
// implementation"): cache blocks of block_size slots, a free list, and per
// sequence the list of its blocks in allocation order.  Tokens are appended
// at the tail of a sequence's last block; evicted entries are dropped for
// good (their slots are never refilled) and a block returns to the free list
// once none of its entries is live.  The device side (slot contents and the
// live marks read by the decode kernel) is updated by the caller with the
// slot lists these calls return.
#include "kvs_cache.h"

#include <algorithm>
#include <climits>
#include <cstdio>
#include <new>

namespace kvs {

SlotMap::Page* SlotMap::page(int idx) {
  if (idx == last_idx_) return last_;
  const auto it = pages_.find(idx);
  if (it == pages_.end()) return nullptr;
  last_idx_ = idx;
  return last_ = it->second.get();
}

int* SlotMap::make(int pos) {
  const int idx = pos >> kBits;
  Page* p = page(idx);
  if (!p) {
    auto fresh = std::make_unique<Page>();
    for (int& s : fresh->slot) s = kNone;
    p = fresh.get();
    pages_.emplace(idx, std::move(fresh));
    last_idx_ = idx;
    last_ = p;
  }
  return &p->slot[pos & kMask];
}

void SlotMap::count(int pos, int d) {
  const int idx = pos >> kBits;
  Page* p = page(idx);
  if (!p) return;
  p->live += d;
  live_ += d;
  if (p->live == 0) {
    pages_.erase(idx);
    last_idx_ = -1;
    last_ = nullptr;
  }
}

void SlotMap::clear() {
  pages_.clear();
  last_idx_ = -1;
  last_ = nullptr;
  live_ = 0;
}

BlockManager::BlockManager(int num_blocks, int block_size, int num_seqs, int max_blocks)
    : nb_(num_blocks), bs_(block_size), ns_(num_seqs), mb_(max_blocks),
      blocks_(num_seqs), tail_fill_(num_seqs, block_size), live_(num_blocks, 0), slot_of_(num_seqs) {
  free_.reserve(num_blocks);
  for (int b = num_blocks - 1; b >= 0; --b) free_.push_back(b);   // block 0 is handed out first
}

static int fail_msg(std::string* err, int code, const char* msg, long long a = 0) {
  if (err) {
    char buf[256];
    snprintf(buf, sizeof(buf), msg, a);
    *err = buf;
  }
  return code;
}

int BlockManager::append(int seq, const int32_t* pos, int n, int32_t* slots, std::string* err) {
  if (seq < 0 || seq >= ns_) return fail_msg(err, kBadArg, "sequence index %lld out of range", seq);
  auto& map = slot_of_[seq];
  // Reserve every position first (a marker no slot has), counted as live so that its page stays, and room for the
  // new blocks; a failure, of an allocation too, takes the markers back.
  constexpr int kReserved = -2;
  int done = 0, code = kOk;
  for (; done < n; ++done) {
    const int p = pos[done];
    if (p < 0) {
      code = fail_msg(err, kBadArg, "negative trace position %lld", p);
      break;
    }
    int* s = nullptr;
    try {
      s = map.make(p);
    } catch (const std::bad_alloc&) {
      code = fail_msg(err, kCapacity, "out of host memory at trace position %lld", p);
      break;
    }
    if (*s != SlotMap::kNone) {
      code = fail_msg(err, kBadState, "trace position %lld is already in the cache", p);
      break;
    }
    *s = kReserved;
    map.count(p, 1);
  }
  // blocks this append needs, checked before anything else changes
  const int room = bs_ - tail_fill_[seq];
  const long long need = n > room ? (n - room + bs_ - 1) / bs_ : 0;
  if (code == kOk && need > (long long)free_.size())
    code = fail_msg(err, kCapacity, "out of cache blocks (%lld more needed)", need);
  if (code == kOk && (long long)blocks_[seq].size() + need > mb_)
    code = fail_msg(err, kCapacity, "sequence would hold more than max_blocks (%lld) blocks", mb_);
  if (code == kOk) try {
      blocks_[seq].reserve(blocks_[seq].size() + need);
    } catch (const std::bad_alloc&) {
      code = fail_msg(err, kCapacity, "out of host memory for %lld blocks", need);
    }
  if (code != kOk) {
    for (int i = 0; i < done; ++i) {
      *map.find(pos[i]) = SlotMap::kNone;
      map.count(pos[i], -1);
    }
    return code;
  }
  for (int i = 0; i < n; ++i) {
    if (tail_fill_[seq] == bs_) {
      blocks_[seq].push_back(free_.back());
      free_.pop_back();
      tail_fill_[seq] = 0;
    }
    const int blk = blocks_[seq].back();
    const int slot = blk * bs_ + tail_fill_[seq]++;
    ++live_[blk];
    *map.find(pos[i]) = slot;
    slots[i] = slot;
  }
  return kOk;
}

// at: where the caller's last block stood in the list, and where this one did; an eviction of consecutive positions
// frees consecutive blocks, so the search for each ends where the last one did.
void BlockManager::drop_block(int seq, int blk, size_t* at) {
  auto& bl = blocks_[seq];
  const bool tail = !bl.empty() && bl.back() == blk;
  const auto it = *at < bl.size() && bl[*at] == blk ? bl.begin() + *at : std::find(bl.begin(), bl.end(), blk);
  *at = it - bl.begin();
  bl.erase(it);
  free_.push_back(blk);
  if (tail) tail_fill_[seq] = bs_;   // the next append opens a new block
}

int BlockManager::evict(int seq, const int32_t* pos, int n, int32_t* slots, std::string* err) {
  if (seq < 0 || seq >= ns_) return fail_msg(err, kBadArg, "sequence index %lld out of range", seq);
  auto& map = slot_of_[seq];
  // Mark every entry as taken first (the sign bit of its slot; no slot gives kNone), so that a repeated position
  // shows; a failure takes the marks back.
  constexpr int kTaken = INT_MIN;
  for (int i = 0; i < n; ++i) {
    int* s = pos[i] < 0 ? nullptr : map.find(pos[i]);
    if (!s || *s < 0) {
      const int code = s && *s != SlotMap::kNone
                           ? fail_msg(err, kBadState, "trace position %lld evicted twice", pos[i])
                           : fail_msg(err, kBadState, "trace position %lld is not in the cache", pos[i]);
      while (--i >= 0) {
        int* t = map.find(pos[i]);
        *t ^= kTaken;
      }
      return code;
    }
    *s ^= kTaken;
  }
  size_t at = 0;
  for (int i = 0; i < n; ++i) {
    const int p = pos[i];
    int* s = map.find(p);
    const int slot = *s ^ kTaken;
    *s = SlotMap::kNone;
    map.count(p, -1);
    slots[i] = slot;
    const int blk = slot / bs_;
    if (--live_[blk] == 0) drop_block(seq, blk, &at);
  }
  return kOk;
}

int BlockManager::release(int seq, int32_t* slots, int* n_slots, std::string* err) {
  if (seq < 0 || seq >= ns_) return fail_msg(err, kBadArg, "sequence index %lld out of range", seq);
  int k = 0;
  slot_of_[seq].each([&](int slot) { slots[k++] = slot; });
  std::sort(slots, slots + k);
  *n_slots = k;
  slot_of_[seq].clear();
  for (int blk : blocks_[seq]) {
    live_[blk] = 0;
    free_.push_back(blk);
  }
  blocks_[seq].clear();
  tail_fill_[seq] = bs_;
  return kOk;
}

void BlockManager::tables(int32_t* block_table, int32_t* seq_blocks) const {
  for (int s = 0; s < ns_; ++s) {
    const auto& bl = blocks_[s];
    seq_blocks[s] = (int32_t)bl.size();
    for (int i = 0; i < mb_; ++i) block_table[(size_t)s * mb_ + i] = i < (int)bl.size() ? bl[i] : 0;
  }
}

int BlockManager::live(int seq) const {
  return (seq >= 0 && seq < ns_) ? slot_of_[seq].live() : -1;
}

}  // namespace kvs
