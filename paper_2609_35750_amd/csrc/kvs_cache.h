// Internal interface of the host-side block manager of the streamed paged KV
// cache (kvs_cache.cpp).  Not part of the public ABI; the C entry points in
// kvs_api.cpp wrap it.
#pragma once

#include <stdint.h>

#include <memory>
#include <string>
#include <unordered_map>
#include <vector>

namespace kvs {

// Slots by trace position.  Positions come in long consecutive stretches, so
// they are kept in pages of 256 found through one hash lookup a page (one a
// token, twice over, made 384 tokens cost 22 us).
class SlotMap {
 public:
  static constexpr int kNone = -1;
  // the entry of a position >= 0 (NULL if its page does not exist; make: the page is made first, and stays empty
  // until something is counted on it)
  int* find(int pos) {
    Page* p = page(pos >> kBits);
    return p ? &p->slot[pos & kMask] : nullptr;
  }
  int* make(int pos);
  int live() const { return live_; }
  void count(int pos, int d);       // d more (or fewer) live entries on the position's page; an empty page is dropped
  void clear();
  template <typename F>
  void each(F f) const {
    for (const auto& kv : pages_)
      for (int s : kv.second->slot)
        if (s != kNone) f(s);
  }

 private:
  static constexpr int kBits = 8, kMask = (1 << kBits) - 1;
  struct Page {
    int live = 0;
    int slot[1 << kBits];
  };
  Page* page(int idx);
  std::unordered_map<int, std::unique_ptr<Page>> pages_;
  int last_idx_ = -1, live_ = 0;
  Page* last_ = nullptr;
};

class BlockManager {
 public:
  enum { kOk = 0, kBadArg = 1, kBadState = 2, kCapacity = 3 };

  BlockManager(int num_blocks, int block_size, int num_seqs, int max_blocks);

  // Slots for n new tokens of sequence seq at trace positions pos[0..n)
  // (all-or-nothing: on error nothing changes).
  int append(int seq, const int32_t* pos, int n, int32_t* slots, std::string* err);
  // Evict the entries at trace positions pos[0..n) (all-or-nothing); writes
  // their slots.  Blocks left with no live entry return to the free list.
  int evict(int seq, const int32_t* pos, int n, int32_t* slots, std::string* err);
  // Drop the whole sequence; writes its live slots (sorted) and their count.
  int release(int seq, int32_t* slots, int* n_slots, std::string* err);
  // block_table [num_seqs][max_blocks] (unused entries 0), seq_blocks [num_seqs].
  void tables(int32_t* block_table, int32_t* seq_blocks) const;
  int free_blocks() const { return (int)free_.size(); }
  int live(int seq) const;

  int num_blocks() const { return nb_; }
  int block_size() const { return bs_; }
  int num_seqs() const { return ns_; }
  int max_blocks() const { return mb_; }

 private:
  void drop_block(int seq, int blk, size_t* at);

  int nb_, bs_, ns_, mb_;
  std::vector<int> free_;                               // free block ids (LIFO)
  std::vector<std::vector<int>> blocks_;                // per sequence, allocation order
  std::vector<int> tail_fill_;                          // per sequence: used slots of its last block
  std::vector<int> live_;                               // per block: live entries
  std::vector<SlotMap> slot_of_;                        // per sequence: trace position -> slot
};

}  // namespace kvs
