// Bookkeeping of kept memory blocks, by size and by age (no calls to the runtime: whoever holds
// the pool allocates and frees).
#pragma once

#include <cstddef>
#include <cstdint>
#include <map>

namespace wc {

class BlockPool {
 public:
  explicit BlockPool(size_t limit) : limit_(limit) {}
  size_t bytes() const { return bytes_; }
  size_t limit() const { return limit_; }

  // Whether a block of this size can be kept beside the others: if not, the holder takes the
  // oldest ones out until it can, or frees a block above the limit.
  bool fits(size_t bytes) const { return bytes <= limit_ && bytes_ <= limit_ - bytes; }

  // Keeps a block that fits; false (nothing changed) if the bookkeeping has no memory.
  bool give(void* p, size_t bytes) noexcept {
    auto it = by_size_.end();
    try {
      it = by_size_.emplace(bytes, Block{p, next_});
      by_age_.emplace(next_, it);
    } catch (...) {
      if (it != by_size_.end()) by_size_.erase(it);
      return false;
    }
    ++next_;
    bytes_ += bytes;
    return true;
  }

  // Takes out the smallest kept block of at least `bytes` and at most a quarter more; null if
  // there is none.
  void* take(size_t bytes, size_t* got) noexcept {
    auto it = by_size_.lower_bound(bytes);
    if (it == by_size_.end() || it->first > bytes + bytes / 4 + 4096) return nullptr;
    return out(it, got);
  }

  // Takes out the block kept longest; null if there is none.
  void* oldest(size_t* got) noexcept { return by_age_.empty() ? nullptr : out(by_age_.begin()->second, got); }

 private:
  struct Block {
    void* p;
    uint64_t age;
  };
  typedef std::multimap<size_t, Block> Sizes;

  void* out(Sizes::iterator it, size_t* got) noexcept {
    void* p = it->second.p;
    if (got) *got = it->first;
    bytes_ -= it->first;
    by_age_.erase(it->second.age);
    by_size_.erase(it);
    return p;
  }

  size_t limit_, bytes_ = 0;
  uint64_t next_ = 0;
  Sizes by_size_;
  std::map<uint64_t, Sizes::iterator> by_age_;
};

}  // namespace wc
