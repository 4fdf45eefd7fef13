// mcrt_blocks.hpp -- which idle device blocks the library keeps between calls,
// which one a call takes and which have to go.  Host code without HIP calls:
// the library passes the question whether a block's last use is over in as a
// function, and frees the blocks that it is handed.  Nothing here allocates or
// throws, so that blocks can be returned from destructors.
#pragma once

#include <algorithm>
#include <cstddef>
#include <mutex>

namespace mcrt {

constexpr size_t kKeepBytes = size_t(64) << 30, kKeepLarge = size_t(256) << 20;
constexpr int kKeepBlocks = 16;  // of one device
constexpr unsigned long long kKeepCalls = 32;  // calls of the library, whatever blocks they take

// What a device with `total_b` bytes, `free_b` of them free beside the idle
// blocks, may keep.
inline size_t keep_budget(size_t free_b, size_t total_b) {
  return free_b < total_b / 2 ? 0 : std::min(kKeepBytes, total_b / 4);
}

// What tells streams apart.  The handle of the stream that every thread has
// of its own (per_thread) is the same in all of them: there the thread itself
// does.
inline const void* stream_key(const void* st, const void* per_thread) noexcept {
  static thread_local const char own = 0;
  return st == per_thread ? static_cast<const void*>(&own) : st;
}

struct Block {
  unsigned char* ptr;
  size_t bytes;
  int dev;
  const void* st;  // stream of the last use (stream_key)
  void* done;      // event: end of the last use
  unsigned long long use;
};

class BlockStore {
 public:
  // A call of the library begins.
  void call() noexcept {
    std::lock_guard<std::mutex> lock(mu_);
    ++clock_;
  }
  // A block of at least `bytes` from the kept ones; false: none fits.
  // over(block): whether its last use has ended.
  template <class Over>
  bool take(size_t bytes, int dev, const void* st, Over over, Block& out) noexcept {
    std::lock_guard<std::mutex> lock(mu_);
    int best = n_;
    for (int i = 0; i < n_; ++i) {
      const Block& b = idle_[i];
      if (b.dev != dev || b.bytes < bytes || b.bytes / 4 > std::max(bytes, size_t(16) << 20)) continue;
      if (b.st != st && !over(b)) continue;
      if (best == n_ || b.bytes < idle_[best].bytes) best = i;
    }
    if (best == n_) return false;
    out = remove(best);
    return true;
  }
  // Keeps a block; false: there is no room for it.
  bool keep(Block b) noexcept {
    std::lock_guard<std::mutex> lock(mu_);
    if (n_ == kRoom) return false;
    b.use = clock_;
    idle_[n_++] = b;
    return true;
  }
  // A block that has to go when device `dev` has kept one: the device's
  // longest unused, or one of another device that is too old (over(block) says
  // that nothing has to be waited for there); false: none.
  template <class Over>
  bool excess(int dev, size_t budget, Over over, Block& out) noexcept {
    std::lock_guard<std::mutex> lock(mu_);
    size_t total = 0;
    int count = 0, old = n_;
    for (int i = 0; i < n_; ++i) {
      if (idle_[i].dev != dev) continue;
      total += idle_[i].bytes;
      ++count;
      if (old == n_ || idle_[i].use < idle_[old].use) old = i;
    }
    if (old < n_ && (total > budget || count > kKeepBlocks || aged(idle_[old]))) {
      out = remove(old);
      return true;
    }
    for (int i = 0; i < n_; ++i)
      if (idle_[i].dev != dev && aged(idle_[i]) && over(idle_[i])) {
        out = remove(i);
        return true;
      }
    return false;
  }
  // Any block of a device (dev < 0: of all); false: none is left.
  bool drop(int dev, Block& out) noexcept {
    std::lock_guard<std::mutex> lock(mu_);
    for (int i = 0; i < n_; ++i)
      if (dev < 0 || idle_[i].dev == dev) {
        out = remove(i);
        return true;
      }
    return false;
  }
  size_t idle_bytes(int dev) noexcept {
    std::lock_guard<std::mutex> lock(mu_);
    size_t n = 0;
    for (int i = 0; i < n_; ++i)
      if (idle_[i].dev == dev) n += idle_[i].bytes;
    return n;
  }

 private:
  bool aged(const Block& b) const noexcept { return b.use + kKeepCalls < clock_; }
  Block remove(int i) noexcept {
    const Block b = idle_[i];
    for (--n_; i < n_; ++i) idle_[i] = idle_[i + 1];
    return b;
  }
  static constexpr int kRoom = 1024;
  std::mutex mu_;
  Block idle_[kRoom];
  int n_ = 0;
  unsigned long long clock_ = 0;
};

}  // namespace mcrt
