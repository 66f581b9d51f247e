// Device workspaces of finished calls, kept for the next one: hipMalloc and
// hipFree of a step-level call's blocks cost more than its kernels (a product
// of 8192 x 480 x 8192 in FP32: 4.8 ms, of which 0.62 ms in kernels).
//
// A cache belongs to a plan (or to a device's rafeast_gemm calls); a block goes
// back to it only after the call that used it has waited for its work.  One pool
// stands behind all caches of the process and bounds what they keep together:
// past `most` bytes the blocks that were given back longest ago are freed, of
// whichever cache they are.  Every device allocation of the library goes through
// the pool, and one that fails for want of memory is tried again with everything
// idle freed.  Host code only; the allocator is passed in.
#pragma once

#include <stddef.h>

#include <algorithm>
#include <mutex>
#include <vector>

namespace rafeast {

class WorkCache;

class WorkPool {
 public:
  struct Device {
    int (*alloc)(void**, size_t);  // 0: success
    void (*release)(void*);
    int out_of_memory;             // alloc's code for it
  };
  WorkPool(Device dev, size_t most) : dev_(dev), most_(most) {}
  int alloc(void** q, size_t bytes) {
    int e = dev_.alloc(q, bytes);
    if (e == dev_.out_of_memory) {
      // one thread at a time: what another one is freeing here counts for this one
      std::lock_guard<std::mutex> lock(full_mu_);
      for (bool more = true; more && e == dev_.out_of_memory;) {
        more = give_back();
        e = dev_.alloc(q, bytes);
      }
    }
    if (e != 0) *q = nullptr;
    return e;
  }
  bool give_back();  // frees every idle block; false if there was none
  size_t idle_bytes() {
    std::lock_guard<std::mutex> lock(mu_);
    return held_;
  }

 private:
  friend class WorkCache;
  struct Block {
    void* p;
    size_t bytes;
    unsigned long long when;  // given back, in order
  };
  void release(const std::vector<Block>& blocks) {
    for (const Block& b : blocks) dev_.release(b.p);
  }
  const Device dev_;
  const size_t most_;
  std::mutex full_mu_;
  std::mutex mu_;  // of the pool and all its caches; never held across dev_'s calls
  std::vector<WorkCache*> caches_;
  size_t held_ = 0;
  unsigned long long clock_ = 0;
};

class WorkCache {
 public:
  // keeps at most `most` bytes itself
  WorkCache(WorkPool& pool, size_t most) : pool_(pool), most_(most) {
    std::lock_guard<std::mutex> lock(pool_.mu_);
    pool_.caches_.push_back(this);
  }
  ~WorkCache() {
    std::vector<WorkPool::Block> out;
    {
      std::lock_guard<std::mutex> lock(pool_.mu_);
      take_all(out);
      pool_.caches_.erase(std::find(pool_.caches_.begin(), pool_.caches_.end(), this));
    }
    pool_.release(out);
  }
  WorkCache(const WorkCache&) = delete;
  WorkCache& operator=(const WorkCache&) = delete;
  // bytes in: wanted, out: the block's size.  A kept block serves if it is at
  // most twice as large.
  int get(void** q, size_t& bytes) {
    bytes = (std::max<size_t>(bytes, 1) + 255) / 256 * 256;
    {
      std::lock_guard<std::mutex> lock(pool_.mu_);
      size_t best = idle_.size();
      for (size_t i = 0; i < idle_.size(); ++i)
        if (idle_[i].bytes >= bytes && idle_[i].bytes / 2 <= bytes &&
            (best == idle_.size() || idle_[i].bytes < idle_[best].bytes))
          best = i;
      if (best < idle_.size()) {
        *q = idle_[best].p;
        bytes = idle_[best].bytes;
        take(best);
        return 0;
      }
    }
    return pool_.alloc(q, bytes);
  }
  void put(void* q, size_t bytes) {
    std::vector<WorkPool::Block> out;
    {
      std::lock_guard<std::mutex> lock(pool_.mu_);
      const WorkPool::Block b{q, bytes, ++pool_.clock_};
      if (bytes > most_ || bytes > pool_.most_) {
        out.push_back(b);
      } else {
        while (held_ + bytes > most_) out.push_back(take(0));
        while (pool_.held_ + bytes > pool_.most_) {
          WorkCache* old = nullptr;
          for (WorkCache* c : pool_.caches_)
            if (!c->idle_.empty() && (!old || c->idle_[0].when < old->idle_[0].when)) old = c;
          out.push_back(old->take(0));
        }
        idle_.push_back(b);
        held_ += bytes;
        pool_.held_ += bytes;
      }
    }
    pool_.release(out);
  }

 private:
  friend class WorkPool;
  WorkPool::Block take(size_t i) {
    const WorkPool::Block b = idle_[i];
    idle_.erase(idle_.begin() + i);
    held_ -= b.bytes;
    pool_.held_ -= b.bytes;
    return b;
  }
  void take_all(std::vector<WorkPool::Block>& out) {
    while (!idle_.empty()) out.push_back(take(idle_.size() - 1));
  }
  WorkPool& pool_;
  const size_t most_;
  std::vector<WorkPool::Block> idle_;  // in the order they were given back
  size_t held_ = 0;
};

inline bool WorkPool::give_back() {
  std::vector<Block> out;
  {
    std::lock_guard<std::mutex> lock(mu_);
    for (WorkCache* c : caches_) c->take_all(out);
  }
  release(out);
  return !out.empty();
}

}  // namespace rafeast
