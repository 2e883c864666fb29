// mem_pool.hpp -- the free list behind mem_alloc and mem_free (mem.hip).
//
// Rules of the list:
//   - a block keeps the device it was allocated on, and only an allocation
//     for that device is served from it, whatever device the releasing
//     thread has current;
//   - it takes only blocks of the device that the release names as idle (no
//     kernel that used a block is still running there, so any thread may use
//     it on any stream); every other block goes back to the runtime;
//   - it holds at most kPoolBytes; the oldest blocks are freed to make room,
//     and so is a block that kPoolAge later releases did not need;
//   - when an allocation fails, the whole list is given back and the
//     allocation tried again; trim() gives it back at any time.
//
// RT is the runtime's part: the type Error with values kOk and kNoMemory, and
// static `Error device(int*)` (the current device), `Error alloc(void**,
// size_t)` on it and `void release(void*)`.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <mutex>
#include <new>
#include <unordered_map>
#include <vector>

namespace mad {

constexpr size_t kPoolBytes = size_t(2) << 30;
constexpr uint64_t kPoolAge = 1024;

template <class RT>
class MemPool {
 public:
  typedef typename RT::Error Error;

  // *out = at least `bytes` bytes on the current device
  Error alloc(void** out, size_t bytes) {
    *out = nullptr;
    const size_t want = rounded(bytes > 0 ? bytes : 1);
    int dev = 0;
    Error e = RT::device(&dev);
    if (e != RT::kOk) return e;
    try {
      {
        std::lock_guard<std::mutex> lock(mu_);
        // the smallest block that fits and wastes at most a quarter
        size_t best = free_.size();
        for (size_t q = 0; q < free_.size(); ++q) {
          const Block& b = free_[q];
          if (b.dev != dev || b.bytes < want || b.bytes > want + want / 4)
            continue;
          if (best == free_.size() || b.bytes < free_[best].bytes) best = q;
        }
        if (best != free_.size()) {
          const Block b = free_[best];
          live_.emplace(b.p, Live{b.bytes, b.dev});
          free_.erase(free_.begin() + (long)best);
          held_ -= b.bytes;
          *out = b.p;
          return RT::kOk;
        }
      }
      e = RT::alloc(out, want);
      if (e != RT::kOk && trim() > 0) e = RT::alloc(out, want);
      if (e != RT::kOk) {
        *out = nullptr;
        return e;
      }
      std::lock_guard<std::mutex> lock(mu_);
      live_.emplace(*out, Live{want, dev});
    } catch (const std::bad_alloc&) {
      if (*out) RT::release(*out);
      *out = nullptr;
      return RT::kNoMemory;
    }
    return RT::kOk;
  }

  // idle: the device that has been synchronised and whose blocks are kept
  // (-1: none, the block is freed)
  void release(void* p, int idle) {
    if (!p) return;
    std::vector<void*> drop;
    try {
      std::lock_guard<std::mutex> lock(mu_);
      Live l{0, -1};
      const auto it = live_.find(p);
      if (it != live_.end()) {
        l = it->second;
        live_.erase(it);
      }
      if (idle < 0 || l.dev != idle || l.bytes > kPoolBytes) {
        drop.push_back(p);
      } else {
        free_.reserve(free_.size() + 1);  // nothing below throws
        drop.reserve(free_.size());
        ++releases_;
        size_t gone = 0;
        while (gone < free_.size() &&
               (held_ + l.bytes > kPoolBytes ||
                free_[gone].born + kPoolAge < releases_)) {
          held_ -= free_[gone].bytes;
          drop.push_back(free_[gone].p);
          ++gone;
        }
        free_.erase(free_.begin(), free_.begin() + (long)gone);
        free_.push_back(Block{p, l.bytes, l.dev, releases_});
        held_ += l.bytes;
      }
    } catch (const std::bad_alloc&) {
      RT::release(p);
      return;
    }
    for (void* q : drop) RT::release(q);
  }

  // gives the whole list back; returns its bytes
  size_t trim() {
    std::vector<Block> back;
    size_t bytes = 0;
    {
      std::lock_guard<std::mutex> lock(mu_);
      back.swap(free_);
      bytes = held_;
      held_ = 0;
    }
    for (const Block& b : back) RT::release(b.p);
    return bytes;
  }

 private:
  struct Block {
    void* p;
    size_t bytes;
    int dev;
    uint64_t born;  // release count when it was put
  };
  struct Live {
    size_t bytes;
    int dev;
  };

  // whole pages for large blocks, so that sizes that differ a little match
  static size_t rounded(size_t bytes) {
    const size_t unit = bytes >= (size_t(1) << 20) ? size_t(1) << 21 : 256;
    return (bytes + unit - 1) / unit * unit;
  }

  std::mutex mu_;
  std::vector<Block> free_;  // oldest first
  std::unordered_map<void*, Live> live_;  // every block given out
  size_t held_ = 0;
  uint64_t releases_ = 0;
};

}  // namespace mad
