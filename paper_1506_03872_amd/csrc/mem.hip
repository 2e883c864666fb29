// mem.hip -- device memory of plans and workspaces.
//
// A plan made for one question takes 20 to 50 allocations and gives them
// back at once; hipMalloc and hipFree map and unmap the pages each time
// (create + topk + destroy of a sparse plan of 50,000 vectors with s = 1e7,
// 0.7 GB: 9.3 ms, or 56 in a process with other plans alive; 3.8 ms from the
// free list).  Blocks that a destroyed plan held therefore go to a free list,
// from which later allocations are served:
//   - only destroyed plans put blocks there, after the device has been
//     synchronised: no kernel that used a block is still running, so any
//     thread may use it on any stream (buffers that grow during a plan's
//     life are freed by hipFree, which waits for the device itself);
//   - the list holds at most kPoolBytes; the oldest blocks are freed to make
//     room, and so is a block that kPoolAge later releases did not need;
//   - when an allocation fails, the whole list is given back and the
//     allocation tried again.
// Contents are not cleared, as hipMalloc's are not.
#include <mutex>
#include <new>
#include <unordered_map>
#include <vector>

#include "plan.hpp"

namespace mad {

namespace {

constexpr size_t kPoolBytes = size_t(2) << 30;
constexpr uint64_t kPoolAge = 1024;

struct Block {
  void* p;
  size_t bytes;
  int dev;
  uint64_t born;  // release count when it was put
};

struct Pool {
  std::mutex mu;
  std::vector<Block> free_list;  // oldest first
  std::unordered_map<void*, size_t> live;  // capacity of every block given out
  size_t held = 0;
  uint64_t releases = 0;
};

// never destroyed: at process exit the runtime may be gone before it
Pool& pool() {
  static Pool* p = new Pool();
  return *p;
}

thread_local bool t_pooling = false;

// whole pages for large blocks, so that sizes that differ a little match
size_t rounded(size_t bytes) {
  const size_t unit = bytes >= (size_t(1) << 20) ? size_t(1) << 21 : 256;
  return (bytes + unit - 1) / unit * unit;
}

}  // namespace

PoolScope::PoolScope() { t_pooling = true; }
PoolScope::~PoolScope() { t_pooling = false; }

hipError_t mem_alloc(void** out, size_t bytes) {
  *out = nullptr;
  const size_t want = rounded(bytes > 0 ? bytes : 1);
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  Pool& P = pool();
  std::vector<Block> back;
  try {
    {
      std::lock_guard<std::mutex> lock(P.mu);
      // the smallest block that fits and wastes at most a quarter
      size_t best = P.free_list.size();
      for (size_t q = 0; q < P.free_list.size(); ++q) {
        const Block& b = P.free_list[q];
        if (b.dev != dev || b.bytes < want || b.bytes > want + want / 4)
          continue;
        if (best == P.free_list.size() || b.bytes < P.free_list[best].bytes)
          best = q;
      }
      if (best != P.free_list.size()) {
        const Block b = P.free_list[best];
        P.live.emplace(b.p, b.bytes);
        P.free_list.erase(P.free_list.begin() + (long)best);
        P.held -= b.bytes;
        *out = b.p;
        return hipSuccess;
      }
    }
    e = hipMalloc(out, want);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      {
        std::lock_guard<std::mutex> lock(P.mu);
        back.swap(P.free_list);
        P.held = 0;
      }
      if (back.empty()) return e;
      for (const Block& b : back) (void)hipFree(b.p);
      e = hipMalloc(out, want);
      if (e != hipSuccess) return e;
    }
    std::lock_guard<std::mutex> lock(P.mu);
    P.live.emplace(*out, want);
  } catch (const std::bad_alloc&) {
    if (*out) (void)hipFree(*out);
    *out = nullptr;
    return hipErrorOutOfMemory;
  }
  return hipSuccess;
}

void mem_free(void* p) {
  if (!p) return;
  Pool& P = pool();
  std::vector<void*> drop;
  try {
    std::lock_guard<std::mutex> lock(P.mu);
    size_t bytes = 0;
    const auto it = P.live.find(p);
    if (it != P.live.end()) {
      bytes = it->second;
      P.live.erase(it);
    }
    int dev = 0;
    if (!t_pooling || bytes == 0 || bytes > kPoolBytes ||
        hipGetDevice(&dev) != hipSuccess) {
      drop.push_back(p);
    } else {
      ++P.releases;
      size_t gone = 0;
      while (gone < P.free_list.size() &&
             (P.held + bytes > kPoolBytes ||
              P.free_list[gone].born + kPoolAge < P.releases)) {
        P.held -= P.free_list[gone].bytes;
        drop.push_back(P.free_list[gone].p);
        ++gone;
      }
      P.free_list.erase(P.free_list.begin(), P.free_list.begin() + (long)gone);
      P.free_list.push_back(Block{p, bytes, dev, P.releases});
      P.held += bytes;
    }
  } catch (const std::bad_alloc&) {
    (void)hipFree(p);
    return;
  }
  for (void* q : drop) (void)hipFree(q);
}

hipError_t dev_alloc(DeviceBuffer& b, size_t bytes) {
  if (b.bytes >= bytes && b.p) return hipSuccess;
  dev_free(b);
  if (bytes == 0) return hipSuccess;
  const hipError_t e = mem_alloc(&b.p, bytes);
  if (e == hipSuccess) b.bytes = bytes;
  return e;
}

void dev_free(DeviceBuffer& b) {
  mem_free(b.p);
  b.p = nullptr;
  b.bytes = 0;
}

}  // namespace mad
