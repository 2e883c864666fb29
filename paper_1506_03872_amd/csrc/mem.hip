// mem.hip -- device memory of plans and workspaces.
//
// A plan made for one question takes 20 to 50 allocations and gives them
// back at once; hipMalloc and hipFree map and unmap the pages each time
// (create + topk + destroy of a sparse plan of 50,000 vectors with s = 1e7,
// 0.7 GB: 9.3 ms, or 56 in a process with other plans alive; 3.8 ms from the
// free list).  Blocks that a destroyed plan held therefore go to a free list
// (mem_pool.hpp), from which later allocations on the same device are
// served.  Only destroyed plans put blocks there, after the plan's device
// has been synchronised (buffers that grow during a plan's life are freed by
// hipFree, which waits for the device itself).  Contents are not cleared, as
// hipMalloc's are not.
#include "mem_pool.hpp"
#include "plan.hpp"

namespace mad {

namespace {

struct HipRuntime {
  typedef hipError_t Error;
  static constexpr Error kOk = hipSuccess, kNoMemory = hipErrorOutOfMemory;
  static Error device(int* dev) { return hipGetDevice(dev); }
  static Error alloc(void** p, size_t bytes) {
    const hipError_t e = hipMalloc(p, bytes);
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
  }
  static void release(void* p) { (void)hipFree(p); }
};

// never destroyed: at process exit the runtime may be gone before it
MemPool<HipRuntime>& pool() {
  static MemPool<HipRuntime>* p = new MemPool<HipRuntime>();
  return *p;
}

thread_local int t_idle_dev = -1;

}  // namespace

PoolScope::PoolScope(int idle_dev) { t_idle_dev = idle_dev; }
PoolScope::~PoolScope() { t_idle_dev = -1; }

hipError_t mem_alloc(void** out, size_t bytes) {
  return pool().alloc(out, bytes);
}

void mem_free(void* p) { pool().release(p, t_idle_dev); }

size_t mem_trim() { return pool().trim(); }

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
