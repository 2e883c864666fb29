// Checks of the free list of destroyed plans' memory (mem_pool.hpp) against a
// runtime of two devices on the host.  Exit status 0: all hold.
#include "../paper_1506_03872_amd/csrc/mem_pool.hpp"

#include <stdio.h>
#include <stdlib.h>

#include <map>
#include <set>
#include <thread>

namespace {

std::mutex g_mu;
std::map<void*, int> g_where;     // allocated blocks and their device
std::set<int> g_full;             // devices whose next allocation fails
thread_local int t_dev = 0;       // current device
uintptr_t g_next = 4096;          // blocks are never touched: addresses only

struct Fake {
  typedef int Error;
  static constexpr int kOk = 0, kNoMemory = 2;
  static int device(int* d) {
    *d = t_dev;
    return 0;
  }
  static int alloc(void** p, size_t bytes) {
    std::lock_guard<std::mutex> l(g_mu);
    if (g_full.erase(t_dev)) return kNoMemory;
    *p = (void*)g_next;
    g_next += bytes;
    g_where[*p] = t_dev;
    return 0;
  }
  static void release(void* p) {
    std::lock_guard<std::mutex> l(g_mu);
    if (g_where.erase(p) != 1) {
      printf("released a block twice, or one never allocated\n");
      abort();
    }
  }
};

typedef mad::MemPool<Fake> Pool;

int failed = 0;
void expect(bool ok, const char* what) {
  if (!ok) {
    printf("FAILED: %s\n", what);
    failed = 1;
  }
}

void* take(Pool& p, size_t bytes) {
  void* b = nullptr;
  expect(p.alloc(&b, bytes) == 0 && b, "an allocation succeeds");
  return b;
}

void devices() {
  Pool p;
  t_dev = 0;
  void* a = take(p, 1 << 20);
  // released while another device is current: still device 0's
  t_dev = 1;
  p.release(a, 0);
  void* b = take(p, 1 << 20);
  expect(g_where[b] == 1, "a block goes back to its own device only");
  t_dev = 0;
  void* c = take(p, 1 << 20);
  expect(c == a, "and serves the next allocation there");
  // device 1 is idle, the block is device 0's: not kept
  p.release(c, 1);
  expect(!g_where.count(c), "a block of a device that may be busy is freed");
  t_dev = 1;
  p.release(b, 1);
  expect(p.trim() > 0 && g_where.empty(), "trim gives everything back");
  expect(p.trim() == 0, "and then there is nothing left");
  t_dev = 0;
}

void sizes() {
  Pool p;
  void* a = take(p, 1000);
  p.release(a, 0);
  void* b = take(p, 2000);
  expect(b != a, "a block is not given out for more than it holds");
  void* c = take(p, 500);
  expect(c != a, "nor where it wastes more than a quarter");
  void* d = take(p, 1020);
  expect(d == a, "the block that fits is taken");
  p.release(b, -1);
  expect(!g_where.count(b), "outside of a destroyed plan blocks are freed");
  p.release(c, 0);
  p.release(d, 0);
  p.release(nullptr, 0);
  p.trim();
  expect(g_where.empty(), "nothing is lost");
}

void bounds() {
  Pool p;
  const size_t gib = size_t(1) << 30;
  void* a = take(p, gib);
  void* b = take(p, gib / 2);
  void* c = take(p, gib);
  p.release(a, 0);
  p.release(b, 0);
  expect(g_where.size() == 3, "up to 2 GiB are kept");
  p.release(c, 0);
  expect(!g_where.count(a) && g_where.count(b) && g_where.count(c),
         "the oldest blocks make room");
  void* big = take(p, 2 * gib + 1);
  p.release(big, 0);
  expect(!g_where.count(big) && g_where.count(c),
         "a block over the bound is freed and costs no other its place");
  for (uint64_t q = 0; q <= mad::kPoolAge; ++q) {
    void* s = take(p, 256);
    p.release(s, 0);
  }
  expect(!g_where.count(b) && !g_where.count(c), "unused blocks age out");
  p.trim();
  expect(g_where.empty(), "nothing is lost");
}

void failure() {
  Pool p;
  void* a = take(p, 1 << 21);
  p.release(a, 0);
  g_full.insert(0);  // the first attempt fails
  void* b = take(p, 1 << 24);
  expect(!g_where.count(a), "a failed allocation gives the list back");
  g_full.insert(0);
  void* c = nullptr;
  expect(p.alloc(&c, 1 << 24) == Fake::kNoMemory && !c,
         "with nothing to give back the error is the runtime's");
  p.release(b, -1);
  expect(g_where.empty(), "nothing is lost");
}

void threads() {
  Pool p;
  std::vector<std::thread> ts;
  for (int w = 0; w < 8; ++w)
    ts.emplace_back([&p, w] {
      t_dev = w & 1;
      unsigned r = 77u + (unsigned)w;
      std::vector<void*> mine;
      for (int q = 0; q < 4000; ++q) {
        r = r * 1664525u + 1013904223u;
        if (mine.size() < 20 && (r >> 24) % 2) {
          void* b = nullptr;
          if (p.alloc(&b, 1 + (r >> 8) % 65536) == 0) {
            {
              std::lock_guard<std::mutex> l(g_mu);
              if (g_where[b] != t_dev) failed = 1;
            }
            mine.push_back(b);
          }
        } else if (!mine.empty()) {
          p.release(mine.back(), (r >> 20) % 3 ? t_dev : -1);
          mine.pop_back();
        }
        if ((r >> 10) % 500 == 0) p.trim();
      }
      for (void* b : mine) p.release(b, t_dev);
    });
  for (std::thread& t : ts) t.join();
  expect(!failed, "threads on two devices share the list");
  p.trim();
  expect(g_where.empty(), "nothing is lost");
}

}  // namespace

int main() {
  devices();
  sizes();
  bounds();
  failure();
  threads();
  if (!failed) printf("ok\n");
  return failed;
}
