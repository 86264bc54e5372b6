// Checks of HostPool (csrc/host_pool.h) with ordinary memory; prints what failed.
#include "host_pool.h"

#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <thread>
#include <vector>

static std::atomic<int> gets{0}, puts_{0}, live{0}, most{0};
static std::atomic<bool> refuse{false};
static void* get(size_t n) {
  if (refuse) return nullptr;
  ++gets;
  int l = ++live, m = most;
  while (l > m && !most.compare_exchange_weak(m, l)) {}
  return std::malloc(n);
}
static void put(void* p) {
  ++puts_;
  --live;
  std::free(p);
}
static int failed = 0;
#define CHECK(x) do { if (!(x)) { ++failed; std::printf("line %d: %s\n", __LINE__, #x); } } while (0)

int main() {
  constexpr int K = eco::HostPool::kMost;
  {   // one buffer stands ready for the transfers of any number of objects, one after another
    eco::HostPool pool(64, get, put);
    for (int i = 0; i < 50; ++i) pool.join();
    CHECK(gets == 1);
    for (int i = 0; i < 50; ++i) {
      void* p = pool.take();
      CHECK(p);
      pool.give(p);
    }
    CHECK(gets == 1);
    for (int i = 0; i < 49; ++i) pool.leave();
    CHECK(live == 1);
    pool.leave();
    CHECK(live == 0);
    pool.join();   // the next first object
    CHECK(gets == 2 && live == 1);
    pool.leave();
    CHECK(live == 0);
  }
  {   // at most K at once; the next one has none until one is back
    eco::HostPool pool(64, get, put);
    pool.join();
    std::vector<void*> p;
    for (int i = 0; i < K; ++i) p.push_back(pool.take());
    for (void* q : p) CHECK(q);
    CHECK(live == K && !pool.take());
    pool.give(p.back());
    CHECK(pool.take() == p.back());
    for (void* q : p) pool.give(q);
    pool.leave();
    CHECK(live == 0);
  }
  {   // no memory: no buffer, and another try later
    eco::HostPool pool(64, get, put);
    refuse = true;
    pool.join();
    CHECK(!pool.take());
    refuse = false;
    void* p = pool.take();
    CHECK(p);
    pool.give(p);
    pool.leave();
    CHECK(live == 0);
  }
  {   // one that is not given back (its object ended with the device in error) is not handed out again
    eco::HostPool pool(64, get, put);
    pool.join();
    pool.join();
    void* lost = pool.take();
    pool.leave();
    for (int i = 0; i < 3; ++i) {
      void* p = pool.take();
      CHECK(p && p != lost);
      pool.give(p);
    }
    pool.leave();
    CHECK(live == 1);
    pool.join();
    CHECK(pool.take() != lost);
    put(lost);
    live = 0;
  }
  {   // many threads, more than buffers: a buffer has one user at a time
    most = 0;
    eco::HostPool pool(256, get, put);
    std::atomic<int> clash{0}, had{0};
    std::vector<std::thread> t;
    for (int k = 0; k < 2 * K; ++k)
      t.emplace_back([&, k] {
        for (int i = 0; i < 3000; ++i) {
          pool.join();
          if (unsigned char* p = (unsigned char*)pool.take()) {
            ++had;
            std::memset(p, k, 256);
            for (int j = 0; j < 256; j += 15) clash += p[j] != k;
            pool.give(p);
          }
          pool.leave();
        }
      });
    for (auto& x : t) x.join();
    CHECK(clash == 0 && had > 0 && most <= K && live == 0);
  }
  return failed != 0;
}
