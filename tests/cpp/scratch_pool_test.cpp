// csrc/scratch_pool.h on a stub device of limited memory: what is kept, evicted and given back,
// under the budget, when the device is full (the pool's own blocks, then those of the others), and
// from several threads.  Prints "scratch_pool ok" when every check holds.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <thread>
#include <vector>

#include "scratch_pool.h"

static int failures = 0;
#define CHECK(c) \
  do { \
    if (!(c)) { \
      std::printf("FAIL line %d: %s\n", __LINE__, #c); \
      ++failures; \
    } \
  } while (0)

struct Device {
  std::mutex mu;
  size_t total, used = 0, gets = 0, waits = 0;
  std::map<void*, size_t> live;
};
struct Stub;
using Pool = rsv::ScratchPool<Stub>;
static std::vector<Pool*> pools;
struct Stub {
  Device* d;
  bool get(size_t bytes, void** p) {
    std::lock_guard<std::mutex> lk(d->mu);
    if (d->used + bytes > d->total) return false;
    *p = std::malloc(1);
    d->live[*p] = bytes;
    d->used += bytes;
    ++d->gets;
    return true;
  }
  void put(void* p) {
    std::lock_guard<std::mutex> lk(d->mu);
    CHECK(d->live.count(p) == 1);
    d->used -= d->live[p];
    d->live.erase(p);
    std::free(p);
  }
  void wait() {
    std::lock_guard<std::mutex> lk(d->mu);
    ++d->waits;
  }
  bool half_free() {
    std::lock_guard<std::mutex> lk(d->mu);
    return d->total - d->used >= d->total / 2;
  }
  void reclaim();
};
void Stub::reclaim() {
  for (Pool* p : pools) p->trim();
}

int main() {
  const size_t K = 4096, L = Pool::kLarge;
  Device d;
  d.total = 100 * L;
  void *a, *b, *c;
  {  // kept for the next borrower of the size (in pages), not for allocations
    Pool p(0, 10 * K, Stub{&d});
    CHECK(p.borrow(K - 5, &a) == Pool::kOk && p.in_use() == K - 5);
    p.give_back(a, K - 5, true);
    CHECK(p.in_use() == 0 && d.used == K && d.waits == 0);
    CHECK(p.alloc(K, &b) == Pool::kOk && b != a && d.used == 2 * K);
    CHECK(p.borrow(K, &c) == Pool::kOk && c == a && d.used == 2 * K);
    p.release(b, K);
    CHECK(d.used == K);
    p.give_back(c, K, false);
    CHECK(d.waits == 1 && d.used == K && p.trim() == K && d.used == 0 && p.trim() == 0);
    // at most keep_max bytes and kMaxKept blocks, the oldest go first
    std::vector<void*> v(Pool::kMaxKept + 4);
    for (size_t i = 0; i < 4; ++i) CHECK(p.borrow((i + 1) * K, &v[i]) == Pool::kOk);
    for (size_t i = 0; i < 4; ++i) p.give_back(v[i], (i + 1) * K, true);
    CHECK(d.used == 10 * K);
    CHECK(p.borrow(5 * K, &a) == Pool::kOk);
    p.give_back(a, 5 * K, true);  // 1 + 2 + 3 make way
    CHECK(d.used == 9 * K);
    CHECK(p.borrow(11 * K, &a) == Pool::kOk);
    p.give_back(a, 11 * K, true);  // more than keep_max is not kept, and evicts nothing
    CHECK(d.used == 9 * K && p.trim() == 9 * K);
  }
  {
    Pool p(0, 1000 * K, Stub{&d});
    std::vector<void*> v(Pool::kMaxKept + 4);
    for (void*& x : v) CHECK(p.borrow(K, &x) == Pool::kOk);
    for (void* x : v) p.give_back(x, K, true);
    CHECK(d.used == Pool::kMaxKept * K);
  }
  CHECK(d.used == 0);  // the pool's end gives everything back
  {  // large blocks only while half of the device is free
    Pool p(0, 60 * L, Stub{&d});
    CHECK(p.borrow(40 * L, &a) == Pool::kOk && p.borrow(20 * L, &b) == Pool::kOk && p.borrow(K, &c) == Pool::kOk);
    p.give_back(b, 20 * L, true);
    CHECK(d.used == 40 * L + K);
    p.give_back(c, K, true);
    CHECK(d.used == 40 * L + K);
    p.give_back(a, 40 * L, true);
    CHECK(d.used == 40 * L + K && p.trim() == 40 * L + K);
  }
  {  // the budget: refused on what is in use, kept blocks make way
    Pool p(10 * K, 100 * K, Stub{&d});
    CHECK(p.borrow(6 * K, &a) == Pool::kOk);
    CHECK(p.borrow(5 * K, &b) == Pool::kOverBudget && b == nullptr && p.in_use() == 6 * K);
    CHECK(p.alloc(size_t(-1), &b) == Pool::kOverBudget);
    p.give_back(a, 6 * K, true);
    CHECK(d.used == 6 * K);
    CHECK(p.alloc(4 * K, &b) == Pool::kOk && d.used == 10 * K);  // fits beside it
    CHECK(p.borrow(2 * K, &c) == Pool::kOk && d.used == 6 * K);  // fits only without it
    p.give_back(c, 2 * K, true);
    p.release(b, 4 * K);
    CHECK(p.in_use() == 0 && d.used == 2 * K);
  }
  {  // a full device: the own kept blocks first, then the other pools', then a refusal
    d.total = 10 * K;
    Pool p(0, 100 * K, Stub{&d}), q(0, 100 * K, Stub{&d});
    pools = {&p, &q};
    CHECK(p.borrow(4 * K, &a) == Pool::kOk && q.borrow(4 * K, &b) == Pool::kOk);
    p.give_back(a, 4 * K, true);
    q.give_back(b, 4 * K, true);
    CHECK(d.used == 8 * K && p.alloc(6 * K, &a) == Pool::kOk && d.used == 10 * K);
    CHECK(p.borrow(3 * K, &b) == Pool::kOk && d.used == 9 * K);
    CHECK(q.borrow(2 * K, &c) == Pool::kNoMemory && c == nullptr && q.in_use() == 0);
    p.give_back(b, 3 * K, true);
    CHECK(q.alloc(4 * K, &c) == Pool::kOk && d.used == 10 * K);
    p.release(a, 6 * K);
    q.release(c, 4 * K);
    CHECK(d.used == 0);
    pools.clear();
  }
  {  // threads share a pool while another trims it
    d.total = 100 * L;
    Pool p(0, 64 * K, Stub{&d});
    std::vector<std::thread> ts;
    for (int t = 0; t < 6; ++t)
      ts.emplace_back([&, t] {
        for (int i = 0; i < 2000; ++i) {
          void* x = nullptr;
          const size_t n = (size_t)(1 + (i * 7 + t) % 5) * K;
          if (p.borrow(n, &x) != Pool::kOk) std::abort();
          p.give_back(x, n, true);
          if (t == 0 && i % 50 == 0) p.trim();
        }
      });
    for (std::thread& t : ts) t.join();
    CHECK(p.in_use() == 0);
    const size_t used = d.used;
    CHECK(p.trim() == used && d.used == 0);
  }
  if (failures == 0) std::printf("scratch_pool ok\n");
  return failures != 0;
}
