// Checks mlkv_pool.h on the CPU against a device of its own: the HIP calls the
// pool makes are defined here, over a budget of bytes that are never touched.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <map>
#include <thread>
#include <vector>

#include "mlkv_pool.h"

namespace {
struct Alloc {
  size_t bytes;
  unsigned long long id;
};
std::mutex mu;
std::map<char*, Alloc> live;
size_t budget = ~0ull, used = 0;
unsigned long long next_id = 1;
char* next_ptr = reinterpret_cast<char*>(1ull << 40);
int device = 0, mallocs = 0, bad_frees = 0;

void reset_device() {  // as a device reset: every allocation ends, addresses are used again
  live.clear();
  used = 0;
  next_ptr = reinterpret_cast<char*>(1ull << 40);
}

int failures = 0;
void check(bool ok, const char* what, int line) {
  if (!ok) {
    std::printf("line %d: %s\n", line, what);
    ++failures;
  }
}
#define CHECK(x) check((x), #x, __LINE__)
constexpr size_t MB = 1ull << 20;

void* taken(mlkv::DevicePool& pool, size_t want, size_t* got) {
  void* p = nullptr;
  *got = want;
  return pool.take(&p, got) == hipSuccess ? p : nullptr;
}
}  // namespace

extern "C" {
hipError_t hipMalloc(void** p, size_t bytes) {
  std::lock_guard<std::mutex> lock(mu);
  if (used + bytes > budget) return hipErrorOutOfMemory;
  ++mallocs;
  used += bytes;
  live[next_ptr] = {bytes, next_id++};
  *p = next_ptr;
  next_ptr += (bytes + 4095) / 4096 * 4096;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  std::lock_guard<std::mutex> lock(mu);
  auto it = live.find(static_cast<char*>(p));
  if (it == live.end()) {
    ++bad_frees;
    return hipErrorInvalidValue;
  }
  used -= it->second.bytes;
  live.erase(it);
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = device;
  return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipPointerGetAttribute(void* data, hipPointer_attribute, hipDeviceptr_t p) {
  std::lock_guard<std::mutex> lock(mu);
  auto it = live.find(static_cast<char*>(p));
  if (it == live.end()) return hipErrorInvalidValue;
  *static_cast<unsigned long long*>(data) = it->second.id;
  return hipSuccess;
}
}

int main() {
  size_t got;
  {  // a block comes back for the next table, also a slightly smaller one, on its device
    mlkv::DevicePool pool;
    void* a = taken(pool, 100 * MB, &got);
    pool.give(0, a, got);
    const int before = mallocs;
    CHECK(taken(pool, 90 * MB, &got) == a && got == 100 * MB && mallocs == before);
    pool.give(0, a, got);
    device = 1;
    void* b = taken(pool, 100 * MB, &got);
    CHECK(b != a && got == 100 * MB);
    device = 0;
    void* c = taken(pool, 79 * MB, &got);  // 100 MB is more than a quarter larger
    CHECK(c != a && got == 79 * MB);
    void* d = taken(pool, 101 * MB, &got);
    CHECK(d != a && got == 101 * MB);
    CHECK(pool.trim() == 100 * MB && pool.trim() == 0);
    CHECK(used == 280 * MB);
    for (void* p : {b, c, d}) (void)hipFree(p);
  }
  {  // at most kPoolBytes are kept, the oldest freed first; a larger block is never kept
    mlkv::DevicePool pool;
    void* p[12];
    for (int k = 0; k < 12; ++k) p[k] = taken(pool, 40 * MB, &got);
    for (int k = 0; k < 12; ++k) {
      pool.give(0, p[k], 40 * MB);
      CHECK(used - (size_t)(11 - k) * 40 * MB <= mlkv::kPoolBytes);
    }
    CHECK(used == 240 * MB && live.count(static_cast<char*>(p[5])) == 0 && live.count(static_cast<char*>(p[6])) == 1);
    void* big = taken(pool, mlkv::kPoolBytes + 1, &got);
    pool.give(0, big, got);
    CHECK(used == 240 * MB);
    CHECK(pool.trim() == 240 * MB && used == 0);
    std::vector<void*> many;
    for (int k = 0; k < mlkv::kPoolBlocks + 5; ++k) many.push_back(taken(pool, 1000, &got));
    for (void* q : many) pool.give(0, q, 1000);
    CHECK(live.size() == (size_t)mlkv::kPoolBlocks);
    CHECK(pool.trim() == 1000u * mlkv::kPoolBlocks && used == 0);
  }
  {  // kept blocks go before any allocation fails
    mlkv::DevicePool pool;
    budget = 300 * MB;
    void* a = taken(pool, 200 * MB, &got);
    pool.give(0, a, got);
    void* b = nullptr;
    CHECK(pool.alloc(&b, 150 * MB) == hipSuccess && used == 150 * MB);
    void* c = taken(pool, 100 * MB, &got);
    pool.give(0, c, got);
    void* d = taken(pool, 140 * MB, &got);
    CHECK(d != nullptr && used == 290 * MB);
    void* e = nullptr;
    CHECK(pool.alloc(&e, 20 * MB) == hipErrorOutOfMemory && e == nullptr);
    for (void* p : {b, d}) (void)hipFree(p);
    budget = ~0ull;
    CHECK(used == 0);
  }
  {  // blocks that ended with a device reset are forgotten, also when their address is in use again
    reset_device();
    mlkv::DevicePool pool;
    void* a = taken(pool, 50 * MB, &got);
    pool.give(0, a, got);
    reset_device();
    void* b = taken(pool, 50 * MB, &got);
    CHECK(b == a && used == 50 * MB);  // new memory, at the old address
    pool.give(0, b, got);
    reset_device();
    void* other = nullptr;
    CHECK(hipMalloc(&other, 50 * MB) == hipSuccess && other == b);  // the program's own
    void* c = taken(pool, 50 * MB, &got);
    CHECK(c != other);
    CHECK(pool.trim() == 0 && live.count(static_cast<char*>(other)) == 1);
    reset_device();
  }
  {  // no block is given to two threads
    mlkv::DevicePool pool;
    std::mutex held_mu;
    std::map<void*, int> held;
    auto work = [&] {
      for (int k = 0; k < 2000; ++k) {
        size_t g = 0;
        void* p = taken(pool, 1 * MB, &g);
        {
          std::lock_guard<std::mutex> lock(held_mu);
          CHECK(p != nullptr && ++held[p] == 1);
        }
        std::this_thread::yield();
        {
          std::lock_guard<std::mutex> lock(held_mu);
          --held[p];
        }
        pool.give(0, p, g);
      }
    };
    std::vector<std::thread> t;
    for (int k = 0; k < 4; ++k) t.emplace_back(work);
    for (auto& x : t) x.join();
    pool.trim();
    CHECK(used == 0 && live.empty());
  }
  CHECK(bad_frees == 0);
  if (failures == 0) std::puts("ok");
  return failures ? 1 : 0;
}
