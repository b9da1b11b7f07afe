// The scratch that a handle keeps for bulk insertion and cleanup, on a GPU with
// little memory: the library's host code with the stand-in launchers and a limit
// on what hipMalloc hands out.  What fits beside a handle that keeps nothing has
// to fit beside one that keeps its scratch.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <map>
#include <mutex>

#include "lsm.h"

static std::mutex g_mu;
static std::map<void*, size_t> g_live;
static size_t g_used = 0, g_limit = ~size_t(0);

extern "C" {
hipError_t __real__Z9hipMallocPPvm(void** p, size_t bytes);
hipError_t __real__Z7hipFreePv(void* p);
hipError_t __wrap__Z9hipMallocPPvm(void** p, size_t bytes) {
  std::lock_guard<std::mutex> lock(g_mu);
  *p = nullptr;
  if (g_used + bytes > g_limit) return hipErrorOutOfMemory;
  const hipError_t e = __real__Z9hipMallocPPvm(p, bytes);
  if (e == hipSuccess) {
    g_live[*p] = bytes;
    g_used += bytes;
  }
  return e;
}
hipError_t __wrap__Z7hipFreePv(void* p) {
  std::lock_guard<std::mutex> lock(g_mu);
  if (p != nullptr) {
    g_used -= g_live[p];
    g_live.erase(p);
  }
  return __real__Z7hipFreePv(p);
}
}

static int g_fail = 0;
#define CHECK(c) \
  do { \
    if (!(c)) { \
      std::fprintf(stderr, "line %d: %s (used %zu of %zu)\n", __LINE__, #c, g_used, g_limit); \
      ++g_fail; \
    } \
  } while (0)

static uint64_t held(lsm_t h) {
  lsm_stats_t st;
  return lsm_get_stats(h, &st) == LSM_OK ? st.device_bytes : 0;
}

int main() {
  const uint32_t b = 4096;
  static uint32_t words[1 << 21];  // the caller's keys and values
  const uint64_t n = sizeof(words) / sizeof(words[0]);

  // Another handle's allocations find the memory that an idle scratch holds.
  {
    lsm_t one = nullptr, two = nullptr;
    CHECK(lsm_create(&one, b, 0, nullptr) == LSM_OK);
    const uint64_t empty = held(one);
    CHECK(lsm_bulk_insert(one, words, words, n) == LSM_OK);
    const uint64_t levels = 2 * n * 4, kept = held(one) - empty - levels;
    CHECK(kept > 4 * n * 4);
    g_limit = g_used + empty / 2;
    CHECK(lsm_create(&two, b, 0, nullptr) == LSM_OK);
    CHECK(held(one) < empty + levels + levels / 8);
    CHECK(lsm_insert_batch(two, words, words, b) == LSM_OK);
    // And the first handle's next call takes it again when there is room.
    g_limit = ~size_t(0);
    CHECK(lsm_cleanup(one, nullptr) == LSM_OK);
    CHECK(held(one) > empty + levels + levels / 2);
    CHECK(lsm_destroy(one) == LSM_OK);
    CHECK(lsm_destroy(two) == LSM_OK);
    CHECK(g_used == 0);
  }

  // A call's levels find the memory that its own, larger scratch holds.
  {
    lsm_t h = nullptr;
    CHECK(lsm_create(&h, b, 0, nullptr) == LSM_OK);
    CHECK(lsm_bulk_insert(h, words, words, n) == LSM_OK);  // level 9
    g_limit = g_used + 64 * b;                             // not enough for level 6
    CHECK(lsm_bulk_insert(h, words, words, 64 * b) == LSM_OK);
    g_limit = ~size_t(0);
    CHECK(lsm_destroy(h) == LSM_OK);
    CHECK(g_used == 0);
  }

  // No more than 2 GiB are kept.
  {
    lsm_t h = nullptr;
    void* keys = nullptr;
    const uint64_t many = 1ull << 27;
    CHECK(hipMalloc(&keys, many * 4) == hipSuccess);
    CHECK(lsm_create(&h, 1u << 16, 0, nullptr) == LSM_OK);
    const uint64_t empty = held(h);
    const uint32_t* k = static_cast<const uint32_t*>(keys);
    CHECK(lsm_bulk_insert(h, k, k, many) == LSM_OK);
    CHECK(held(h) < empty + 2 * many * 4 + (many * 4) / 16);
    CHECK(lsm_destroy(h) == LSM_OK);
    CHECK(hipFree(keys) == hipSuccess);
    CHECK(g_used == 0);
  }
  if (g_fail == 0) std::printf("kept scratch: ok\n");
  return g_fail == 0 ? 0 : 1;
}
