// Bulk insertions whose parts lie on both sides of the largest digit-pass sort
// that counts into the global histogram, on the CPU: the library's host code with
// the stand-in launchers, and every sort's use of the histogram's two buffers
// followed as the kernels use them.  A sort that counts adds to hist[parity],
// which has to be all zero, and clears the other buffer; a larger one touches
// neither.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <cstring>
#include <initializer_list>

#include "lsm.h"
#include "lsm_internal.h"

static long g_counted = 0, g_large = 0, g_dirty = 0;

#define LAUNCH_SORT _ZN3lsm11launch_sortERKNS_8SortArgsEP12ihipStream_tPKNS_6KTimerEPi
#define NAME2(a, b) a##b
#define NAME(a, b) NAME2(a, b)
extern "C" {
hipError_t NAME(__real_, LAUNCH_SORT)(const lsm::SortArgs&, hipStream_t, const lsm::KTimer*, int*);
hipError_t NAME(__wrap_, LAUNCH_SORT)(const lsm::SortArgs& a, hipStream_t s, const lsm::KTimer* t,
                                      int* launched) {
  using namespace lsm;
  constexpr uint32_t kWords = kMaxPasses * kRadix;
  uint32_t* mine = a.meta.hist + static_cast<uint64_t>(a.meta.parity) * kWords;
  uint32_t* other = a.meta.hist + static_cast<uint64_t>(a.meta.parity ^ 1) * kWords;
  const bool counts =
      a.path == kSortLsd && a.meta.num_sort_tiles <= static_cast<uint32_t>(kMsdMaxTiles);
  uint32_t before[2 * kWords];
  std::memcpy(before, a.meta.hist, sizeof(before));
  const hipError_t e = NAME(__real_, LAUNCH_SORT)(a, s, t, launched);
  std::memcpy(a.meta.hist, before, sizeof(before));  // what the stand-in touched
  g_large += a.path == kSortLsd && !counts;
  if (counts) {
    ++g_counted;
    for (uint32_t i = 0; i < kWords; ++i)
      if (mine[i] != 0u) {
        ++g_dirty;
        break;
      }
    std::memset(other, 0, kWords * sizeof(uint32_t));
    for (uint32_t i = 0; i < kWords; ++i) mine[i] += a.src.b / kRadix + 1u;
  }
  return e;
}
}

int main() {
  // Batch size, batches before, batches in the call: 16 tiles a batch at 2^15.
  const uint32_t b = 1u << 15;
  for (uint64_t r0 : {0ull, 1ull, 7ull, 31ull, 63ull, 64ull, 100ull}) {
    for (uint64_t k : {1ull, 3ull, 16ull, 33ull, 49ull, 50ull, 120ull}) {
      lsm_t h = nullptr;
      void* keys = nullptr;
      if (lsm_create(&h, b, 0, nullptr) != LSM_OK) return 1;
      if (hipMalloc(&keys, k * b * sizeof(uint32_t)) != hipSuccess) return 1;
      const uint32_t* p = static_cast<const uint32_t*>(keys);
      if (lsm_set_sort_path(h, LSM_SORT_DIGIT_PASSES) != LSM_OK) return 1;
      for (uint64_t i = 0; i < r0; ++i)
        if (lsm_insert_batch(h, p, p, b) != LSM_OK) return 1;
      for (int twice = 0; twice < 2; ++twice)
        if (lsm_bulk_insert(h, p, p, k * b) != LSM_OK) return 1;
      if (lsm_num_batches(h) != r0 + 2 * k || lsm_destroy(h) != LSM_OK) return 1;
      (void)hipFree(keys);
    }
  }
  std::printf("histogram: %ld sorts counted, %ld larger, %ld began with counts left over\n", g_counted,
              g_large, g_dirty);
  return g_dirty == 0 && g_counted > 1000 && g_large > 20 ? 0 : 1;
}
