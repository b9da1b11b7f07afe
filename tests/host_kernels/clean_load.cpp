// Cleanup's loads of a thread's eight elements (clean_load) on the CPU, at both ends
// of lists of every length near a multiple of eight, up to the longest list, whose
// last thread starts at element 2^32 - 8.  Only the end of a list exists, in a heap
// array of its own, so that the sanitizer reports a read past it.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <initializer_list>

#include "lsm_internal.h"

#define __forceinline__ inline
struct alignas(16) uint4 {
  uint32_t x, y, z, w;
};

namespace lsm {
#include "kernel_gen.inc"
}  // namespace lsm

int main() {
  using namespace lsm;
  for (uint64_t top : {uint64_t(8), uint64_t(4096), uint64_t(1) << 31, uint64_t(1) << 32}) {
    for (uint32_t less = 0; less < 10; ++less) {
      if (top - less > 0xFFFFFFFFull || less >= top) continue;
      const uint32_t n = static_cast<uint32_t>(top - less);
      const uint32_t e0 = static_cast<uint32_t>((n - 1u) & ~7u), m = n - e0;
      uint32_t* end = new uint32_t[m];
      for (uint32_t i = 0; i < m; ++i) end[i] = i + 1u;
      const uint32_t* list =
          reinterpret_cast<const uint32_t*>(reinterpret_cast<uintptr_t>(end) - 4ull * e0);
      uint32_t x[kCleanItems];
      clean_load(list, n, e0, x);
      for (uint32_t i = 0; i < 8; ++i) {
        if (x[i] != (i < m ? i + 1u : 0u)) {
          std::fprintf(stderr, "n %u: element %u of the last thread\n", n, i);
          return 1;
        }
      }
      delete[] end;
    }
  }
  std::printf("clean load: ok\n");
  return 0;
}
