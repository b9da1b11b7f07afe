// The walk back to the start of a key's run (run_start) on the CPU: runs of 1 to 300
// elements at the front, in the middle and at the end of a level, from each of
// their elements, the level in a heap array of its own length.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>

#include "lsm_internal.h"

#define __forceinline__ inline
static const uint32_t* as_global(const uint32_t* p) { return p; }

namespace lsm {
#include "kernel_gen.inc"
}  // namespace lsm

int main() {
  for (uint32_t run = 1; run <= 300; ++run) {
    for (uint32_t before = 0; before < 5; ++before) {
      const uint32_t n = before + run + before;
      uint32_t* kv = new uint32_t[n];
      for (uint32_t i = 0; i < n; ++i) {
        const uint32_t key = i < before ? i : i < before + run ? 100u : 200u + i;
        kv[i] = (key << 1) | (i & 1u);
      }
      for (uint32_t c = before; c < before + run; ++c) {
        if (lsm::run_start(kv, c, 100u) != before) {
          std::fprintf(stderr, "run of %u after %u, from %u\n", run, before, c);
          return 1;
        }
      }
      delete[] kv;
    }
  }
  std::printf("run start: ok\n");
  return 0;
}
