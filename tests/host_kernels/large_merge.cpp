// The merge of runs larger than LDS (merge_large) on the CPU: a work-group of 256
// threads, with the work-group's barrier and a wave's ballot as the only things
// that order them, under ThreadSanitizer.  LDS words that one wave may still read
// while another writes them are reported as a race.  Also checks the output:
// runs with long runs of one key, newest first among equal keys.
#include <hip/hip_runtime.h>
#include <pthread.h>

#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <random>
#include <thread>
#include <vector>

#include "lsm_internal.h"

#define __forceinline__ inline

static pthread_barrier_t g_group, g_wave[lsm::kWaves];
static uint64_t g_bits[lsm::kWaves][64];
struct Dim {
  uint32_t x;
};
static thread_local Dim threadIdx;
static void __syncthreads() { pthread_barrier_wait(&g_group); }
static uint32_t lane_id() { return threadIdx.x & 63u; }
static uint64_t ballot(bool p) {
  const uint32_t w = threadIdx.x >> 6;
  g_bits[w][lane_id()] = p ? 1u : 0u;
  pthread_barrier_wait(&g_wave[w]);
  uint64_t m = 0;
  for (int i = 0; i < 64; ++i) m |= g_bits[w][i] << i;
  pthread_barrier_wait(&g_wave[w]);
  return m;
}
static int __popcll(uint64_t m) { return __builtin_popcountll(m); }
static const uint32_t* as_global(const uint32_t* p) { return p; }

namespace lsm {
#include "kernel_gen.inc"
}  // namespace lsm

static lsm::LocalLds L;

int main() {
  using namespace lsm;
  std::mt19937 rng(3);
  pthread_barrier_init(&g_group, nullptr, kThreads);
  for (auto& b : g_wave) pthread_barrier_init(&b, nullptr, 64);
  long copies = 0;
  for (int round = 0; round < 12; ++round) {
    // Runs of both kinds: one hot key that fills its parts, keys between.
    const int R = 2 + round % 4;
    std::vector<std::vector<uint32_t>> k(R), v(R);
    std::vector<std::pair<uint32_t, uint32_t>> want;  // kv, value
    for (int r = 0; r < R; ++r) {
      const uint32_t n = 300 + rng() % 2500;
      const uint32_t hot = 100 + rng() % 3;
      for (uint32_t i = 0; i < n; ++i) {
        const uint32_t key = rng() % 10 < 7 ? hot : rng() % 400;
        k[r].push_back((key << 1) | (rng() & 1u));
        v[r].push_back(rng());
      }
      std::stable_sort(k[r].begin(), k[r].end(), [](uint32_t a, uint32_t b) { return (a >> 1) < (b >> 1); });
      copies += n;
    }
    for (int r = 0; r < R; ++r)
      for (size_t i = 0; i < k[r].size(); ++i) want.push_back({k[r][i], v[r][i]});
    std::stable_sort(want.begin(), want.end(), [](const auto& a, const auto& b) { return (a.first >> 1) < (b.first >> 1); });
    for (int r = 0; r < R; ++r) {
      L.run_k[r] = k[r].data();
      L.run_v[r] = v[r].data();
      L.cur[r] = 0;
      L.len[r] = static_cast<uint32_t>(k[r].size());
    }
    std::vector<std::pair<uint32_t, uint32_t>> got(want.size());
    std::vector<uint8_t> times(want.size());
    std::vector<std::thread> group;
    for (uint32_t t = 0; t < static_cast<uint32_t>(kThreads); ++t)
      group.emplace_back([&, t] {
        threadIdx.x = t;
        merge_large(L, R, [&](uint32_t x, uint32_t kv, uint32_t val) {
          got[x] = {kv, val};
          ++times[x];
        });
      });
    for (auto& t : group) t.join();
    for (uint8_t c : times)
      if (c != 1) return 1;
    if (got != want) {
      std::fprintf(stderr, "round %d: wrong order\n", round);
      return 1;
    }
  }
  std::printf("large merge: ok, %ld elements\n", copies);
  return 0;
}
