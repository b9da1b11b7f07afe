// The lane walks of counts and emission (count_narrow, emit_narrow) as one lane, on
// the CPU: dictionaries of 1 to 10 levels with keys up to 2^31 - 1, every level in a
// heap array of its own length, so that the sanitizer reports a read past its end.
// Counts and pairs against a search of all levels.  (The walks' ballots only
// decide whether to go on for another lane's sake, so one lane does what each of
// a wave's does.)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <map>
#include <random>
#include <vector>

#include "lsm_internal.h"

#define __forceinline__ inline
static uint64_t ballot(bool p) { return p ? 1 : 0; }
static const uint32_t* as_global(const uint32_t* p) { return p; }

namespace lsm {
#include "kernel_gen.inc"
}  // namespace lsm

int main() {
  using namespace lsm;
  std::mt19937 rng(1);
  uint64_t checked = 0, counted = 0, top_emitted = 0;
  for (int round = 0; round < 200000; ++round) {
    const int count = 1 + static_cast<int>(rng() % kNarrowLevels);
    std::vector<uint32_t*> kv(count), val(count);
    QLevels lv{};
    lv.count = count;
    std::map<uint32_t, std::pair<bool, uint32_t>> newest;  // key -> regular, value
    const uint32_t span = 1 + rng() % 12;
    for (int l = 0; l < count; ++l) {
      const uint32_t n = 1 + rng() % 6;
      std::vector<uint32_t> x(n);
      for (uint32_t& y : x) {
        const uint32_t key = rng() % 8 == 0 ? rng() % 4 : kMaxKey - rng() % span;
        y = (key << 1) | (rng() % 4 != 0 ? 1u : 0u);
      }
      std::stable_sort(x.begin(), x.end(), [](uint32_t a, uint32_t b) { return (a >> 1) < (b >> 1); });
      kv[l] = new uint32_t[n];
      val[l] = new uint32_t[n];
      for (uint32_t i = 0; i < n; ++i) {
        kv[l][i] = x[i];
        val[l][i] = rng();
        newest.emplace(x[i] >> 1, std::make_pair((x[i] & 1u) != 0u, val[l][i]));
      }
      lv.v[l].kv = kv[l];
      lv.v[l].val = val[l];
      lv.v[l].len = n;
    }
    const uint32_t k1 = rng() % 3 == 0 ? 0u : kMaxKey - rng() % (span + 1);
    const uint32_t k2 = rng() % 3 == 0 ? 0xFFFFFFFFu : rng() % 2 == 0 ? kMaxKey : kMaxKey - rng() % span;
    std::vector<std::pair<uint32_t, uint32_t>> want;
    for (const auto& e : newest)
      if (e.first >= k1 && e.first <= k2 && e.second.first) want.push_back({e.first, e.second.second});
    std::vector<uint32_t> cur(64 * count);
    for (int l = 0; l < count; ++l)
      while (cur[l * 64] < lv.v[l].len && (kv[l][cur[l * 64]] >> 1) < k1) ++cur[l * 64];
    std::vector<uint32_t> keys(want.size() + 2, 7u), vals(want.size() + 2, 7u);
    const uint32_t h = ((k2 < kMaxKey ? k2 : kMaxKey) << 1) | 1u;
    uint32_t n = 0;
    const bool done = count <= 3 ? count_narrow<3>(lv, cur.data(), h, rng() % 8, &n)
                                 : count_narrow<kNarrowLevels>(lv, cur.data(), h, rng() % 8, &n);
    if (done && ++counted && n != want.size()) {
      std::fprintf(stderr, "round %d: %u pairs counted, not %zu\n", round, n, want.size());
      return 1;
    }
    if (count <= 6 && count > 3
            ? emit_narrow<6, true>(lv, cur.data(), k2, 1, 1 + want.size(), keys.data(), vals.data())
            : emit_narrow<kNarrowLevels, false>(lv, cur.data(), k2, 1, 1 + want.size(), keys.data(),
                                                vals.data())) {
      ++checked;
      for (size_t i = 0; i < want.size(); ++i) {
        if (keys[1 + i] != want[i].first || vals[1 + i] != want[i].second) {
          std::fprintf(stderr, "round %d: pair %zu is (%u, %u), not (%u, %u)\n", round, i, keys[1 + i],
                       vals[1 + i], want[i].first, want[i].second);
          return 1;
        }
        top_emitted += want[i].first == kMaxKey;
      }
      if (keys[0] != 7u || keys.back() != 7u || vals[0] != 7u || vals.back() != 7u) return 1;
    }
    for (int l = 0; l < count; ++l) {
      delete[] kv[l];
      delete[] val[l];
    }
  }
  std::printf("narrow walk: ok, %llu walks and %llu counts, key 2^31 - 1 in %llu\n",
              static_cast<unsigned long long>(checked), static_cast<unsigned long long>(counted),
              static_cast<unsigned long long>(top_emitted));
  return checked > 100000 && counted > 100000 && top_emitted > 10000 ? 0 : 1;
}
