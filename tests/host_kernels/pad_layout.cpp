// Where padding and digit counts live, on the CPU.  For batch sizes across tile
// edges and both sides of 256 tiles: every slot's padding element lies inside the
// sort scratch, on a 16-byte boundary, apart from every other region of any slot;
// and the counts and totals of digit passes above 256 tiles fit the look-back
// words that they are kept in, for every number of tiles.  Then, with the
// library's host code and the stand-in launchers: every bucket sort is told of
// each of its batches what the batch's scatter was told (its elements, and the
// place of its padding element), and the number of copies over the group.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <initializer_list>
#include <map>
#include <random>
#include <vector>

#include "lsm.h"
#include "lsm_internal.h"

namespace lsm {
#include "kernel_gen.inc"
}  // namespace lsm

using namespace lsm;

static int g_fail = 0;
#define CHECK(c) \
  do { \
    if (!(c) && g_fail++ < 20) std::fprintf(stderr, "line %d: %s\n", __LINE__, #c); \
  } while (0)

static std::map<const uint32_t*, uint32_t> g_scattered;  // padding element -> the batch's elements
static long g_sorts = 0, g_padded = 0;
static uint32_t g_b = 0;

static void scattered(const SortArgs& a) { g_scattered[a.meta.pad] = a.src.n; }
static void sorted(const SortArgs& a) {
  ++g_sorts;
  uint32_t pads = 0;
  CHECK(a.group >= 1 && a.group <= static_cast<uint32_t>(kMaxGroup));
  for (uint32_t q = 0; q < a.group; ++q) {
    CHECK(g_scattered.count(a.grp_pad[q]) == 1 && g_scattered[a.grp_pad[q]] == a.grp_real[q]);
    CHECK(a.grp_real[q] >= 1 && a.grp_real[q] <= g_b);
    CHECK(a.grp_pad[q] == a.grp_n[q] + kTopBuckets);  // of the same slot
    pads += g_b - a.grp_real[q];
    g_scattered.erase(a.grp_pad[q]);
  }
  CHECK(a.pads == pads && a.pad_shift == sort_top_shift(a));
  g_padded += pads != 0;
}

extern "C" {
hipError_t __real__ZN3lsm14launch_scatterERKNS_8SortArgsEP12ihipStream_tPKNS_6KTimerE(
    const SortArgs&, hipStream_t, const KTimer*);
hipError_t __wrap__ZN3lsm14launch_scatterERKNS_8SortArgsEP12ihipStream_tPKNS_6KTimerE(
    const SortArgs& a, hipStream_t s, const KTimer* t) {
  scattered(a);
  return __real__ZN3lsm14launch_scatterERKNS_8SortArgsEP12ihipStream_tPKNS_6KTimerE(a, s, t);
}
hipError_t __real__ZN3lsm14launch_bucketsERKNS_8SortArgsEP12ihipStream_tPKNS_6KTimerE(
    const SortArgs&, hipStream_t, const KTimer*);
hipError_t __wrap__ZN3lsm14launch_bucketsERKNS_8SortArgsEP12ihipStream_tPKNS_6KTimerE(
    const SortArgs& a, hipStream_t s, const KTimer* t) {
  sorted(a);
  return __real__ZN3lsm14launch_bucketsERKNS_8SortArgsEP12ihipStream_tPKNS_6KTimerE(a, s, t);
}
hipError_t __real__ZN3lsm16launch_sort_stepERKNS_8SortArgsES2_P12ihipStream_tPKNS_6KTimerE(
    const SortArgs&, const SortArgs&, hipStream_t, const KTimer*);
hipError_t __wrap__ZN3lsm16launch_sort_stepERKNS_8SortArgsES2_P12ihipStream_tPKNS_6KTimerE(
    const SortArgs& bk, const SortArgs& sc, hipStream_t s, const KTimer* t) {
  sorted(bk);
  scattered(sc);
  return __real__ZN3lsm16launch_sort_stepERKNS_8SortArgsES2_P12ihipStream_tPKNS_6KTimerE(bk, sc, s, t);
}
}

int main() {
  // The scratch layout.
  for (uint32_t b : {1u, 2u, 2047u, 2048u, 2049u, 65536u, 1u << 18, (1u << 19) - 1u, 1u << 19,
                     (1u << 19) + 1u, 1u << 20, 50000000u}) {
    const uint64_t words = sort_meta_words(b);
    uint32_t* const base = reinterpret_cast<uint32_t*>(uintptr_t(1) << 20);
    struct Region {
      uint64_t at, len;
    };
    std::vector<Region> all, pads;
    for (int slot = 0; slot < kSortSlots; ++slot) {
      const SortMeta m = sort_meta_carve(base, b, 0, slot);
      const uint64_t ns = m.num_sort_tiles;
      if (slot == 0) {
        all.push_back({static_cast<uint64_t>(m.hist - base), 2ull * kMaxPasses * kRadix});
        all.push_back({static_cast<uint64_t>(m.status - base), kMaxPasses * ns * kRadix});
        all.push_back({static_cast<uint64_t>(m.tile_ctr - base), kMaxPasses});
        all.push_back({static_cast<uint64_t>(m.err - base), 4});
      }
      all.push_back({static_cast<uint64_t>(m.tile_cnt - base), ns * (kTopBuckets / 2)});
      all.push_back({static_cast<uint64_t>(m.bucket_n - base), kTopBuckets});
      pads.push_back({static_cast<uint64_t>(m.pad - base), 4});
      CHECK(reinterpret_cast<uintptr_t>(m.pad) % 16 == 0);
    }
    all.insert(all.end(), pads.begin(), pads.end());
    for (size_t i = 0; i < all.size(); ++i) {
      CHECK(all[i].at + all[i].len <= words);
      for (size_t j = i + 1; j < all.size(); ++j)
        CHECK(all[i].at + all[i].len <= all[j].at || all[j].at + all[j].len <= all[i].at);
    }
  }
  // Counts of the larger digit passes; every tile is in one group.
  for (uint64_t tiles = kMsdMaxTiles + 1; tiles < 40000; ++tiles) {
    for (uint64_t b : {tiles * kSortTile, tiles * kSortTile - kSortTile + 1}) {
      const LsdGrid g = lsd_grid(static_cast<uint32_t>(b));
      CHECK(g.groups <= kLsdMaxGroups && static_cast<uint64_t>(kRadix) * g.groups + kRadix <=
                                             static_cast<uint64_t>(kMaxPasses) * tiles * kRadix);
      const uint64_t chunk = static_cast<uint64_t>(g.tiles_per_group) * kLsdTile;
      CHECK(g.groups * chunk >= b && (g.groups - 1) * chunk < b);
    }
  }
  // What the host tells the launchers.
  std::mt19937 rng(5);
  for (uint32_t b : {2u, 4096u, 70000u}) {
    g_b = b;
    static uint32_t words[70000];
    static uint8_t flags[70000];
    for (int group : {1, 2, 4}) {
      lsm_t h = nullptr;
      CHECK(lsm_create(&h, b, 0, nullptr) == LSM_OK && lsm_set_grouping(h, group) == LSM_OK);
      CHECK(lsm_set_sort_path(h, LSM_SORT_TOP_DIGIT) == LSM_OK);
      g_scattered.clear();
      for (int i = 0; i < 300; ++i) {
        const uint32_t n = rng() % 3 == 0 ? b : 1 + rng() % b;
        switch (rng() % 6) {
          case 0: CHECK(lsm_delete_batch(h, words, n) == LSM_OK); break;
          case 1: CHECK(lsm_update_batch(h, words, words, flags, n) == LSM_OK); break;
          case 2: CHECK(lsm_submit(h, words, words, n, 0) == LSM_OK); break;
          case 3: CHECK(lsm_flush(h) == LSM_OK); break;
          default: CHECK(lsm_insert_batch(h, words, words, n) == LSM_OK);
        }
      }
      CHECK(lsm_flush(h) == LSM_OK);
      CHECK(g_scattered.empty());  // every scattered batch was sorted
      CHECK(lsm_destroy(h) == LSM_OK);
    }
  }
  CHECK(g_sorts > 500 && g_padded > 300);
  if (g_fail == 0) std::printf("padding and digit counts: ok, %ld sorts, %ld padded\n", g_sorts, g_padded);
  return g_fail == 0 ? 0 : 1;
}
