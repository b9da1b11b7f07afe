// gfx950 kernels of the batched LSM dictionary.
//
// Most kernels run in work-groups of four wave64 waves.  Nothing here is a
// dense contraction, so there is no MFMA: the batch sort and the level
// merges are HBM/L2 streams, the searches are random-access.
//
//   k_sort_hist / k_sort_pass : stable LSD radix sort of one batch (the
//       "sort the batch" step of sec. III-B / Fig. 2(a)): one histogram
//       kernel, then one counting pass per 8-bit digit with decoupled
//       look-back (k_lsd_up / k_lsd_scan / k_lsd_down: a pass over more than
//       256 tiles, with none).  The batch is read back to front, so among equal key
//       variables the later batch position comes first (the last duplicate
//       wins), and padded with copies of its last element (sec. IV-A).
//   k_msd_scatter / k_local_sort : the same stable order for batches of at
//       most 256 tiles: each tile grouped by its top digit in place, then one
//       work-group gathers and sorts each top-digit bucket in LDS (k_sort_step:
//       that beside the grouping of a later batch).
//   Every kernel that writes a level also writes its fences (the original
//       key of every 32nd element), which the searches use first.
//   k_merge : merge of a newer run with an older run on the original key,
//       the newer element first on equal keys (sec. IV-A), merge-path
//       partitioned with a 64-ary wave search.
//   k_lookup : per-query lower bound over the occupied levels, newest first,
//       stopping at the first hit (sec. III-D, IV-B).  k_lookup_few and
//       k_count_few : the same for few queries, the levels dealt to the waves.
//   k_count / k_range_emit : per-query bounds in every occupied level and a
//       merge of the per-level candidate runs in level order, keeping the
//       first element of each key run when it is a regular element
//       (sec. III-E, IV-C, IV-D), eight lanes a query or, where every query of
//       a wave has few candidates, one.  k_range_emit_one : the emission with one
//       occupied level, a wave copying one query's candidates at a time.
//   k_scan : single-pass exclusive scan with decoupled look-back for the
//       range output offsets (stage 2 of sec. IV-C).
//   k_successor / k_predecessor : the order queries of the sec. I-B
//       footnote, the same walk as count stopped at the first live key.
//   k_clean_count / k_clean_scatter / k_clean_pad : cleanup (sec. III-E,
//       IV-D) after the levels are merged: mark stale elements, compact the
//       valid ones straight into the new levels, pad with placebos.
#include <hip/hip_ext.h>

#include "lsm_internal.h"

#include <mutex>
#include <type_traits>

namespace lsm {
namespace {

// ------------------------------------------------------------ wave helpers
__device__ __forceinline__ uint32_t lane_id() {
  return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}
// Number of set bits of m below this lane.
__device__ __forceinline__ uint32_t count_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32),
                                   __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u));
}
__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// Inclusive scan over the wave (every lane active).  Within each row of 16
// lanes, four DPP row shifts by 1, 2, 4 and 8 (lanes shifted in from outside
// the row read 0); then each row adds the totals of the rows below it, read
// from lanes 15, 31 and 47.
template <int kCtrl>
__device__ __forceinline__ uint32_t dpp_row_shr(uint32_t x) {
  return static_cast<uint32_t>(
      __builtin_amdgcn_update_dpp(0, static_cast<int>(x), kCtrl, 0xf, 0xf, true));
}
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x, uint32_t lane) {
  x += dpp_row_shr<0x111>(x);  // row_shr:1
  x += dpp_row_shr<0x112>(x);  // row_shr:2
  x += dpp_row_shr<0x114>(x);  // row_shr:4
  x += dpp_row_shr<0x118>(x);  // row_shr:8
  const uint32_t r0 = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(x), 15));
  const uint32_t r1 = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(x), 31));
  const uint32_t r2 = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(x), 47));
  const uint32_t row = lane >> 4;
  return x + (row > 0 ? r0 : 0u) + (row > 1 ? r1 : 0u) + (row > 2 ? r2 : 0u);
}
__device__ __forceinline__ uint64_t wave_incl_scan64(uint64_t x, uint32_t lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    uint64_t y = __shfl_up(x, o, 64);
    if (lane >= static_cast<uint32_t>(o)) x += y;
  }
  return x;
}
__device__ __forceinline__ uint64_t wave_sum64(uint64_t x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// Exclusive scan over the work-group, one value per thread.  tmp holds
// kWaves words; the call contains two barriers.
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t x, uint32_t* tmp) {
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t inc = wave_incl_scan(x, lane);
  if (lane == 63) tmp[wave] = inc;
  __syncthreads();
  uint32_t pre = 0;
  for (uint32_t w = 0; w < wave; ++w) pre += tmp[w];
  __syncthreads();
  return pre + inc - x;
}

// Two exclusive scans over the work-group in one pass (the barriers of one).
// tmp holds 2 kWaves words.
__device__ __forceinline__ void block_excl_scan2(uint32_t& x, uint32_t& y, uint32_t* tmp) {
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t ix = wave_incl_scan(x, lane), iy = wave_incl_scan(y, lane);
  if (lane == 63) {
    tmp[wave] = ix;
    tmp[kWaves + wave] = iy;
  }
  __syncthreads();
  uint32_t px = 0, py = 0;
  for (uint32_t w = 0; w < wave; ++w) {
    px += tmp[w];
    py += tmp[kWaves + w];
  }
  __syncthreads();
  x = px + ix - x;
  y = py + iy - y;
}

// Writes the largest of the work-group's 256 per-thread values to *out
// (thread 0).  tmp holds kWaves words; two barriers, so the whole
// work-group must call it.
__device__ void record_max(uint32_t x, uint32_t* out, uint32_t* tmp) {
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = max(x, static_cast<uint32_t>(__shfl_xor(x, o, 64)));
  if (lane == 0) tmp[wave] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t r = tmp[0];
    for (int w = 1; w < kWaves; ++w) r = max(r, tmp[w]);
    *out = r;
  }
  __syncthreads();
}

// What is recorded of a bucket of n elements that is not known to be large
// because of one key: above the top-digit sort's limit when it outgrows LDS.
__device__ __forceinline__ uint32_t large_bucket(uint32_t n) {
  return n > static_cast<uint32_t>(kLocalCap) ? max(n, kMsdMaxBucket + 1) : n;
}

// Device-scope relaxed atomics for the look-back words: each word carries
// its own payload, so no other memory needs ordering with it.
__device__ __forceinline__ uint32_t ld_dev(const uint32_t* p) {
  return __hip_atomic_load(const_cast<uint32_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_dev(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t ld_dev64(const uint64_t* p) {
  return __hip_atomic_load(const_cast<uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_dev64(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// A pointer known to address global memory (loads through it are global,
// not flat, loads).
__device__ __forceinline__ const __attribute__((address_space(1))) uint32_t* as_global(
    const uint32_t* p) {
  return (const __attribute__((address_space(1))) uint32_t*)(p);
}


// ------------------------------------------------------------ searches
// Sum over the eight lanes of an octet (lanes 8o .. 8o + 7), in every lane
// of it: DPP swaps with lane ^ 1 and lane ^ 2, then the half-row mirror
// (lane i with lane 7 - i inside each group of eight).  Every lane of the
// octet must be active.
__device__ __forceinline__ uint32_t octet_sum(uint32_t x) {
  x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0xB1, 0xf, 0xf, true));
  x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x4E, 0xf, 0xf, true));
  x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x141, 0xf, 0xf, true));
  return x;
}

// The upper part of every occupied level's fence tree in LDS: of each level the
// lowest tree level that has at most `cap` entries, the levels' parts one
// after another, each in whole blocks of 64 words.  A search then
// starts there with a binary search of its own lane and reads only the tree
// levels below from memory: with ten levels of 2^16 .. 2^25 elements 24
// lines a query instead of 45.  cap is halved from kTopEntries until all parts
// fit (at most kTopWords, 16 KB: with 32 KB lookups are no faster and the order queries,
// which keep cursors beside the tops, take 356 us instead of 262).
constexpr uint32_t kTopEntries = 2048;
constexpr uint32_t kTopWords = 4096;
static_assert(kMaxLevels * 64 <= kTopWords, "32 levels of at most 32 entries always fit");

// The occupied levels as the query kernels take them, newest first: what a
// search reads of a level stands together (one or two cache lines of the
// kernel's arguments, which every launch reads afresh).
struct QLevel {
  const uint32_t* kv;
  const uint32_t* val;
  const uint32_t* fence;
  uint32_t len;
  uint32_t top_at;   // first LDS word of the level's top
  uint32_t top_cnt;  // its entries
  uint32_t top_off;  // where the tree level above which the search starts ends
  uint32_t top_t;    // and which one it is
};
struct QLevels {
  int count;
  uint32_t words;  // LDS words of all tops
  QLevel v[kMaxLevels];
};
// words: the most LDS words for the tops; 0 for none (every search then starts
// at the root).
inline QLevels query_levels(const LevelSet& lv, uint32_t words) {
  QLevels s{};
  s.count = lv.count;
  for (uint64_t cap = words == 0 ? 32 : kTopEntries;; cap /= 2) {
    s.words = 0;
    for (int l = 0; l < lv.count; ++l) {
      uint64_t off = 0, c = (static_cast<uint64_t>(lv.len[l]) + 31) / 32;
      uint32_t t = 1;
      while (c > cap) {
        off += fence_pad(c);
        c = (c + 31) / 32;
        ++t;
      }
      QLevel& q = s.v[l];
      q.kv = lv.kv[l];
      q.val = lv.val[l];
      q.fence = lv.fence[l];
      q.len = lv.len[l];
      if (words == 0) {
        q.top_off = static_cast<uint32_t>(off + fence_pad(c));
        q.top_t = t + 1;
        continue;
      }
      q.top_at = s.words;
      q.top_cnt = static_cast<uint32_t>(c);
      q.top_off = static_cast<uint32_t>(off);
      q.top_t = t;
      s.words += (static_cast<uint32_t>(c) + 63u) & ~63u;
    }
    if (s.words <= words || cap <= 32) return s;
  }
}

// Entry i of a part stands at word i with its low six bits exclusive-ored by
// its block: the probes of a binary search are multiples of a power of two
// apart, which would all fall on one LDS bank.
__device__ __forceinline__ uint32_t top_word(uint32_t i) { return i ^ ((i >> 6) & 63u); }

// Loads every part (all threads of the work-group; kN waves).  The blocks of
// 64 words are dealt to the waves in turn, eight in flight.
template <int kN>
__device__ __forceinline__ void load_tops(const QLevels& lv, uint32_t* top) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wave = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
  const uint32_t blocks = lv.words >> 6;
  for (uint32_t b0 = wave; b0 < blocks; b0 += 8 * kN) {
    uint32_t v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint32_t blk = b0 + u * kN;
      v[u] = 0u;
      if (blk < blocks) {
        int l = 0;
        while (l + 1 < lv.count && lv.v[l + 1].top_at <= blk * 64u) ++l;
        const uint32_t i = blk * 64u - lv.v[l].top_at + lane;
        if (i < lv.v[l].top_cnt) v[u] = lv.v[l].fence[lv.v[l].top_off + i];
      }
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint32_t blk = b0 + u * kN;
      if (blk < blocks) {
        int l = 0;
        while (l + 1 < lv.count && lv.v[l + 1].top_at <= blk * 64u) ++l;
        top[lv.v[l].top_at + top_word(blk * 64u - lv.v[l].top_at + lane)] = v[u];
      }
    }
  }
  __syncthreads();
}

// Number of the cnt entries of a part that are < k (upper: <= k).
template <bool kUpper>
__device__ __forceinline__ uint32_t top_count(const uint32_t* part, uint32_t cnt, uint32_t k) {
  uint32_t p = 0;
  for (uint32_t step = 1u << (31 - __builtin_clz(cnt)); step > 0; step >>= 1) {
    const uint32_t q = p + step;
    const uint32_t x = part[top_word((q < cnt ? q : cnt) - 1u)];
    p = (q <= cnt && (kUpper ? x <= k : x < k)) ? q : p;
  }
  return p;
}

// x of lane j of the octet, in all eight lanes.
template <int kJ>
__device__ __forceinline__ uint32_t octet_lane(uint32_t x) {
  return static_cast<uint32_t>(
      __builtin_amdgcn_ds_swizzle(static_cast<int>(x), (kJ << 5) | 0x18));
}
__device__ __forceinline__ void octet_lanes(uint32_t x, uint32_t (&q)[8]) {
  q[0] = octet_lane<0>(x);
  q[1] = octet_lane<1>(x);
  q[2] = octet_lane<2>(x);
  q[3] = octet_lane<3>(x);
  q[4] = octet_lane<4>(x);
  q[5] = octet_lane<5>(x);
  q[6] = octet_lane<6>(x);
  q[7] = octet_lane<7>(x);
}

// Lower / upper bound of original key k in a level of n elements through its fence
// tree: the first index whose original key is >= k (upper: > k), or n.  For a whole
// wave at once, from the level's part of the LDS tops on: each lane counts its own
// key there, then the eight lanes of an octet search the octet's eight queries
// together: at every tree level lane s of the
// octet reads bytes 16 s .. 16 s + 15 of each of the eight queries' 128-byte
// lines, so a load instruction of the wave reads eight whole lines instead of
// 64 scattered 16-byte pieces of 64 lines (a per-lane search keeps the texture
// addresser busy nearly all the time).  Entry counts are summed over the
// octet.  kq: the octet's keys (octet_lanes of k).  Each lane passes its own
// key and receives its own bound; every lane of the wave must call it (lanes
// without a query pass any key and ignore the result).  With kFind, *hit
// receives whether the element at the bound can hold key k: exactly, or true
// when it stands in the next line (one time in 32).
template <bool kTop, bool kUpper, bool kFind>
__device__ __forceinline__ uint32_t octet_bound(const QLevels& lv,
                                                const uint32_t* top, int l, uint32_t k,
                                                const uint32_t (&kq)[8], bool* hit) {
  static_assert(!kUpper || !kFind, "the bound of a key that is looked for is the lower one");
  const uint32_t lane = lane_id(), sub = lane & 7u;
  const uint32_t n = lv.v[l].len;
  if (n == 0) {
    if (kFind) *hit = false;
    return 0u;
  }
  uint32_t g[8];
  if constexpr (kTop) {
    octet_lanes(top_count<kUpper>(top + lv.v[l].top_at, lv.v[l].top_cnt, k), g);
  } else {  // no tops: from the root, which is the first line of its tree level
#pragma unroll
    for (int j = 0; j < 8; ++j) g[j] = 1u;
  }
  const uint32_t* tree = lv.v[l].fence;
  uint32_t off = lv.v[l].top_off;
  // A tree level's answer lies in the line that starts at its parent's entry
  // g - 1; the line's first entry qualifies with its parent, and with g = 0
  // no entry of line 0 qualifies, so a plain count serves both.
  for (uint32_t t = lv.v[l].top_t - 1; t >= 1; --t) {
    const uint32_t ct = static_cast<uint32_t>((static_cast<uint64_t>(n) + (1ull << (5 * t)) - 1) >> (5 * t));
    off -= static_cast<uint32_t>(fence_pad(ct));
    const uint32_t* line = tree + off + 4u * sub;
    uint4 w[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      g[j] = g[j] > 0 ? (g[j] - 1u) * 32u : 0u;  // the line's first entry
      w[j] = *reinterpret_cast<const uint4*>(line + g[j]);
    }
    if ((ct & 31u) == 0) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const uint32_t e4[4] = {w[j].x, w[j].y, w[j].z, w[j].w};
        uint32_t cnt = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) cnt += (kUpper ? e4[r] <= kq[j] : e4[r] < kq[j]) ? 1u : 0u;
        g[j] += octet_sum(cnt);
      }
    } else {  // the last line is partly filled
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const uint32_t e4[4] = {w[j].x, w[j].y, w[j].z, w[j].w};
        uint32_t cnt = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          cnt += (g[j] + 4u * sub + r < ct && (kUpper ? e4[r] <= kq[j] : e4[r] < kq[j])) ? 1u : 0u;
        g[j] += octet_sum(cnt);
      }
    }
  }
  // The level's own line.  Key variables are compared whole: below 2 k, or at
  // most 2 k + 1.  (Keys from 2^31 on are above every element.)
  const uint32_t* kv = lv.v[l].kv;
  uint4 w[8];
  if ((n & 31u) == 0) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      g[j] = g[j] > 0 ? (g[j] - 1u) * 32u : 0u;
      w[j] = *reinterpret_cast<const uint4*>(kv + g[j] + 4u * sub);
    }
  } else {  // the last line may be partial: read what exists
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      g[j] = g[j] > 0 ? (g[j] - 1u) * 32u : 0u;
      const uint32_t i0 = g[j] + 4u * sub;
      if (i0 + 4u <= n) {
        w[j] = *reinterpret_cast<const uint4*>(kv + i0);
      } else {
        w[j].x = i0 < n ? kv[i0] : 0u;
        w[j].y = i0 + 1u < n ? kv[i0 + 1u] : 0u;
        w[j].z = i0 + 2u < n ? kv[i0 + 2u] : 0u;
        w[j].w = 0u;
      }
    }
  }
  uint32_t res = 0;
  bool h = false;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const uint32_t e4[4] = {w[j].x, w[j].y, w[j].z, w[j].w};
    const uint32_t kl = kq[j] << 1, ku = kl | 1u;
    uint32_t lt = 0, le = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool in = (n & 31u) == 0 || g[j] + 4u * sub + r < n;
      if (!kUpper) lt += (in && e4[r] < kl) ? 1u : 0u;
      if (kUpper || kFind) le += (in && e4[r] <= ku) ? 1u : 0u;
    }
    const uint32_t sum = octet_sum(kUpper ? le : kFind ? (lt | (le << 16)) : lt);
    if (sub == static_cast<uint32_t>(j)) {
      res = g[j] + (kFind ? sum & 0xFFFFu : sum);
      if (kFind) h = (sum >> 16) != (sum & 0xFFFFu) || (sum & 0xFFFFu) == 32u;
    }
  }
  if (k > 0x7FFFFFFFu) {
    res = n;
    h = false;
  }
  if (kFind) *hit = h;
  return res;
}

// Records output position o of a level of n elements in the level's fence
// tree: in tree level t when o is a multiple of 32^t.
__device__ __forceinline__ void put_fence(uint32_t* tree, uint64_t n, uint64_t o, uint32_t kv) {
  if (tree == nullptr || (o & 31u) != 0) return;
  const uint32_t key = kv >> 1;
  uint64_t off = 0, c = (n + 31) / 32, q = o >> 5;
  for (;;) {
    tree[off + q] = key;
    if (c <= 32 || (q & 31u) != 0) break;
    off += fence_pad(c);
    c = (c + 31) / 32;
    q >>= 5;
  }
}

// ------------------------------------------------------------ radix sort
constexpr uint32_t kFlagAgg = 1u << 30;  // tile aggregate published
constexpr uint32_t kFlagInc = 2u << 30;  // inclusive prefix published
constexpr uint32_t kCountMask = (1u << 30) - 1;

// Every device-side wait is bounded: after kSpinLimit polls the waiter
// records kFaultTimeout in the fault word and stops waiting; writes whose
// position could then be wrong are skipped, so a broken protocol can give
// wrong results (reported by lsm_sync) but never hangs or writes out of
// bounds.  A correct run never reaches the limit: every tile a look-back
// waits for has already started.
constexpr uint32_t kSpinLimit = 1u << 24;
constexpr uint32_t kFaultTimeout = 2u;

// One thread's kN items of the tile starting at tb (positions tile_pos).
// Element e of the batch as the sort sees it: read back to front and padded
// with copies of the caller's last element, so e = 0 .. b-n-1 are padding and
// e = b-n .. b-1 are the caller's elements n-1 .. 0.  Written so that the
// tile's loads are all in flight together.  Every load is issued unconditionally (the source index is
// clamped, so each address is in bounds; deletions read their values from the
// keys and drop them), only a mixed batch's flags sit behind a branch (on the
// batch mode, uniform), and the key variables are formed afterwards.  Items
// at or past b are invalid and read as 0.
template <int kN>
__device__ __forceinline__ void tile_items(const BatchSrc& s, uint32_t tb, uint32_t wave,
                                           uint32_t lane, uint32_t (&kv)[kN], uint32_t (&val)[kN],
                                           uint32_t (&key)[kN], bool (&valid)[kN]) {
  const uint32_t* vp = s.vals != nullptr ? s.vals : s.keys;
  uint32_t src[kN], rk[kN], rv[kN], st[kN];
#pragma unroll
  for (int i = 0; i < kN; ++i) {
    const uint32_t e = tb + wave * 64 * kN + static_cast<uint32_t>(i) * 64 + lane;
    valid[i] = e < s.b;
    const uint32_t x = s.b - 1 - e;
    src[i] = x < s.n - 1 ? x : s.n - 1;
  }
#pragma unroll
  for (int i = 0; i < kN; ++i) rk[i] = s.keys[src[i]];
#pragma unroll
  for (int i = 0; i < kN; ++i) rv[i] = vp[src[i]];
  if (s.mode == kMixed) {
#pragma unroll
    for (int i = 0; i < kN; ++i) st[i] = s.is_delete[src[i]] ? 0u : 1u;
  } else {
    const uint32_t c = s.mode == kDelete ? 0u : 1u;
#pragma unroll
    for (int i = 0; i < kN; ++i) st[i] = c;
  }
  const bool enc = s.mode == kEncoded;
#pragma unroll
  for (int i = 0; i < kN; ++i) {
    const uint32_t x = enc ? rk[i] : ((rk[i] << 1) | st[i]);
    const uint32_t v = (enc || st[i] != 0u) ? rv[i] : 0u;  // tombstones carry value 0
    kv[i] = valid[i] ? x : 0u;
    val[i] = valid[i] ? v : 0u;
    key[i] = valid[i] ? (enc ? rk[i] >> 1 : rk[i]) : 0u;
  }
}

struct SortLds {
  uint32_t kv[kSortTile];
  uint32_t val[kSortTile];
  uint32_t wcnt[kWaves][kRadix];
  uint32_t local[kRadix];
  uint32_t gbase[kRadix];
  uint32_t gstart[kRadix];
  uint32_t hist[kMaxPasses * kRadix];
  uint32_t tmp[kWaves];
  uint32_t abort;
};

// Item i of lane l of wave w holds tile position w*64*I + i*64 + l, so
// (item, lane) order is batch order.
__device__ __forceinline__ uint32_t tile_pos(uint32_t wave, int i, uint32_t lane) {
  return wave * 64 * kSortItems + static_cast<uint32_t>(i) * 64 + lane;
}

// One stable counting pass over one tile held in registers: wave64 match-any
// ranking, publication of the tile's digit counts, decoupled look-back over
// the tiles before it, and a scatter through LDS so consecutive threads
// write consecutive output addresses.
__device__ void sort_tile_pass(const uint32_t (&kv)[kSortItems], const uint32_t (&val)[kSortItems],
                               uint32_t tile, uint32_t b, int shift, uint32_t* st,
                               uint32_t* out_kv, uint32_t* out_val, uint32_t* out_fence,
                               bool coherent_out, uint32_t* fault, SortLds& L) {
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t tbase = tile * kSortTile;
  for (uint32_t i = tid; i < kWaves * kRadix; i += kThreads) (&L.wcnt[0][0])[i] = 0u;
  if (tid == 0) L.abort = 0u;
  __syncthreads();

  uint32_t off[kSortItems];
#pragma unroll
  for (int i = 0; i < kSortItems; ++i) {
    const bool valid = tbase + tile_pos(wave, i, lane) < b;
    const uint32_t d = (kv[i] >> shift) & (kRadix - 1);
    uint64_t peers = ballot(valid);
#pragma unroll
    for (int bit = 0; bit < kRadixBits; ++bit) {
      const bool set = (d >> bit) & 1u;
      const uint64_t m = ballot(set);
      peers &= set ? m : ~m;
    }
    const uint32_t r = count_below(peers);
    uint32_t prev = 0;
    if (valid) prev = L.wcnt[wave][d];
    if (valid && r == 0) L.wcnt[wave][d] = prev + static_cast<uint32_t>(__popcll(peers));
    off[i] = prev + r;
  }
  __syncthreads();

  // Thread tid owns digit d = tid (kThreads == kRadix).
  const uint32_t d = tid;
  uint32_t tile_count = 0;
  for (uint32_t w = 0; w < kWaves; ++w) {
    const uint32_t c = L.wcnt[w][d];
    L.wcnt[w][d] = tile_count;
    tile_count += c;
  }
  if (tile == 0) st_dev(&st[d], kFlagInc | tile_count);
  else st_dev(&st[static_cast<size_t>(tile) * kRadix + d], kFlagAgg | tile_count);
  L.local[d] = block_excl_scan(tile_count, L.tmp);

  // Look back in chunks of kChunk predecessors (loads issued together).
  constexpr int kChunk = 16;
  uint32_t excl = 0;
  if (tile > 0) {
    int64_t j = static_cast<int64_t>(tile) - 1;
    uint32_t spins = 0;
    for (;;) {
      const int nchunk = j + 1 < kChunk ? static_cast<int>(j + 1) : kChunk;
      uint32_t w[kChunk];
#pragma unroll
      for (int k = 0; k < kChunk; ++k)
        w[k] = (k < nchunk) ? ld_dev(&st[static_cast<size_t>(j - k) * kRadix + d]) : 0u;
      int used = 0;
      bool done = false;
#pragma unroll
      for (int k = 0; k < kChunk; ++k) {
        if (k >= nchunk || done) break;
        const uint32_t f = w[k] & ~kCountMask;
        if (f == 0u) break;
        excl += w[k] & kCountMask;
        ++used;
        if (f == kFlagInc) done = true;
      }
      if (done) break;
      j -= used;
      if (used == 0) {
        __builtin_amdgcn_s_sleep(1);
        if (++spins == kSpinLimit) {
          atomicOr(fault, kFaultTimeout);
          L.abort = 1u;
          break;
        }
      }
    }
    st_dev(&st[static_cast<size_t>(tile) * kRadix + d], kFlagInc | (excl + tile_count));
  }
  L.gbase[d] = L.gstart[d] + excl;
  __syncthreads();

#pragma unroll
  for (int i = 0; i < kSortItems; ++i) {
    if (tbase + tile_pos(wave, i, lane) < b) {
      const uint32_t dd = (kv[i] >> shift) & (kRadix - 1);
      const uint32_t pos = L.local[dd] + L.wcnt[wave][dd] + off[i];
      L.kv[pos] = kv[i];
      L.val[pos] = val[i];
    }
  }
  __syncthreads();
  const uint32_t tile_n = (b - tbase) < static_cast<uint32_t>(kSortTile) ? (b - tbase) : kSortTile;
  if (L.abort == 0u) {
    for (uint32_t x = tid; x < tile_n; x += kThreads) {
      const uint32_t k = L.kv[x];
      const uint32_t dd = (k >> shift) & (kRadix - 1);
      const uint32_t o = L.gbase[dd] + (x - L.local[dd]);
      if (o < b) {
        if (coherent_out) {  // read by other work-groups after a grid barrier
          st_dev(&out_kv[o], k);
          st_dev(&out_val[o], L.val[x]);
        } else {
          out_kv[o] = k;
          out_val[o] = L.val[x];
          put_fence(out_fence, b, o, k);
        }
      }
    }
  }
  __syncthreads();
}

// Digit histograms of every pass in one read of the batch, a tile a work-group,
// accumulated into hist[parity] (LDS first, then one global atomic per non-zero
// bucket).
// Also clears hist[parity ^ 1] for the next sort, and this sort's look-back
// words and tile counters.
__global__ __launch_bounds__(kThreads) void k_sort_hist(SortArgs a) {
  __shared__ uint32_t s_h[kMaxPasses * kRadix];
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const SortMeta& m = a.meta;
  const size_t gthreads = static_cast<size_t>(gridDim.x) * kThreads;
  const size_t gid = static_cast<size_t>(blockIdx.x) * kThreads + tid;
  const size_t nstatus = static_cast<size_t>(a.passes) * m.num_sort_tiles * kRadix;
  for (size_t i = gid; i < nstatus; i += gthreads) m.status[i] = 0u;
  uint32_t* other = m.hist + static_cast<size_t>(m.parity ^ 1) * kMaxPasses * kRadix;
  for (size_t i = gid; i < static_cast<size_t>(kMaxPasses) * kRadix; i += gthreads) other[i] = 0u;
  if (gid < static_cast<size_t>(kMaxPasses)) m.tile_ctr[gid] = 0u;
  for (uint32_t i = tid; i < static_cast<uint32_t>(kMaxPasses * kRadix); i += kThreads) s_h[i] = 0u;
  __syncthreads();

  uint32_t kv[kSortItems], key[kSortItems], val[kSortItems];
  bool valid[kSortItems];
  tile_items<kSortItems>(a.src, blockIdx.x * kSortTile, wave, lane, kv, val, key, valid);
#pragma unroll
  for (int i = 0; i < kSortItems; ++i) {
    if (!valid[i]) continue;
    for (int p = 0; p < a.passes; ++p)
      atomicAdd(&s_h[p * kRadix + ((kv[i] >> (a.lo_bit + kRadixBits * p)) & (kRadix - 1))], 1u);
  }
  __syncthreads();
  uint32_t* mine = m.hist + static_cast<size_t>(m.parity) * kMaxPasses * kRadix;
  for (uint32_t i = tid; i < static_cast<uint32_t>(a.passes * kRadix); i += kThreads)
    if (s_h[i] != 0u) atomicAdd(&mine[i], s_h[i]);
}

// Where element e < b of the batch, as the sort sees it (read back to front and
// padded in front), stands in the caller's arrays.
__device__ __forceinline__ uint32_t src_index(const BatchSrc& s, uint32_t e) {
  const uint32_t x = s.b - 1 - e;
  return x < s.n - 1 ? x : s.n - 1;
}
__device__ __forceinline__ uint32_t src_kv(const BatchSrc& s, uint32_t raw, uint32_t i) {
  if (s.mode == kEncoded) return raw;
  const uint32_t st = s.mode == kMixed ? (s.is_delete[i] ? 0u : 1u) : (s.mode == kDelete ? 0u : 1u);
  return (raw << 1) | st;
}

// One stable counting pass of the batch sort on digit `pass`.  Tiles take
// dynamic ids in start order (so every predecessor a tile waits for has
// started); the tile a work-group most likely receives is loaded while the
// id is in flight.
__global__ __launch_bounds__(kThreads) void k_sort_pass(SortArgs a, int pass) {
  __shared__ SortLds L;
  __shared__ uint32_t s_tile;
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const SortMeta& m = a.meta;
  const uint32_t b = a.src.b;
  if (tid == 0) s_tile = atomicAdd(&m.tile_ctr[pass], 1u);
  const uint32_t* mine = m.hist + static_cast<size_t>(m.parity) * kMaxPasses * kRadix;
  const uint32_t gtotal = mine[static_cast<size_t>(pass) * kRadix + tid];
  const uint32_t* in_kv = (pass == 0) ? nullptr : a.tmp_kv[(pass - 1) & 1];
  const uint32_t* in_val = (pass == 0) ? nullptr : a.tmp_val[(pass - 1) & 1];
  uint32_t* o_kv = (pass == a.passes - 1) ? a.out_kv : a.tmp_kv[pass & 1];
  uint32_t* o_val = (pass == a.passes - 1) ? a.out_val : a.tmp_val[pass & 1];

  uint32_t kv[kSortItems], val[kSortItems];
  auto load_tile = [&](uint32_t t) {
    const uint32_t tb = t * kSortTile;
    if (in_kv == nullptr) {
      uint32_t key[kSortItems];
      bool valid[kSortItems];
      tile_items<kSortItems>(a.src, tb, wave, lane, kv, val, key, valid);
      return;
    }
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
      const uint32_t e = tb + tile_pos(wave, i, lane);
      const uint32_t ec = e < b ? e : b - 1;  // in bounds; the item is dropped below
      kv[i] = in_kv[ec];
      val[i] = in_val[ec];
    }
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
      const bool ok = tb + tile_pos(wave, i, lane) < b;
      kv[i] = ok ? kv[i] : 0u;
      val[i] = ok ? val[i] : 0u;
    }
  };
  load_tile(blockIdx.x);
  L.gstart[tid] = block_excl_scan(gtotal, L.tmp);  // contains the barrier publishing s_tile
  const uint32_t tile = s_tile;
  if (tile != blockIdx.x) load_tile(tile);
  // The largest top digit, for the choice of the next sorts: without the batch's
  // padding, which the top-digit sort does not sort either.
  if (pass == 0 && tile == 0 && a.skew_out != nullptr) {
    const int top = a.passes - 1;
    uint32_t c = mine[static_cast<size_t>(top) * kRadix + tid];
    if (a.src.n < b) {
      const uint32_t kv_last = src_kv(a.src, a.src.keys[a.src.n - 1], a.src.n - 1);
      if (((kv_last >> (a.lo_bit + kRadixBits * top)) & (kRadix - 1)) == tid) c -= b - a.src.n;
    }
    record_max(large_bucket(c), a.skew_out, L.tmp);
  }
  uint32_t* st = m.status + static_cast<size_t>(pass) * m.num_sort_tiles * kRadix;
  sort_tile_pass(kv, val, tile, b, a.lo_bit + kRadixBits * pass, st, o_kv, o_val,
                 (pass == a.passes - 1) ? a.out_fence : nullptr, false, &m.err[1], L);
}

// ------------------------------------------------------------ large digit passes
// Stable ranking of one item per lane by digit d among the valid lanes of
// the wave: returns the item's position after the entries already counted
// in wcnt[d], and adds the wave's count of d to wcnt[d].
template <int kBits>
__device__ __forceinline__ uint32_t wave_rank(uint32_t d, bool valid, uint32_t* wcnt) {
  const uint64_t on = ballot(valid);
  uint32_t lo = static_cast<uint32_t>(on), hi = static_cast<uint32_t>(on >> 32);
#pragma unroll
  for (int bit = 0; bit < kBits; ++bit) {
    // x is all ones where the lane's bit is set: the lanes that agree with
    // it are ~(m ^ x), one three-input logic operation a half.
    const uint32_t x = static_cast<uint32_t>(__builtin_amdgcn_sbfe(static_cast<int>(d), bit, 1));
    const uint64_t m = ballot(x != 0u);
    lo &= ~(static_cast<uint32_t>(m) ^ x);
    hi &= ~(static_cast<uint32_t>(m >> 32) ^ x);
  }
  const uint64_t peers = (static_cast<uint64_t>(hi) << 32) | lo;
  const uint32_t r = count_below(peers);
  uint32_t prev = 0;
  if (valid) prev = wcnt[d];
  if (valid && r == 0) wcnt[d] = prev + static_cast<uint32_t>(__popcll(peers));
  return prev + r;
}

// The digit passes of a sort of more than kMsdMaxTiles tiles.  Such a pass is
// bound by memory, and a decoupled look-back keeps it from it: every tile's
// 256 counts travel between the 8 XCDs through memory, some microseconds a
// hop, with hundreds of tiles waiting.  Here a fixed set of work-groups
// each owns one contiguous chunk of the input for the whole pass: k_lsd_up
// counts the digits of every chunk, k_lsd_scan turns the counts into each
// chunk's first output position per digit (a work-group per digit), and
// k_lsd_down walks its chunk tile by tile with running positions.  No
// work-group waits for another, for 4 B per element read once more.
// A pass over 2^25 pairs takes 216 us in all (about 400 with the look-back
// over tiles of 2048), of which reading and writing alone take 124, the
// ranking 59 and the scattered writes 42.  Tiles of 8192: a digit's run in a
// tile is then 32 elements, one 128-byte line; tiles of 4096 took 257 us (256
// threads) and of 16384 240 us (one work-group a CU).
constexpr int kLsdThreads = 512;
constexpr int kLsdWaves = kLsdThreads / 64;
constexpr int kLsdItems = 16;
constexpr uint32_t kLsdTile = kLsdThreads * kLsdItems;
constexpr uint32_t kLsdMaxGroups = 512;  // two work-groups on each of 256 CUs

// Work-groups of a pass over b elements and the tiles that each takes.
struct LsdGrid {
  uint32_t groups, tiles_per_group;
};
inline LsdGrid lsd_grid(uint32_t b) {
  const uint32_t tiles = static_cast<uint32_t>((static_cast<uint64_t>(b) + kLsdTile - 1) / kLsdTile);
  const uint32_t per = (tiles + kLsdMaxGroups - 1) / kLsdMaxGroups;
  return {(tiles + per - 1) / per, per};
}

// Input of a pass: the previous pass's output, or nulls for the caller's batch.
struct LsdSrc {
  const uint32_t* kv;
  const uint32_t* val;
};

__global__ __launch_bounds__(kLsdThreads) void k_lsd_up(SortArgs a, LsdSrc in, int shift,
                                                        uint32_t tiles_per_group,
                                                        uint32_t* counts) {
  __shared__ uint32_t h[kLsdWaves][kRadix];
  const uint32_t tid = threadIdx.x, wave = tid >> 6;
  const uint32_t b = a.src.b;
  for (uint32_t i = tid; i < kLsdWaves * kRadix; i += kLsdThreads) (&h[0][0])[i] = 0u;
  __syncthreads();
  const uint64_t lo = static_cast<uint64_t>(blockIdx.x) * tiles_per_group * kLsdTile;
  const uint64_t hi64 = lo + static_cast<uint64_t>(tiles_per_group) * kLsdTile;
  const uint32_t hi = hi64 < b ? static_cast<uint32_t>(hi64) : b;
  constexpr int kU = 8;  // loads in flight per thread
  for (uint64_t base = lo; base < hi; base += static_cast<uint64_t>(kLsdThreads) * kU) {
    uint32_t x[kU], idx[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const uint64_t e = base + static_cast<uint64_t>(u) * kLsdThreads + tid;
      const uint32_t ec = e < hi ? static_cast<uint32_t>(e) : hi - 1;
      idx[u] = in.kv == nullptr ? src_index(a.src, ec) : ec;
      x[u] = in.kv == nullptr ? a.src.keys[idx[u]] : in.kv[idx[u]];
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const uint64_t e = base + static_cast<uint64_t>(u) * kLsdThreads + tid;
      const uint32_t kv = in.kv == nullptr ? src_kv(a.src, x[u], idx[u]) : x[u];
      if (e < hi) atomicAdd(&h[wave][(kv >> shift) & (kRadix - 1)], 1u);
    }
  }
  __syncthreads();
  if (tid < kRadix) {
    uint32_t c = 0;
#pragma unroll
    for (int w = 0; w < kLsdWaves; ++w) c += h[w][tid];
    counts[static_cast<size_t>(tid) * gridDim.x + blockIdx.x] = c;
  }
}

// Work-group d: the exclusive scan of digit d's counts over the chunks (at
// most 2 kThreads of them), in place; the digit's total goes to totals[d].
static_assert(kLsdMaxGroups <= 2 * kThreads, "two counts per thread");
__global__ __launch_bounds__(kThreads) void k_lsd_scan(uint32_t* counts, uint32_t groups,
                                                       uint32_t* totals) {
  __shared__ uint32_t tmp[kWaves];
  uint32_t* row = counts + static_cast<size_t>(blockIdx.x) * groups;
  const uint32_t i = 2 * threadIdx.x;
  const uint32_t c0 = i < groups ? row[i] : 0u, c1 = i + 1 < groups ? row[i + 1] : 0u;
  const uint32_t ex = block_excl_scan(c0 + c1, tmp);
  if (i < groups) row[i] = ex;
  if (i + 1 < groups) row[i + 1] = ex + c0;
  if (threadIdx.x == kThreads - 1) totals[blockIdx.x] = ex + c0 + c1;
}

struct LsdLds {
  uint32_t kv[kLsdTile];
  uint32_t val[kLsdTile];
  uint32_t wcnt[kLsdWaves][kRadix];
  uint32_t run[kRadix];  // the tile's first output position of each digit, minus its first in LDS
  uint32_t tmp[kLsdWaves];
};

// kFirst: pass 0, which reads the caller's batch.
template <bool kFirst>
__global__ __launch_bounds__(kLsdThreads, 4) void k_lsd_down(SortArgs a, LsdSrc in, int shift,
                                                          uint32_t tiles_per_group,
                                                          const uint32_t* counts,
                                                          const uint32_t* totals, uint32_t* o_kv,
                                                          uint32_t* o_val, uint32_t* o_fence) {
  __shared__ LsdLds L;
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t b = a.src.b;
  // Work-group-wide exclusive scan of one value per digit thread.
  auto scan = [&](uint32_t x) {
    const uint32_t inc = wave_incl_scan(x, lane);
    if (lane == 63) L.tmp[wave] = inc;
    __syncthreads();
    uint32_t pre = 0;
    for (uint32_t w = 0; w < wave; ++w) pre += L.tmp[w];
    __syncthreads();
    return pre + inc - x;
  };
  const uint32_t tot = tid < kRadix ? totals[tid] : 0u;
  const uint32_t first = scan(tot);
  uint32_t pos = 0;  // digit thread: next output position of digit tid
  if (tid < kRadix) pos = first + counts[static_cast<size_t>(tid) * gridDim.x + blockIdx.x];

  // Item i of lane l of wave w is tile element w * 64 * I + 64 i + l.  A whole
  // tile (and, in pass 0, one without padding) is read from a uniform base
  // with constant offsets between a thread's items; others clamp each index.
  const uint32_t at0 = wave * 64 * kLsdItems + lane;
  const uint32_t* vp = a.src.vals != nullptr ? a.src.vals : a.src.keys;
  uint32_t kv[kLsdItems], val[kLsdItems];
  auto load_tile = [&](uint32_t tb) {
    const bool whole = b - tb >= kLsdTile;
    if (kFirst && whole && tb >= b - a.src.n && a.src.mode != kMixed) {
      const uint32_t x0 = b - tb - kLsdTile, y = kLsdTile - 1 - at0;
      const uint32_t* pk = a.src.keys + x0;
      const uint32_t* pv = vp + x0;
#pragma unroll
      for (int i = 0; i < kLsdItems; ++i) kv[i] = pk[y - i * 64];
#pragma unroll
      for (int i = 0; i < kLsdItems; ++i) val[i] = pv[y - i * 64];
    } else if (!kFirst && whole) {
      const uint32_t* pk = in.kv + tb;
      const uint32_t* pv = in.val + tb;
#pragma unroll
      for (int i = 0; i < kLsdItems; ++i) kv[i] = pk[at0 + i * 64];
#pragma unroll
      for (int i = 0; i < kLsdItems; ++i) val[i] = pv[at0 + i * 64];
    } else {
#pragma unroll
      for (int i = 0; i < kLsdItems; ++i) {
        const uint32_t e = tb + at0 + i * 64, ec = e < b ? e : b - 1;
        const uint32_t x = kFirst ? src_index(a.src, ec) : ec;
        kv[i] = kFirst ? a.src.keys[x] : in.kv[x];
        val[i] = kFirst ? vp[x] : in.val[x];
        if (kFirst && a.src.mode == kMixed) {
          kv[i] = src_kv(a.src, kv[i], x);
          if ((kv[i] & 1u) == 0u) val[i] = 0u;
        }
      }
    }
    if (kFirst && a.src.mode != kMixed && a.src.mode != kEncoded) {
      const uint32_t st = a.src.mode == kDelete ? 0u : 1u;
#pragma unroll
      for (int i = 0; i < kLsdItems; ++i) {
        kv[i] = (kv[i] << 1) | st;
        val[i] = st ? val[i] : 0u;  // tombstones carry value 0
      }
    }
  };
  const uint32_t t0 = blockIdx.x * tiles_per_group;
  const uint32_t tiles = static_cast<uint32_t>((static_cast<uint64_t>(b) + kLsdTile - 1) / kLsdTile);
  const uint32_t t1 = t0 + tiles_per_group < tiles ? t0 + tiles_per_group : tiles;
  for (uint32_t t = t0; t < t1; ++t) {
    const uint32_t tb = t * kLsdTile;
    const uint32_t n = (b - tb) < kLsdTile ? (b - tb) : kLsdTile;
    load_tile(tb);
    for (uint32_t i = lane; i < kRadix; i += 64) L.wcnt[wave][i] = 0u;  // this wave's own
    uint32_t off[kLsdItems];
    if (n == kLsdTile) {
#pragma unroll
      for (int i = 0; i < kLsdItems; ++i)
        off[i] = wave_rank<kRadixBits>((kv[i] >> shift) & (kRadix - 1), true, L.wcnt[wave]);
    } else {
#pragma unroll
      for (int i = 0; i < kLsdItems; ++i)
        off[i] = wave_rank<kRadixBits>((kv[i] >> shift) & (kRadix - 1), at0 + i * 64 < n,
                                       L.wcnt[wave]);
    }
    __syncthreads();
    uint32_t c = 0;
    if (tid < kRadix) {
#pragma unroll
      for (int w = 0; w < kLsdWaves; ++w) {
        const uint32_t x = L.wcnt[w][tid];
        L.wcnt[w][tid] = c;
        c += x;
      }
    }
    const uint32_t loc = scan(c);
    if (tid < kRadix) {
#pragma unroll
      for (int w = 0; w < kLsdWaves; ++w) L.wcnt[w][tid] += loc;
      L.run[tid] = pos - loc;
      pos += c;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kLsdItems; ++i) {
      if (at0 + i * 64 < n) {
        const uint32_t at = L.wcnt[wave][(kv[i] >> shift) & (kRadix - 1)] + off[i];
        L.kv[at] = kv[i];
        L.val[at] = val[i];
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kLsdItems; ++i) {
      const uint32_t x = static_cast<uint32_t>(i) * kLsdThreads + tid;
      if (x < n) {
        const uint32_t k = L.kv[x];
        const uint32_t o = L.run[(k >> shift) & (kRadix - 1)] + x;
        o_kv[o] = k;
        o_val[o] = L.val[x];
        put_fence(o_fence, b, o, k);
      }
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------ MSD sort
// For batches of at most kMsdMaxTiles tiles the sort exchanges data across
// the device only once: each tile grouped in place by its top kTopBits-bit
// digit (with the batch's digit totals and each tile's group starts), then
// each of the kTopBuckets buckets gathered from every tile and sorted on
// its own by one work-group on the remaining bits (in LDS when it fits,
// streaming through the bucket's global range otherwise).  Two kernels
// instead of 1 + passes, and no look-back chains.

// Stable ranks of a wave's items among equal top digits, item i of every
// lane after item i - 1 (tile order is item-major within the wave).  The
// 10-bit digit is split into two 5-bit halves with a table of lane masks
// each: for every item, each lane ORs its lane bit into the entry of its
// high half in one table and of its low half in the other, reads both
// entries back and clears them, and the AND of the two masks is the set of
// lanes whose item has the same digit.  The six LDS operations of all items
// are issued back to back (one wave's LDS operations are applied in issue
// order, so each item sees exactly its own lanes).  Invalid items use the
// spare entry kHalf of both tables.  Then the lowest lane of each digit
// group adds the group's size to wcnt[d] with an LDS fetch-and-add, items in
// order, and its old count is broadcast to the group.  The tables are this
// wave's own, so no work-group barrier is needed; their entries are zero
// before and after.
constexpr uint32_t kHalfBits = kTopBits / 2;
constexpr uint32_t kHalf = 1u << kHalfBits;
static_assert(2 * kHalfBits == kTopBits, "the top digit splits into two equal halves");
template <int kN>
__device__ __forceinline__ void wave_rank_items(const uint32_t (&d)[kN], const bool (&valid)[kN],
                                                uint64_t* mhi, uint64_t* mlo, uint32_t* wcnt,
                                                uint32_t (&off)[kN]) {
  const uint32_t lane = lane_id();
  const uint64_t bit = 1ull << lane;
  uint64_t grp[kN];
#pragma unroll
  for (int i = 0; i < kN; ++i) {
    uint64_t* eh = &mhi[valid[i] ? (d[i] >> kHalfBits) : kHalf];
    uint64_t* el = &mlo[valid[i] ? (d[i] & (kHalf - 1)) : kHalf];
    __hip_atomic_fetch_or(eh, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __hip_atomic_fetch_or(el, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    grp[i] = *eh & *el;
    *eh = 0ull;
    *el = 0ull;
  }
  uint32_t r[kN], lead[kN], size[kN];
#pragma unroll
  for (int i = 0; i < kN; ++i) {
    r[i] = count_below(grp[i]);
    lead[i] = static_cast<uint32_t>(__builtin_ctzll(grp[i] | (1ull << 63)));
    size[i] = static_cast<uint32_t>(__popcll(grp[i]));
  }
  // Every lane issues the add (others add 0, so the leader's old count is the
  // count before this item whatever order the lanes are applied in).  The
  // counts are 16-bit halves of wcnt's words (digit d in half d & 1 of word
  // d >> 1): a wave adds at most 64 kN <= 65535 per digit, so no carry
  // crosses into the other half.
  static_assert(64 * kN <= 0xFFFF, "per-wave digit counts fit 16 bits");
  uint32_t prev[kN];
#pragma unroll
  for (int i = 0; i < kN; ++i) {
    const uint32_t dd = valid[i] ? d[i] : 0u;
    const uint32_t sh = (dd & 1u) * 16u;
    prev[i] = atomicAdd(&wcnt[dd >> 1], ((valid[i] && r[i] == 0) ? size[i] : 0u) << sh) >> sh;
  }
#pragma unroll
  for (int i = 0; i < kN; ++i)
    off[i] = (static_cast<uint32_t>(__shfl(static_cast<int>(prev[i]), static_cast<int>(lead[i]), 64)) &
              0xFFFFu) + r[i];
}

// Stable scatter of one tile on the top digit, tile-major: the tile's
// elements, grouped by digit (stable within a digit), go back to the tile's
// own range of tmp_kv[0] / tmp_val[0] with coalesced writes, and the tile
// records where each digit's group starts (two 16-bit starts per word; a
// tile holds at most kSortTile elements).  A bucket's elements are then its
// digit's group in every tile, in tile order.  Thread t owns the digits
// [kTopPer t, kTopPer t + kTopPer).  Tile 0 also hands the largest bucket
// recorded by the previous sort in this scratch slot to the host-visible
// hint and restarts the record, and first writes the launch's sequence
// number to the host-visible progress word (the launch has started, so every
// earlier launch on the stream has finished).
struct ScatterLds {
  // Per-wave digit counts, then each wave's offset inside each digit's
  // group: 16-bit halves, digit d in half d & 1 of word d >> 1.
  uint32_t wcnt[kWaves][kTopBuckets / 2];
  uint32_t kv[kSortTile];              // the tile grouped by digit
  uint32_t val[kSortTile];
  union {
    uint64_t mask[kWaves][2][kHalf + 1];  // ranking tables, zero between items
    uint32_t local[kTopBuckets];          // each digit's group start in the tile
  } u;
  uint32_t tmp[2 * kWaves];
  uint32_t rmax[kWaves];
};

// What the tile half needs (a launch reads its arguments afresh, so they are
// kept short).
struct ScatterArgs {
  BatchSrc src;
  uint32_t* kv;         // the slot's scattered batch
  uint32_t* val;
  uint32_t* tile_cnt;   // its group starts
  uint32_t* bucket_n;   // its bucket-size record
  uint32_t* pad;        // its padding element
  uint32_t* skew_out;
  uint64_t* progress;
  uint64_t seq;
  int top_shift;
};

__device__ void tile_scatter(const ScatterArgs& a, uint32_t tile, ScatterLds& S) {
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  BatchSrc src = a.src;
  src.b = src.n;  // the padding is not scattered
  const uint32_t b = src.b;
  const uint32_t tbase = tile * kSortTile;
  const uint32_t d0 = tid * kTopPer;
  static_assert(kTopPer == 4 && kSortTile < 65536, "four digits per thread, 16-bit starts");
  uint32_t kv[kSortItems], val[kSortItems], off[kSortItems], dg[kSortItems], key[kSortItems];
  bool valid[kSortItems];
  tile_items<kSortItems>(src, tbase, wave, lane, kv, val, key, valid);
  if (tile == 0 && tid == 0 && a.progress != nullptr)
    __hip_atomic_store(a.progress, a.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  // Tile 0 hands over the largest bucket of the slot's previous bucket sort
  // (a hint for the choice of the next sorts): its loads go out now, the
  // maximum is taken after the tile's ranking.
  static_assert(kTopBuckets == 4 * kThreads, "four bucket records per thread");
  const bool hand = tile == 0 && a.skew_out != nullptr;
  uint4 rec4 = make_uint4(0u, 0u, 0u, 0u);
  if (hand) rec4 = reinterpret_cast<const uint4*>(a.bucket_n)[tid];
  // Rank the tile: each wave clears and fills its own tables.
  for (uint32_t i = lane; i < kTopBuckets / 2; i += 64) S.wcnt[wave][i] = 0u;
  for (uint32_t i = lane; i < 2 * (kHalf + 1); i += 64) (&S.u.mask[wave][0][0])[i] = 0ull;
#pragma unroll
  for (int i = 0; i < kSortItems; ++i) dg[i] = (kv[i] >> a.top_shift) & (kTopBuckets - 1);
  wave_rank_items(dg, valid, S.u.mask[wave][0], S.u.mask[wave][1], S.wcnt[wave], off);
  __syncthreads();  // every wave is done with its tables: S.u.local may be written
  // This thread's four digits are the halves of words d0 / 2 and d0 / 2 + 1;
  // the wave offsets inside a group are below kSortTile, so they fit too.
  uint32_t cnt[kTopPer], tsum = 0;
  uint32_t wpk[kWaves][2];
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    wpk[w][0] = S.wcnt[w][d0 / 2];
    wpk[w][1] = S.wcnt[w][d0 / 2 + 1];
  }
  uint32_t wo[kWaves][kTopPer];
#pragma unroll
  for (int q = 0; q < kTopPer; ++q) {
    uint32_t run = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      wo[w][q] = run;
      run += (wpk[w][q >> 1] >> ((q & 1) * 16)) & 0xFFFFu;
    }
    cnt[q] = run;
    tsum += run;
  }
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    S.wcnt[w][d0 / 2] = wo[w][0] | (wo[w][1] << 16);
    S.wcnt[w][d0 / 2 + 1] = wo[w][2] | (wo[w][3] << 16);
  }
  uint32_t lrun = block_excl_scan(tsum, S.tmp);
  uint32_t start[kTopPer];
#pragma unroll
  for (int q = 0; q < kTopPer; ++q) {
    start[q] = lrun;
    S.u.local[d0 + q] = lrun;
    lrun += cnt[q];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kSortItems; ++i) {
    if (valid[i]) {
      const uint32_t dd = dg[i];
      const uint32_t wof = (S.wcnt[wave][dd >> 1] >> ((dd & 1u) * 16u)) & 0xFFFFu;
      const uint32_t pos = S.u.local[dd] + wof + off[i];
      S.kv[pos] = kv[i];
      S.val[pos] = val[i];
    }
  }
  __syncthreads();
  if (hand) {
    uint32_t x = max(max(rec4.x, rec4.y), max(rec4.z, rec4.w));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x = max(x, static_cast<uint32_t>(__shfl_xor(x, o, 64)));
    if (lane == 0) S.rmax[wave] = x;
    __syncthreads();
    if (tid == 0) {
      uint32_t mx = 0;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) mx = max(mx, S.rmax[w]);
      *a.skew_out = mx;
    }
  }
  // Global writes last, so that no barrier waits for them: the group starts
  // and the grouped tile.
  uint32_t* row = a.tile_cnt + static_cast<size_t>(tile) * (kTopBuckets / 2);
  row[2 * tid] = start[0] | (start[1] << 16);
  row[2 * tid + 1] = start[2] | (start[3] << 16);
  if (tile == 0 && tid == 0 && a.src.n < a.src.b) {  // the batch's last element
    a.pad[0] = kv[0];
    a.pad[1] = val[0];
  }
  const uint32_t tile_n = (b - tbase) < static_cast<uint32_t>(kSortTile) ? (b - tbase) : kSortTile;
  for (uint32_t x = tid; x < tile_n; x += kThreads) {
    a.kv[tbase + x] = S.kv[x];
    a.val[tbase + x] = S.val[x];
  }
  (void)key;
}

__global__ __launch_bounds__(kThreads) void k_msd_scatter(ScatterArgs a) {
  __shared__ ScatterLds S;
  tile_scatter(a, blockIdx.x, S);
}

struct alignas(16) LocalLds {
  uint32_t k[2][kLocalCap];
  uint32_t v[2][kLocalCap];
  uint32_t wcnt[kWaves][kRadix];
  uint32_t tmp[2 * kWaves + 2];  // scans; then the bucket's start and size
  uint32_t lo[kMaxFuse];      // fused cascade: start of the digit's range per level
  uint32_t rs[kMaxFuse + 2];  // run starts in the concatenated runs
  const uint32_t* run_k[kMaxFuse + 1];  // fused load: source of each run
  const uint32_t* run_v[kMaxFuse + 1];
  uint32_t run_delta[kMaxFuse + 1];
  uint32_t pad_at[kMaxGroup];  // place of each batch's padding in the bucket's output
  // Merge of runs larger than LDS: each run's next element, its end, the part
  // of it in LDS and how much of that is merged.
  uint32_t cur[kMaxFuse + 1], len[kMaxFuse + 1], win[kMaxFuse + 2], cut[kMaxFuse + 1];
};

// One stable counting pass over n <= kLocalCap elements in LDS, from
// buffer `from` to buffer 1 - from, on the digit at `shift`.  Wave w owns
// positions [w*S, (w+1)*S) in (item, lane) order, S a multiple of 64.
__device__ void lds_pass(LocalLds& L, int from, uint32_t n, int shift) {
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t S = ((n + kThreads - 1) / kThreads) * 64;
  const uint32_t* sk = L.k[from];
  const uint32_t* sv = L.v[from];
  uint32_t* dk = L.k[1 - from];
  uint32_t* dv = L.v[1 - from];
  for (uint32_t i = tid; i < kWaves * kRadix; i += kThreads) (&L.wcnt[0][0])[i] = 0u;
  __syncthreads();
  for (uint32_t it = 0; it < S / 64; ++it) {
    const uint32_t pos = wave * S + it * 64 + lane;
    const bool valid = pos < n;
    (void)wave_rank<kRadixBits>(valid ? (sk[pos] >> shift) & (kRadix - 1) : 0u, valid, L.wcnt[wave]);
  }
  __syncthreads();
  uint32_t tot = 0;
  for (uint32_t w = 0; w < kWaves; ++w) {
    const uint32_t c = L.wcnt[w][tid];
    L.wcnt[w][tid] = tot;
    tot += c;
  }
  const uint32_t local = block_excl_scan(tot, L.tmp);
  for (uint32_t w = 0; w < kWaves; ++w) L.wcnt[w][tid] += local;
  __syncthreads();
  for (uint32_t it = 0; it < S / 64; ++it) {
    const uint32_t pos = wave * S + it * 64 + lane;
    const bool valid = pos < n;
    const uint32_t x = valid ? sk[pos] : 0u;
    const uint32_t o = wave_rank<kRadixBits>((x >> shift) & (kRadix - 1), valid, L.wcnt[wave]);
    if (valid) {
      dk[o] = x;
      dv[o] = sv[pos];
    }
  }
  __syncthreads();
}

// Stable passes over a bucket too large for LDS.  The bucket is first
// gathered from the tile-major scatter (group table segb / segp over ntiles
// tiles) into one of two global buffers at the bucket's own range: the
// output (out_kv at s) or the second scratch buffer (tmp_kv[1] at s), chosen
// so that the passes, ping-ponging between the two, end in the output (or, to
// leave room for padding, in the scratch buffer: to_tmp).  Nothing else reads
// either range.
__device__ void local_sort_streaming(const SortArgs& a, int lo_bit, int passes, uint32_t s,
                                     uint32_t n, LocalLds& L, const uint32_t* segb,
                                     const uint32_t* segp, uint32_t ntiles, bool to_tmp) {
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t* bk[2] = {a.out_kv + s, a.tmp_kv[1] + s};
  uint32_t* bv[2] = {a.out_val + s, a.tmp_val[1] + s};
  const int first = (passes & 1) ^ (to_tmp ? 1 : 0);
  uint32_t* fence = to_tmp ? nullptr : a.out_fence;
  for (uint32_t x = tid; x < n; x += kThreads) {
    uint32_t g = 0;
    for (uint32_t step = 1u << (31 - __builtin_clz(ntiles)); step > 0; step >>= 1) {
      const uint32_t probe = g + step;
      if (probe < ntiles && segp[probe] <= x) g = probe;
    }
    const uint32_t at = segb[g] + (x - segp[g]);
    const uint32_t k = a.tmp_kv[0][at];
    bk[first][x] = k;
    bv[first][x] = a.tmp_val[0][at];
    if (passes == 0) put_fence(fence, a.out_n, s + x, k);
  }
  if (passes == 0) return;
  __threadfence_block();
  __syncthreads();
  uint32_t* run = L.k[0];       // running output position per digit
  uint32_t* chunk_cnt = L.k[1];
  for (int p = 0; p < passes; ++p) {
    const int shift = lo_bit + kRadixBits * p;
    const int cur = first ^ (p & 1);  // the last pass writes buffer 0 (to_tmp: 1)
    const uint32_t* ik = bk[cur];
    const uint32_t* iv = bv[cur];
    uint32_t* ok = bk[cur ^ 1];
    uint32_t* ov = bv[cur ^ 1];
    run[tid] = 0u;
    __syncthreads();
    // Every pass reads this work-group's own writes.
    for (uint32_t x = tid; x < n; x += kThreads) {
      const uint32_t k = ik[x];
      atomicAdd(&run[(k >> shift) & (kRadix - 1)], 1u);
    }
    __syncthreads();
    const uint32_t c = run[tid];
    __syncthreads();
    run[tid] = block_excl_scan(c, L.tmp);
    __syncthreads();
    for (uint32_t cb = 0; cb < n; cb += kSortTile) {
      uint32_t kv[kSortItems], vv[kSortItems], off[kSortItems];
#pragma unroll
      for (int i = 0; i < kSortItems; ++i) {
        const uint32_t e = cb + tile_pos(wave, i, lane);
        kv[i] = e < n ? ik[e] : 0u;
        vv[i] = e < n ? iv[e] : 0u;
      }
      for (uint32_t i = tid; i < kWaves * kRadix; i += kThreads) (&L.wcnt[0][0])[i] = 0u;
      __syncthreads();
#pragma unroll
      for (int i = 0; i < kSortItems; ++i)
        off[i] = wave_rank<kRadixBits>((kv[i] >> shift) & (kRadix - 1), cb + tile_pos(wave, i, lane) < n,
                            L.wcnt[wave]);
      __syncthreads();
      uint32_t tot = 0;
      for (uint32_t w = 0; w < kWaves; ++w) {
        const uint32_t cc = L.wcnt[w][tid];
        L.wcnt[w][tid] = tot;
        tot += cc;
      }
      chunk_cnt[tid] = tot;
      __syncthreads();
#pragma unroll
      for (int i = 0; i < kSortItems; ++i) {
        if (cb + tile_pos(wave, i, lane) < n) {
          const uint32_t dd = (kv[i] >> shift) & (kRadix - 1);
          const uint32_t o = run[dd] + L.wcnt[wave][dd] + off[i];
          if (o < n) {
            ok[o] = kv[i];
            ov[o] = vv[i];
            if (p == passes - 1) put_fence(fence, a.out_n, s + o, kv[i]);
          }
        }
      }
      __syncthreads();
      run[tid] += chunk_cnt[tid];
      __syncthreads();
    }
  }
}

// Stable merge in LDS of a = src[0, A) (newer) and b = src[B, B + c), B >= A
// (older), into dst[0, A + c), a first on equal original keys.  Each thread
// finds the merge-path split of its share of the output by binary search,
// then merges it sequentially.  Ends with a barrier.
__device__ void lds_merge_pair(const uint32_t* sk, const uint32_t* sv, uint32_t A, uint32_t B,
                               uint32_t c, uint32_t* dk, uint32_t* dv) {
  const uint32_t total = A + c;
  const uint32_t per = (total + kThreads - 1) / kThreads;
  const uint32_t d0 = threadIdx.x * per < total ? threadIdx.x * per : total;
  const uint32_t d1 = d0 + per < total ? d0 + per : total;
  uint32_t lo = d0 > c ? d0 - c : 0, hi = d0 < A ? d0 : A;
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if ((sk[mid] >> 1) <= (sk[B + d0 - 1 - mid] >> 1)) lo = mid + 1;
    else hi = mid;
  }
  uint32_t ia = lo, ib = d0 - lo;
  for (uint32_t o = d0; o < d1; ++o) {
    const bool take_a = ia < A && (ib >= c || (sk[ia] >> 1) <= (sk[B + ib] >> 1));
    const uint32_t src = take_a ? ia : B + ib;
    dk[o] = sk[src];
    dv[o] = sv[src];
    ia += take_a ? 1u : 0u;
    ib += take_a ? 0u : 1u;
  }
  __syncthreads();
}

// Stable rank sort of the bucket's n <= kRankSortMax elements, held in
// L.k[0] / L.v[0], into L.k[1] / L.v[1].  fld[0, n8) holds each element's
// sort key (field << 8) | x, where the field is bits [lo_bit, lo_bit + 8
// passes) of its key variable (at most 24 bits: the bits below the top
// digit) and x its position; n8 = n rounded up to 8, with 0xFFFFFFFF past n.
// The keys are distinct, so the rank of element x, the number of smaller
// keys, orders by field and then by position (a stable sort, the same order
// as the radix passes over those bits).  The keys are read four at a time
// (16-byte LDS reads, eight in flight); the entries past n are above every
// element's key.  Waves without elements skip the count.
__device__ void rank_sort(LocalLds& L, const uint32_t* fld, uint32_t n) {
  static_assert(kRankSortMax <= 256u && kRankSortMax <= static_cast<uint32_t>(kThreads),
                "positions fit 8 bits; one element per thread");
  const uint32_t tid = threadIdx.x;
  if ((tid & ~63u) < n) {
    const uint32_t n8 = (n + 7u) & ~7u;
    const uint32_t cx = tid < n ? fld[tid] : 0u;
    uint32_t rank = 0;
    const uint4* f4 = reinterpret_cast<const uint4*>(fld);
    auto below = [cx](const uint4& p) {
      return (p.x < cx ? 1u : 0u) + (p.y < cx ? 1u : 0u) + (p.z < cx ? 1u : 0u) +
             (p.w < cx ? 1u : 0u);
    };
    uint32_t y = 0;
    for (; y + 32u <= n8; y += 32u) {  // eight 16-byte reads in flight
      uint4 p[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) p[u] = f4[y / 4 + u];
#pragma unroll
      for (int u = 0; u < 8; ++u) rank += below(p[u]);
    }
    for (; y < n8; y += 8u) {
      const uint4 p = f4[y / 4];
      const uint4 q = f4[y / 4 + 1];
      rank += below(p) + below(q);
    }
    if (tid < n) {
      L.k[1][rank] = L.k[0][tid];
      L.v[1][rank] = L.v[0][tid];
    }
  }
  __syncthreads();
}

// Bound of original key k in the sorted segment [lo, hi) of s (LDS or
// global): first position whose key is >= k (upper: > k).
__device__ __forceinline__ uint32_t seg_bound(const uint32_t* s, uint32_t lo, uint32_t hi,
                                              uint32_t k, bool upper) {
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    const uint32_t x = s[mid] >> 1;
    if (upper ? x <= k : x < k) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// A bucket larger than LDS that is large because of one key: sorts it when the
// most frequent key of 64 sampled elements holds all but kLocalCap of them.
// Elements of equal keys are in order as they come, so that key's go straight
// to their places and only the others are sorted, in LDS.  put(x, kv, value)
// writes element x of the sorted bucket.  Each wave takes a quarter of the
// groups, once to count and once to place.  Returns false, with nothing
// written, when the bucket is not of this kind.  One work-group's instruction
// stream bounds it: Zipf(1.1) pairs of 32 768, whose first key takes 8 %, take
// 15.5 us a sort (by digits each batch took a histogram and three passes of
// 10.3 us).
template <typename Put>
__device__ __forceinline__ bool sort_hot(const SortArgs& a, int lo_bit, int passes, uint32_t fmask, uint32_t n,
                         LocalLds& L, uint32_t* fld, const uint32_t* segb, const uint32_t* segp,
                         uint32_t nta, Put put) {
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  auto field = [&](uint32_t kv) { return (kv >> lo_bit) & fmask; };
  // The sample, the same in every wave.
  uint32_t g = 0;
  const uint32_t sx = static_cast<uint32_t>((static_cast<uint64_t>(lane) * n) >> 6);
  for (uint32_t step = 1u << (31 - __builtin_clz(nta)); step > 0; step >>= 1) {
    const uint32_t probe = g + step;
    if (probe < nta && segp[probe] <= sx) g = probe;
  }
  const uint32_t sf = field(a.tmp_kv[0][segb[g] + (sx - segp[g])]);
  uint32_t same = 0;
  for (int i = 0; i < 64; ++i)
    same += static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(sf), i)) == sf ? 1u : 0u;
  uint32_t best = (same << 6) | lane;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) best = max(best, static_cast<uint32_t>(__shfl_xor(best, o, 64)));
  if ((best >> 6) < 4u) return false;
  const uint32_t K = static_cast<uint32_t>(__shfl(static_cast<int>(sf), static_cast<int>(best & 63u), 64));
  const uint32_t g0 = wave * nta / kWaves, g1 = (wave + 1) * nta / kWaves;
  // each(kv, value, in): 64 elements at a time, in order.  Two pieces of up
  // to 256 elements of one group are loaded together: a tile's group of a hot
  // key is one piece or two, and a wave has few others to hide its loads (one
  // piece at a time, Zipf(1.1) batches of 131 072 take 71.0 us a step, two
  // 62.7, four 59.5 but scratch where batches are padded; loads by bucket
  // position, whose groups have to be searched for, 88).
  constexpr int kPieces = 2;
  auto scan = [&](bool vals, auto each) {
    uint32_t q = g0, j = 0, first = 0, c = 0;
    if (q < g1) {
      first = segb[q];
      c = (q + 1 < nta ? segp[q + 1] : n) - segp[q];
    }
    while (q < g1) {
      uint32_t at[kPieces], cnt[kPieces], k[kPieces][4], v[kPieces][4];
#pragma unroll
      for (int p = 0; p < kPieces; ++p) {
        while (q < g1 && j >= c) {
          j = 0;
          if (++q < g1) {
            first = segb[q];
            c = (q + 1 < nta ? segp[q + 1] : n) - segp[q];
          }
        }
        at[p] = q < g1 ? first + j : 0u;
        cnt[p] = q < g1 ? min(c - j, 256u) : 0u;
        j += 256;
      }
#pragma unroll
      for (int p = 0; p < kPieces; ++p) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const uint32_t x = 64 * u + lane, i = at[p] + (x < cnt[p] ? x : 0u);
          k[p][u] = as_global(a.tmp_kv[0])[i];
          v[p][u] = vals ? as_global(a.tmp_val[0])[i] : 0u;
        }
      }
#pragma unroll
      for (int p = 0; p < kPieces; ++p) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const uint32_t x = 64 * u + lane;
          if (64u * u < cnt[p]) each(k[p][u], v[p][u], x < cnt[p]);
        }
      }
    }
  };
  uint32_t lt = 0, eq = 0, ne = 0;
  scan(false, [&](uint32_t k, uint32_t, bool in) {
    const uint32_t f = field(k);
    lt += static_cast<uint32_t>(__popcll(ballot(in && f < K)));
    eq += static_cast<uint32_t>(__popcll(ballot(in && f == K)));
    ne += static_cast<uint32_t>(__popcll(ballot(in && f != K)));
  });
  if (lane == 0) {
    L.win[wave] = lt;
    L.len[wave] = eq;
    L.cur[wave] = ne;
  }
  __syncthreads();
  uint32_t n_lt = 0, n_eq = 0, m = 0, at_eq = 0, at_ne = 0;
  for (uint32_t w = 0; w < kWaves; ++w) {
    if (w == wave) {
      at_eq = n_eq;
      at_ne = m;
    }
    n_lt += L.win[w];
    n_eq += L.len[w];
    m += L.cur[w];
  }
  if (m > static_cast<uint32_t>(kLocalCap)) return false;
  at_eq += n_lt;
  const bool rank = m <= kRankSortMax;
  scan(true, [&](uint32_t k, uint32_t v, bool in) {
    const uint32_t f = field(k);
    const uint64_t me = ballot(in && f == K), mn = ballot(in && f != K);
    if (in && f == K) put(at_eq + count_below(me), k, v);
    if (in && f != K) {
      const uint32_t x = at_ne + count_below(mn);
      L.k[0][x] = k;
      L.v[0][x] = v;
      if (rank) fld[x] = (f << 8) | x;
    }
    at_eq += static_cast<uint32_t>(__popcll(me));
    at_ne += static_cast<uint32_t>(__popcll(mn));
  });
  if (rank && tid >= m && tid < ((m + 7u) & ~7u)) fld[tid] = 0xFFFFFFFFu;
  __syncthreads();
  int cur = 0;
  if (rank) {
    rank_sort(L, fld, m);
    cur = 1;
  } else {
    for (int p = 0; p < passes; ++p) {
      lds_pass(L, cur, m, lo_bit + kRadixBits * p);
      cur = 1 - cur;
    }
  }
  for (uint32_t x = tid; x < m; x += kThreads)
    put(x < n_lt ? x : x + n_eq, L.k[cur][x], L.v[cur][x]);
  return true;
}

// First position of the sorted run kv in [lo, hi) whose key is above k; the
// whole wave searches, 64 positions a round.
__device__ uint32_t wave_upper(const uint32_t* kv, uint32_t lo, uint32_t hi, uint32_t k) {
  const uint32_t lane = lane_id();
  while (lo < hi) {
    const uint32_t len = hi - lo, step = (len + 63u) / 64u;
    const uint64_t at = static_cast<uint64_t>(lo) + static_cast<uint64_t>(lane + 1) * step - 1;
    const bool below = at < hi && (as_global(kv)[at] >> 1) <= k;
    const uint32_t c = static_cast<uint32_t>(__popcll(ballot(below)));
    const uint64_t nlo = static_cast<uint64_t>(lo) + static_cast<uint64_t>(c) * step;
    const uint64_t nhi = nlo + step - 1;
    lo = nlo < hi ? static_cast<uint32_t>(nlo) : hi;
    hi = nhi < hi ? static_cast<uint32_t>(nhi) : hi;
  }
  return lo;
}

// Merges R sorted runs in global memory (L.run_k / L.run_v, L.len elements
// each, newest first, L.cur = 0) and calls out(i, kv, value) for every output
// position i in turn, newer elements first on equal original keys.  The runs
// are taken part by part: a share of each (by its length) is read into LDS;
// what lies below the smallest last key among the parts that do not end their
// run is complete and is merged pairwise, as the cascade merges whole levels.
// When nothing lies below it, a run of that key fills its part: then the key's
// whole runs are copied, newest first.  Hot keys and padding, which make a
// bucket large, so cost a copy: a bucket with 25 000 copies of one key takes
// about 30 us, 330 when every element was ranked by searches in the others.
template <typename Out>
__device__ __forceinline__ void merge_large(LocalLds& L, int R, Out out) {
  const uint32_t tid = threadIdx.x, wave = tid >> 6;
  constexpr int kPer = kLocalCap / kThreads;
  uint32_t o = 0;
  for (;;) {
    uint32_t rest = 0;
    for (int r = 0; r < R; ++r) rest += L.len[r] - L.cur[r];
    if (rest == 0) break;
    if (tid == 0) {
      uint32_t at = 0;
      for (int r = 0; r < R; ++r) {
        const uint32_t m = L.len[r] - L.cur[r];
        const uint32_t share = static_cast<uint32_t>(
            static_cast<uint64_t>(kLocalCap - kMaxFuse - 1) * m / rest) + 1u;
        L.win[r] = at;
        at += rest <= static_cast<uint32_t>(kLocalCap) || m < share ? m : share;
      }
      L.win[R] = at;
    }
    __syncthreads();
    const uint32_t W = L.win[R];
    uint32_t rk[kPer], rv[kPer], run[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const uint32_t x = tid + i * kThreads;
      run[i] = 0;
      if (x < W) {
        uint32_t r = 0;
        while (static_cast<int>(r) + 1 < R && L.win[r + 1] <= x) ++r;
        const uint32_t at = L.cur[r] + (x - L.win[r]);
        run[i] = r;
        rk[i] = as_global(L.run_k[r])[at];
        rv[i] = as_global(L.run_v[r])[at];
      }
    }
    // Run r's part goes where the pairwise merges find it: run 0 in buffer 0,
    // run r in the buffer that the merge of run r - 1 has left its output in.
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const uint32_t x = tid + i * kThreads;
      if (x < W) {
        const int to = run[i] == 0 || (run[i] & 1u) != 0 ? 0 : 1;
        L.k[to][x] = rk[i];
        L.v[to][x] = rv[i];
      }
    }
    __syncthreads();
    uint32_t B = 0xFFFFFFFFu;
    for (int r = 0; r < R; ++r) {
      const uint32_t w0 = L.win[r], w1 = L.win[r + 1];
      if (w1 > w0 && w1 - w0 < L.len[r] - L.cur[r]) {
        const uint32_t last = L.k[r == 0 || (r & 1) ? 0 : 1][w1 - 1] >> 1;
        B = last < B ? last : B;
      }
    }
    if (tid < static_cast<uint32_t>(R)) {
      const uint32_t w0 = L.win[tid], w1 = L.win[tid + 1];
      L.cut[tid] = B == 0xFFFFFFFFu
                       ? w1 - w0
                       : seg_bound(L.k[tid == 0 || (tid & 1u) ? 0 : 1], w0, w1, B, false) - w0;
    }
    __syncthreads();
    uint32_t total = 0;
    for (int r = 0; r < R; ++r) total += L.cut[r];
    if (total != 0) {
      int acc = 0;
      uint32_t A = L.cut[0];
      for (int r = 1; r < R; ++r) {
        const uint32_t c = L.cut[r];
        lds_merge_pair(L.k[acc], L.v[acc], A, L.win[r], c, L.k[1 - acc], L.v[1 - acc]);
        acc = 1 - acc;
        A += c;
      }
      for (uint32_t x = tid; x < total; x += kThreads) out(o + x, L.k[acc][x], L.v[acc][x]);
      if (tid < static_cast<uint32_t>(R)) L.cur[tid] += L.cut[tid];
    } else {
      // The runs of key B (a run that does not start with it has none here).
      // Their lengths go to L.cut, which every wave has to have summed first.
      __syncthreads();
      for (int r = static_cast<int>(wave); r < R; r += kWaves) {
        const uint32_t e = wave_upper(L.run_k[r], L.cur[r], L.len[r], B);
        if ((tid & 63u) == 0) L.cut[r] = e - L.cur[r];
      }
      __syncthreads();
      for (int r = 0; r < R; ++r) {
        const uint32_t c = L.cut[r], at = L.cur[r];
        const uint32_t* k = L.run_k[r];
        const uint32_t* v = L.run_v[r];
        for (uint32_t x0 = 0; x0 < c; x0 += 8 * kThreads) {
          uint32_t ck[8], cv[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const uint32_t x = x0 + i * kThreads + tid, xc = at + (x < c ? x : c - 1);
            ck[i] = as_global(k)[xc];
            cv[i] = as_global(v)[xc];
          }
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const uint32_t x = x0 + i * kThreads + tid;
            if (x < c) out(o + total + x, ck[i], cv[i]);
          }
        }
        total += c;
      }
      __syncthreads();
      if (tid < static_cast<uint32_t>(R)) L.cur[tid] += L.cut[tid];
    }
    o += total;
    __syncthreads();
  }
}

// One work-group per top-digit bucket d.  The bucket is digit d's group in
// every tile of the tile-major scatter, gathered in tile order (the batch's
// order), and is sorted on the digits below the top one: by ranking up to
// kRankSortMax elements, by LDS radix passes up to kLocalCap, above by setting
// its hot key aside (sort_hot) or, without one, by streaming passes over global
// memory.  Without a fused cascade the sorted bucket is the output.
//
// With a fused cascade (a.fuse.nlev = j > 0), the work-group then merges
// its bucket with the same digit's key range of levels 0..j-1 (read from
// each level's top-digit index) and writes that part of level j, recording
// where it starts in level j's index.  Runs fitting in LDS are merged there
// pairwise, newest first, exactly as the cascade merges whole levels; larger
// ones part by part from global memory (merge_large), in the same order.
// Without fusion, the sort of a level records its buckets'
// starts as that level's top-digit index.
// kPads: some batch of the group is padded (another instantiation, so that full
// batches pay nothing for it).
template <bool kPads>
__device__ void bucket_sort(const SortArgs& a, int lo_bit, int passes, uint32_t d, LocalLds& L) {
  const uint32_t tid = threadIdx.x;
  const SortMeta& m = a.meta;
  const FuseArgs& f = a.fuse;
  const bool fused = f.nlev > 0;
  const int R = f.nlev + 1;  // runs: the batch, then levels 0..j-1
  // Bucket d is digit d's group in every tile of the tile-major scatter, in
  // tile order; its sorted output starts at s, the number of batch elements
  // with a smaller digit, which is the sum over the tiles of the start of
  // digit d's group.  Every load of this prologue is issued unconditionally
  // (clamped index), so each tile's group bounds and the levels' digit
  // ranges are in flight together.
  auto next_of = [](uint32_t q) { return q + 1 < kTopBuckets ? q + 1 : q; };
  // A group (consecutive batches sorted together, the newer first on equal
  // keys) has the newest batch's tiles, then the next older batch's, and so
  // on: nta group-table entries, one per thread.
  const uint32_t G = a.group;
  auto tiles_of = [&](uint32_t q) {
    return q < G ? (kPads ? (a.grp_real[q] + kSortTile - 1) / kSortTile : m.num_sort_tiles) : 0u;
  };
  const uint32_t t1 = tiles_of(0), t2 = t1 + tiles_of(1), t3 = t2 + tiles_of(2);
  const uint32_t nta = t3 + tiles_of(3);
  static_assert(kMsdMaxTiles <= kThreads, "one tile per thread");
  static_assert(kMaxGroup == 4, "the batch of a tile is chosen among four");
  const uint32_t bq = tid >= nta ? 0u
                    : (tid >= t1 ? 1u : 0u) + (tid >= t2 ? 1u : 0u) +
                          (tid >= t3 ? 1u : 0u);  // the tile's batch in the group
  const uint32_t tt = tid < nta ? tid - (bq == 0 ? 0u : bq == 1 ? t1 : bq == 2 ? t2 : t3)
                                : 0u;  // tile in its batch
  const uint32_t real_q = !kPads  ? a.src.b
                        : bq == 0 ? a.grp_real[0] : bq == 1 ? a.grp_real[1]
                        : bq == 2 ? a.grp_real[2] : a.grp_real[3];
  const uint32_t* cnt_q = bq == 0 ? a.grp_cnt[0] : bq == 1 ? a.grp_cnt[1]
                        : bq == 2 ? a.grp_cnt[2] : a.grp_cnt[3];
  const uint32_t off_q = bq == 0 ? a.grp_off[0] : bq == 1 ? a.grp_off[1]
                       : bq == 2 ? a.grp_off[2] : a.grp_off[3];
  const uint32_t* row = cnt_q + static_cast<size_t>(tt) * (kTopBuckets / 2);
  const uint32_t seg_w0 = row[d >> 1];
  const uint32_t seg_w1 = row[next_of(d) >> 1];
  // The digit's range in each fused level, from the level's top-digit index:
  // uniform loads, all issued before any is used (slots past j read level
  // 0's index and are ignored).
  uint32_t dlo[kMaxFuse], dhi[kMaxFuse], dlen[kMaxFuse];
  if (fused) {
#pragma unroll
    for (int q = 0; q < kMaxFuse; ++q) {
      const uint32_t* dp = f.digit[q < f.nlev ? q : 0];
      dlo[q] = dp[d];
      dhi[q] = dp[next_of(d)];
      dlen[q] = q < f.nlev ? f.len[q] : 0u;
    }
  } else {
#pragma unroll
    for (int q = 0; q < kMaxFuse; ++q) dlo[q] = dhi[q] = dlen[q] = 0u;
  }
  // The group of digit d in tile t = tid: [start_t[d], start_t[d + 1]) of
  // the tile (the last digit's ends at the tile's size).
  const uint32_t g_st = (d & 1) ? seg_w0 >> 16 : seg_w0 & 0xFFFFu;
  const uint32_t tile_n =
      tid < nta ? min(real_q - tt * kSortTile, static_cast<uint32_t>(kSortTile)) : 0u;
  const uint32_t g_en = d + 1 < kTopBuckets ? (((d + 1) & 1) ? seg_w1 >> 16 : seg_w1 & 0xFFFFu)
                                            : tile_n;
  const uint32_t g_c = (tid < nta && g_en > g_st) ? g_en - g_st : 0u;
  // One pass of two scans: the group starts (their total is the bucket's
  // output start) and the group sizes (each group's first position in the
  // bucket; their total is the bucket's size).
  const uint32_t g_s0 = tid < nta ? g_st : 0u;
  uint32_t ssum = g_s0, csum = g_c;
  block_excl_scan2(ssum, csum, L.tmp);
  uint32_t* segb = &L.wcnt[0][0] + (kRankSortMax + 8);  // group sources in the batch
  uint32_t* segp = segb + kMsdMaxTiles;                  // group starts in the bucket
  static_assert(kRankSortMax + 8 + 2 * kMsdMaxTiles <= kWaves * kRadix,
                "group tables fit beside the rank-sort keys");
  if (tid < nta) {
    segb[tid] = off_q + tt * kSortTile + g_st;
    segp[tid] = csum;
  }
  if (tid == kThreads - 1) {
    L.tmp[2 * kWaves] = ssum + g_s0;
    L.tmp[2 * kWaves + 1] = csum + g_c;
  }
  if (tid == 0) {  // run 0 of the load table: the scattered batch
    L.run_k[0] = a.tmp_kv[0];
    L.run_v[0] = a.tmp_val[0];
    L.run_delta[0] = 0;
  }
  __syncthreads();
  uint32_t s = L.tmp[2 * kWaves];
  const uint32_t n = L.tmp[2 * kWaves + 1];
  // Padding: the copies of smaller digits come before this bucket, and `here`
  // has a bit for every batch whose copies belong into it.
  uint32_t here = 0u, pad_kv[kMaxGroup], pad_n[kMaxGroup];
  if constexpr (kPads) {
#pragma unroll
    for (uint32_t q = 0; q < kMaxGroup; ++q) {
      pad_n[q] = q < G ? a.src.b - a.grp_real[q] : 0u;
      pad_kv[q] = pad_n[q] != 0 ? a.grp_pad[q][0] : 0u;
      const uint32_t pd = (pad_kv[q] >> a.pad_shift) & (kTopBuckets - 1);
      s += pad_n[q] != 0 && pd < d ? pad_n[q] : 0u;
      here |= pad_n[q] != 0 && pd == d ? 1u << q : 0u;
    }
  }
  // Place in the bucket's output (padding included) of its element x.
  auto place = [&](uint32_t x) {
    uint32_t p = x;
    if (kPads && here != 0) {
#pragma unroll
      for (uint32_t q = 0; q < kMaxGroup; ++q)
        p += ((here >> q) & 1u) != 0 && x >= L.pad_at[q] ? pad_n[q] : 0u;
    }
    return p;
  };
  // Writes the bucket's padding; o: the output position of its first element.
  // One work-group writes all of a batch's copies, four a store (the outputs are
  // 16-byte aligned): 32 partly filled batches of 2^19 take 1719 us, 4081 with one
  // a store (3550 by digit passes); 255 of 2^16 3436, 4566.
  auto write_pads = [&](uint32_t* kv, uint32_t* val, uint32_t* fence, uint64_t len, uint64_t o) {
    if (!kPads || here == 0) return;
#pragma unroll
    for (uint32_t q = 0; q < kMaxGroup; ++q) {
      if (((here >> q) & 1u) == 0) continue;
      uint64_t p = o + L.pad_at[q];
#pragma unroll
      for (uint32_t y = 0; y < kMaxGroup; ++y)
        p += ((here >> y) & 1u) != 0 && L.pad_at[y] < L.pad_at[q] ? pad_n[y] : 0u;
      const uint64_t e = p + pad_n[q] < len ? p + pad_n[q] : len;
      const uint32_t v = a.grp_pad[q][1];
      const uint64_t p4 = min((p + 3) & ~uint64_t(3), e), e4 = max(e & ~uint64_t(3), p4);
      // Up to three copies before the first aligned place and after the last.
      const uint64_t edge = tid < p4 - p ? p + tid : e4 + (tid - (p4 - p));
      if (edge < (tid < p4 - p ? p4 : e)) {
        kv[edge] = pad_kv[q];
        val[edge] = v;
      }
      const uint4 k4 = make_uint4(pad_kv[q], pad_kv[q], pad_kv[q], pad_kv[q]), v4 = make_uint4(v, v, v, v);
      for (uint64_t x = p4 + 4 * tid; x < e4; x += 4 * kThreads) {
        *reinterpret_cast<uint4*>(kv + x) = k4;
        *reinterpret_cast<uint4*>(val + x) = v4;
      }
      if (fence != nullptr)
        for (uint64_t x = ((p + 31) & ~uint64_t(31)) + 32 * tid; x < e; x += 32 * kThreads)
          put_fence(fence, len, x, pad_kv[q]);
    }
  };
  if (kPads && tid < kMaxGroup) L.pad_at[tid] = 0u;
  // The sort's largest bucket, for the choice of the next sorts' path and
  // fused depth (only sizes that can change those choices are recorded).
  // Bucket d's size (for a group, its share per batch) goes to the record of
  // every batch's slot with a plain store: every bucket sort writes all of
  // a record, so no atomics and no clearing are needed; the next scatter
  // into any of the slots takes the largest entry.
  uint32_t* rec = tid == 0 ? a.grp_n[0] : tid == 1 ? a.grp_n[1]
                : tid == 2 ? a.grp_n[2] : a.grp_n[3];
  if (tid < G) rec[d] = (n + G - 1) / G;
  if (!fused && a.out_digit != nullptr && tid == 0) a.out_digit[d] = s;
  if (n == 0 && !fused) return;

  // Run starts in the concatenation (the batch's bucket, then each level's
  // range) and the first output position, computed by every thread (uniform
  // values); thread 0 also keeps them in LDS for the merge code below.
  uint32_t lo_q[kMaxFuse], rs_q[kMaxFuse + 2];
  rs_q[0] = 0;
  rs_q[1] = n;
  uint64_t out0 = s;
  uint32_t T = n;
#pragma unroll
  for (int q = 0; q < kMaxFuse; ++q) {
    const bool on = q < f.nlev;
    const uint32_t len = dlen[q];
    const uint32_t lo = dlo[q] < len ? dlo[q] : len;
    const uint32_t hi_d = d == kTopBuckets - 1 ? len : dhi[q];
    const uint32_t hi = hi_d < lo ? lo : (hi_d < len ? hi_d : len);
    lo_q[q] = lo;
    rs_q[q + 2] = rs_q[q + 1] + (hi - lo);
    out0 += lo;
    T += hi - lo;
    if (on && tid == 0) {
      L.lo[q] = lo;
      L.rs[q + 2] = rs_q[q + 2];
    }
  }
  if (fused && tid == 0) {
    L.rs[0] = 0;
    L.rs[1] = n;
    if (f.out_digit != nullptr) f.out_digit[d] = static_cast<uint32_t>(out0);
  }
  if (T == 0) return;

  // ---- one load phase.  The batch's bucket goes to buffer 0 (the sort's
  // input); when all runs fit in LDS, level l's range goes to its place in
  // [n, T) of buffer buf (l even) or 1 - buf (l odd), buf being the buffer
  // the sorted bucket ends in (the rank sort writes buffer 1, the radix
  // passes alternate from buffer 0): the cascade below then finds each run
  // next to the accumulated one.  Up to kLocalCap / kThreads elements per
  // thread, loads issued unconditionally (clamped position) before any is
  // stored.
  const bool rank_path = n <= kRankSortMax;
  const int buf = (rank_path || (passes & 1)) ? 1 : 0;
  const uint32_t nl = T <= static_cast<uint32_t>(kLocalCap) ? T
                      : (n <= static_cast<uint32_t>(kLocalCap) ? n : 0u);
  // The bits below the top digit: at most 32 - kTopBits, so 8 passes <= 24
  // and the rank sort's (field << 8) | position fits 32 bits.
  static_assert(32 - kTopBits <= 3 * kRadixBits, "local passes <= 3");
  const uint32_t fmask = (kRadixBits * passes >= 24) ? 0xFFFFFFu
                                                     : ((1u << (kRadixBits * passes)) - 1u);
  uint32_t* fld = &L.wcnt[0][0];  // rank-sort keys
  static_assert(kWaves * kRadix >= kRankSortMax + 8, "field scratch");
  const bool levels_in_lds = nl > n;  // fused, and all runs fit
  if (levels_in_lds) {
    // Run table: run q + 1 is level q, whose element x is source position
    // x + delta[q + 1]; run 0, the batch's bucket (written in the
    // prologue), is read through the group table instead.
    if (tid == 0) {
#pragma unroll
      for (int q = 0; q < kMaxFuse; ++q) {
        if (q < f.nlev) {
          L.run_k[q + 1] = f.kv[q];
          L.run_v[q + 1] = f.val[q];
          L.run_delta[q + 1] = lo_q[q] - rs_q[q + 1];
        }
      }
    }
    __syncthreads();
  }
  // The load phase for at most kPer items per thread (instantiated for 1,
  // 4 and 8, so that a small bucket does not search for absent items).
  auto load_phase = [&](auto per_c) {
    constexpr int kPer = decltype(per_c)::value;
    uint32_t rk[kPer], rv[kPer], run[kPer];
    // Each element's run (the number of level starts at or below it); a
    // batch element's position in the scattered batch comes from its
    // tile's group (the last group starting at or below it, by a search
    // over the group starts, the searches of a thread's elements in
    // lockstep), a level element's from the run table; loads issued before
    // any store.
    uint32_t bidx[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const uint32_t x = tid + i * kThreads;
      const uint32_t xc = x < nl ? x : nl - 1;
      run[i] = 0;
      if (levels_in_lds) {
#pragma unroll
        for (int q = 1; q <= kMaxFuse; ++q) run[i] += (q <= f.nlev && xc >= rs_q[q]) ? 1u : 0u;
      }
      bidx[i] = 0;
    }
    // Straight-line searches and table reads for every item (positions
    // clamped, results of items past nl unused), so that the LDS reads of
    // all items are in flight together and the loads below issue back to
    // back.
    // Only items that can hold batch elements search (all kPer, or just the
    // first when the bucket fits one item per thread).
    const uint32_t xbmax = n > 0 ? n - 1 : 0u;
    auto search = [&](auto cnt_c) {
      constexpr int kS = decltype(cnt_c)::value;
      for (uint32_t step = 1u << (31 - __builtin_clz(nta)); step > 0; step >>= 1) {
#pragma unroll
        for (int i = 0; i < kS; ++i) {
          const uint32_t x = tid + i * kThreads;
          const uint32_t xb = x < xbmax ? x : xbmax;
          const uint32_t probe = bidx[i] + step;
          const uint32_t pc = probe < nta ? probe : nta - 1;
          const uint32_t v = segp[pc];
          bidx[i] = ((probe < nta) & (v <= xb)) ? probe : bidx[i];
        }
      }
    };
    if (n <= static_cast<uint32_t>(kThreads))
      search(std::integral_constant<int, 1>{});
    else
      search(std::integral_constant<int, kPer>{});
    const uint32_t* pk[kPer];
    const uint32_t* pv[kPer];
    uint32_t at[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const uint32_t x = tid + i * kThreads;
      const uint32_t xc = x < nl ? x : nl - 1;
      const uint32_t xb = x < xbmax ? x : xbmax;
      const uint32_t r = levels_in_lds ? run[i] : 0u;
      const uint32_t gb = segb[bidx[i]], gp = segp[bidx[i]];
      pk[i] = L.run_k[r];
      pv[i] = L.run_v[r];
      at[i] = r == 0 ? gb + (xb - gp) : xc + L.run_delta[r];
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      if (static_cast<uint32_t>(i) * kThreads < nl) {
        rk[i] = as_global(pk[i])[at[i]];
        rv[i] = as_global(pv[i])[at[i]];
      }
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const uint32_t x = tid + i * kThreads;
      if (static_cast<uint32_t>(i) * kThreads < nl && x < nl) {
        const int to = x < n ? 0 : ((run[i] & 1u) ? buf : 1 - buf);
        L.k[to][x] = rk[i];
        L.v[to][x] = rv[i];
        if (rank_path && x < n) fld[x] = (((rk[i] >> lo_bit) & fmask) << 8) | x;
      }
    }
    if (rank_path && tid >= n && tid < ((n + 7u) & ~7u)) fld[tid] = 0xFFFFFFFFu;
  };
  if (nl > 0) {
    if (nl <= static_cast<uint32_t>(kThreads))
      load_phase(std::integral_constant<int, 1>{});
    else if (nl <= static_cast<uint32_t>(4 * kThreads))
      load_phase(std::integral_constant<int, 4>{});
    else
      load_phase(std::integral_constant<int, kLocalCap / kThreads>{});
  }
  __syncthreads();  // the loaded runs, fields and L.lo / L.rs
  // A batch's padding stands before its last element, the first of its tile 0:
  // how many elements of the bucket come before that one, then how many of
  // the fused levels (those with a smaller key).
  if (kPads && here != 0) {
    if (n <= static_cast<uint32_t>(kLocalCap)) {
#pragma unroll
      for (uint32_t q = 0; q < kMaxGroup; ++q) {
        if (((here >> q) & 1u) == 0) continue;
        const uint32_t xq = segp[q == 0 ? 0u : q == 1 ? t1 : q == 2 ? t2 : t3];
        const uint32_t fq = (pad_kv[q] >> lo_bit) & fmask;
        uint32_t c = 0;
        for (uint32_t x = tid; x < n; x += kThreads) {
          const uint32_t f = (L.k[0][x] >> lo_bit) & fmask;
          c += f < fq || (f == fq && x < xq) ? 1u : 0u;
        }
        if (c != 0) atomicAdd(&L.pad_at[q], c);
      }
    }
    if (fused && tid < 32u && static_cast<int>(tid & 7u) < f.nlev && ((here >> (tid >> 3)) & 1u) != 0) {
      const uint32_t q = tid >> 3, l = tid & 7u;
      const uint32_t key = (q == 0 ? pad_kv[0] : q == 1 ? pad_kv[1] : q == 2 ? pad_kv[2] : pad_kv[3]) >> 1;
      const uint32_t b0 = L.rs[l + 1], b1 = L.rs[l + 2];
      const uint32_t c = levels_in_lds
                             ? seg_bound(L.k[((l + 1) & 1u) ? buf : 1 - buf], b0, b1, key, false) - b0
                             : seg_bound(f.kv[l] + L.lo[l], 0, b1 - b0, key, false);
      if (c != 0) atomicAdd(&L.pad_at[q], c);
    }
    __syncthreads();
  }

  // ---- sort the batch's bucket.  sorted_lds: it ends in LDS buffer buf, else
  // in global memory (at out_k / out_v).
  uint32_t* out_k = a.out_kv + s;
  uint32_t* out_v = a.out_val + s;
  bool sorted_lds = true;
  if (n == 0) {
  } else if (rank_path) {
    rank_sort(L, fld, n);
  } else if (n <= static_cast<uint32_t>(kLocalCap)) {
    int cur = 0;
    for (int p = 0; p < passes; ++p) {
      lds_pass(L, cur, n, lo_bit + kRadixBits * p);
      cur = 1 - cur;
    }
  } else {
    sorted_lds = false;
    if (kPads && here != 0) {
#pragma unroll
      for (uint32_t q = 0; q < kMaxGroup; ++q) {
        if (((here >> q) & 1u) == 0) continue;
        const uint32_t tq = q == 0 ? 0u : q == 1 ? t1 : q == 2 ? t2 : t3;
        const uint32_t fq = (pad_kv[q] >> lo_bit) & fmask;
        uint32_t c = 0;
        for (uint32_t g = 0; g < nta; ++g) {
          const uint32_t end = g + 1 < nta ? segp[g + 1] : n;
          for (uint32_t x = segp[g] + tid; x < end; x += kThreads) {
            const uint32_t y = (a.tmp_kv[0][segb[g] + (x - segp[g])] >> lo_bit) & fmask;
            c += y < fq || (y == fq && x < segp[tq]) ? 1u : 0u;
          }
        }
        if (c != 0) atomicAdd(&L.pad_at[q], c);
      }
    }
    if (kPads) __syncthreads();  // the paddings' places
    const bool hot = sort_hot(a, lo_bit, passes, fmask, n, L, fld, segb, segp, nta,
                              [&](uint32_t x, uint32_t k, uint32_t v) {
                                const uint32_t p = fused ? x : place(x);
                                out_k[p] = k;
                                out_v[p] = v;
                                if (!fused) put_fence(a.out_fence, a.out_n, s + p, k);
                              });
    if (!hot) {
      if (tid < G) rec[d] = large_bucket((n + G - 1) / G);
      const bool to_tmp = kPads && here != 0 && !fused;
      __syncthreads();
      local_sort_streaming(a, lo_bit, passes, s, n, L, segb, segp, nta, to_tmp);
      if (to_tmp) {
        __threadfence_block();
        __syncthreads();
        for (uint32_t x = tid; x < n; x += kThreads) {
          const uint32_t k = a.tmp_kv[1][s + x], p = place(x);
          out_k[p] = k;
          out_v[p] = a.tmp_val[1][s + x];
          put_fence(a.out_fence, a.out_n, s + p, k);
        }
      }
    }
  }

  if (!fused) {
    if (sorted_lds) {
      for (uint32_t x = tid; x < n; x += kThreads) {
        const uint32_t k = L.k[buf][x], p = place(x);
        out_k[p] = k;
        out_v[p] = L.v[buf][x];
        put_fence(a.out_fence, a.out_n, s + p, k);
      }
    }
    write_pads(a.out_kv, a.out_val, a.out_fence, a.out_n, s);
    return;
  }

  if (sorted_lds && T <= static_cast<uint32_t>(kLocalCap)) {
    // A pairwise cascade in LDS: the accumulated run (newer, [0, rs[q]))
    // and the next level's run (older, [rs[q], rs[q + 1]), loaded into the
    // same buffer) are merged into [0, rs[q + 1]) of the other buffer, which
    // holds no run still to be read there.
    int acc = buf;
    for (int q = 1; q < R; ++q) {
      const uint32_t A = L.rs[q], c = L.rs[q + 1] - L.rs[q];
      lds_merge_pair(L.k[acc], L.v[acc], A, A, c, L.k[1 - acc], L.v[1 - acc]);
      acc = 1 - acc;
    }
    for (uint32_t x = tid; x < T; x += kThreads) {
      const uint64_t pos = out0 + place(x);
      if (pos < f.out_len) {
        const uint32_t k = L.k[acc][x];
        f.out_kv[pos] = k;
        f.out_val[pos] = L.v[acc][x];
        put_fence(f.out_fence, f.out_len, pos, k);
      }
    }
    write_pads(f.out_kv, f.out_val, f.out_fence, f.out_len, out0);
    return;
  }

  // Runs too large for LDS: merged from global memory part by part.  The
  // batch's bucket is put in global scratch first (it may be in LDS).
  if (sorted_lds) {
    for (uint32_t x = tid; x < n; x += kThreads) {
      out_k[x] = L.k[buf][x];
      out_v[x] = L.v[buf][x];
    }
  }
  if (tid <= static_cast<uint32_t>(f.nlev)) {
    const uint32_t q = tid;
    L.run_k[q] = q == 0 ? out_k : f.kv[q - 1] + L.lo[q - 1];
    L.run_v[q] = q == 0 ? out_v : f.val[q - 1] + L.lo[q - 1];
    L.cur[q] = 0u;
    L.len[q] = L.rs[q + 1] - L.rs[q];
  }
  __threadfence_block();
  __syncthreads();
  merge_large(L, R, [&](uint32_t x, uint32_t k, uint32_t v) {
    const uint64_t pos = out0 + place(x);
    if (pos < f.out_len) {
      f.out_kv[pos] = k;
      f.out_val[pos] = v;
      put_fence(f.out_fence, f.out_len, pos, k);
    }
  });
  write_pads(f.out_kv, f.out_val, f.out_fence, f.out_len, out0);
}

// Bucket work-group w (counted from the first bucket work-group) takes top
// digit (w % 8) * 128 + w / 8: work-groups go to the 8 XCDs in turn, so the
// work-groups with one w % 8 share an XCD, take 128 consecutive digits and
// read each tile's groups (adjacent in the tile) through that XCD's L2.
__device__ __forceinline__ uint32_t xcd_digit(uint32_t w) {
  return (w & 7u) * (kTopBuckets / 8) + (w >> 3);
}

template <bool kPads>
__global__ __launch_bounds__(kThreads) void k_local_sort(SortArgs a, int lo_bit, int passes) {
  __shared__ LocalLds L;
  bucket_sort<kPads>(a, lo_bit, passes, xcd_digit(blockIdx.x), L);
}

// One step of the pipelined top-digit sort: the first work-groups scatter
// the tiles of the new batch (sc) into one scratch slot while the others
// sort the buckets of the previous batch (bk) out of the other slot, with
// its fused cascade.  The two halves share no memory except what each reads
// from earlier kernels, so they need no synchronisation.
union StepLds {
  ScatterLds S;
  LocalLds L;
};
static_assert(sizeof(ScatterLds) <= sizeof(LocalLds),
              "the scatter half must not raise the step's LDS above the bucket sort's");

template <bool kPads>
__global__ __launch_bounds__(kThreads) void k_sort_step(SortArgs bk, int lo_bit, int passes,
                                                        ScatterArgs sc) {
  __shared__ StepLds U;
  const uint32_t nt = (sc.src.n + kSortTile - 1) / kSortTile;
  if (blockIdx.x < nt) tile_scatter(sc, blockIdx.x, U.S);
  else bucket_sort<kPads>(bk, lo_bit, passes, xcd_digit(blockIdx.x - nt), U.L);
}

// ------------------------------------------------------------ merge
// Number of elements of a (the newer run) among the first `diag` outputs of
// the merge, a first on equal original keys.  The whole wave searches: each
// round tests 64 evenly spaced candidates of the open interval and keeps the
// gap where the predicate flips, so a run of 2^26 takes five rounds.
__device__ uint32_t wave_merge_path(const uint32_t* a, uint32_t na, const uint32_t* bb,
                                    uint32_t nb, uint64_t diag) {
  const uint32_t lane = lane_id();
  uint64_t lo = diag > nb ? diag - nb : 0;
  uint64_t hi = diag < na ? diag : na;
  while (hi > lo) {
    const uint64_t len = hi - lo;
    if (len <= 64) {
      bool p = false;
      if (lane < len) {
        const uint64_t i = lo + lane;
        p = (a[i] >> 1) <= (bb[diag - 1 - i] >> 1);
      }
      return static_cast<uint32_t>(lo + __popcll(ballot(p)));
    }
    const uint64_t pos = lo + ((lane + 1) * len) / 65;
    const bool p = (a[pos] >> 1) <= (bb[diag - 1 - pos] >> 1);
    const uint32_t c = static_cast<uint32_t>(__popcll(ballot(p)));
    if (c == 0) {
      hi = lo + len / 65;
    } else if (c == 64) {
      lo = lo + (64 * len) / 65 + 1;
    } else {
      const uint64_t plo = lo + (c * len) / 65;
      const uint64_t phi = lo + ((c + 1) * len) / 65;
      lo = plo + 1;
      hi = phi;
    }
  }
  return static_cast<uint32_t>(lo);
}


// Merge-path split inside the work-group's windows, held in circular LDS
// buffers: window a is positions [a0, a0 + wa) of run a at slots
// (a0 + i) & mask, window b likewise.  Returns how many of the first dt
// outputs come from a (a first on equal original keys).
__device__ __forceinline__ uint32_t ring_merge_path(const uint32_t* sa, uint32_t a0, uint32_t wa,
                                                    const uint32_t* sb, uint32_t b0, uint32_t wb,
                                                    uint32_t dt, uint32_t mask) {
  uint32_t lo = dt > wb ? dt - wb : 0, hi = dt < wa ? dt : wa;
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if ((sa[(a0 + mid) & mask] >> 1) <= (sb[(b0 + dt - 1 - mid) & mask] >> 1)) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// Merge of run a (newer) with run b (older) on the original key.  Each
// work-group produces one contiguous range of the output, found one of two
// ways:
//   * digit mode (both runs carry a top-digit index): work-group w takes the
//     top digits [w per_wg, (w + 1) per_wg); each index gives the range of its
//     run holding those digits, and the output range starts at the sum of the
//     two starts (equal keys share a digit, so no tie crosses a range
//     boundary).  No search at all.  The output's own index is the sum of the
//     two indexes, digit by digit.
//   * search mode: work-group w takes output tiles [w per_wg, (w + 1) per_wg)
//     and finds the splits at the start and the end of its range with two
//     wave searches in global memory (waves 0 and 1, side by side).
// The range is then produced tile by tile, the tiles anchored at 16-byte
// aligned output positions (the first tile of a range may start inside its
// tile).  Both runs' windows live in LDS ring buffers: a tile's outputs
// consume la elements of a and n - la of b, and the next tile loads exactly
// those counts; windows never extend past the range's end, so every input
// element is read from HBM once.  A window's new elements are all loaded
// before any is stored.  Each thread merges kMergeItems consecutive outputs
// and stores them with 16-byte stores.
struct MergeArgs {
  const uint32_t* a_kv;
  const uint32_t* a_val;
  const uint32_t* b_kv;
  const uint32_t* b_val;
  uint32_t na, nb;
  uint32_t* out_kv;
  uint32_t* out_val;
  uint32_t* out_fence;     // the output level's fence tree, or null
  const uint32_t* a_dig;   // top-digit indexes of both runs, or null
  const uint32_t* b_dig;
  uint32_t* out_dig;       // receives the output's index (both runs indexed), or null
  int digit_mode;          // partition by digit ranges (needs both indexes)
  uint32_t per_wg;         // digits (digit mode) or output tiles per work-group
};

template <int kMergeItems>
__global__ __launch_bounds__(kThreads) void k_merge(MergeArgs m) {
  constexpr uint32_t kMergeTile = kThreads * kMergeItems;
  constexpr uint32_t kMask = kMergeTile - 1;
  static_assert((kMergeTile & kMask) == 0, "merge tile must be a power of two");
  static_assert(kMergeItems % 4 == 0, "16-byte stores");
  __shared__ uint32_t sa_k[kMergeTile], sa_v[kMergeTile], sb_k[kMergeTile], sb_v[kMergeTile];
  __shared__ uint32_t s_split, s_split_end;
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t na = m.na, nb = m.nb;
  const uint64_t total = static_cast<uint64_t>(na) + nb;
  uint32_t a0, b0, a_lim, b_lim;  // the work-group consumes a[a0, a_lim), b[b0, b_lim)
  if (m.digit_mode) {
    const uint32_t q0 = blockIdx.x * m.per_wg;
    if (q0 >= kTopBuckets) return;
    const uint32_t q1 = min(q0 + m.per_wg, kTopBuckets);
    // Index entries are positions in their run; clamped so that a damaged
    // index can only give wrong output, never an access out of bounds.
    a0 = min(m.a_dig[q0], na);
    b0 = min(m.b_dig[q0], nb);
    a_lim = q1 < kTopBuckets ? min(max(m.a_dig[q1], a0), na) : na;
    b_lim = q1 < kTopBuckets ? min(max(m.b_dig[q1], b0), nb) : nb;
    if (m.out_dig != nullptr)
      for (uint32_t q = q0 + tid; q < q1; q += kThreads) m.out_dig[q] = m.a_dig[q] + m.b_dig[q];
  } else {
    if (m.out_dig != nullptr)
      for (uint32_t q = blockIdx.x * kThreads + tid; q < kTopBuckets; q += gridDim.x * kThreads)
        m.out_dig[q] = m.a_dig[q] + m.b_dig[q];
    const uint64_t tiles = (total + kMergeTile - 1) / kMergeTile;
    const uint64_t t = static_cast<uint64_t>(blockIdx.x) * m.per_wg;
    const uint64_t t_end = (t + m.per_wg < tiles) ? t + m.per_wg : tiles;
    if (t >= t_end) return;
    if (wave == 0) {
      const uint32_t sp = wave_merge_path(m.a_kv, na, m.b_kv, nb, t * kMergeTile);
      if (lane == 0) s_split = sp;
    } else if (wave == 1) {
      const uint64_t de = t_end * kMergeTile;
      const uint32_t sp = de >= total ? na : wave_merge_path(m.a_kv, na, m.b_kv, nb, de);
      if (lane == 0) s_split_end = sp;
    }
    __syncthreads();
    a0 = s_split;
    b0 = static_cast<uint32_t>(t * kMergeTile - a0);
    a_lim = s_split_end;
    b_lim = static_cast<uint32_t>((t_end * kMergeTile < total ? t_end * kMergeTile : total) - a_lim);
  }
  const uint64_t o_end = static_cast<uint64_t>(a_lim) + b_lim;
  uint32_t a_end = a0, b_end = b0;  // loaded into the rings up to here
  // New window elements [from, to) of one run into its ring: at most
  // kMergeTile, so kMergeItems per thread; loads at clamped positions first.
  auto fill = [&](const uint32_t* gk, const uint32_t* gv, uint32_t from, uint32_t to,
                  uint32_t* rk_s, uint32_t* rv_s) {
    if (from >= to) return;
    uint32_t k[kMergeItems], v[kMergeItems];
#pragma unroll
    for (int j = 0; j < kMergeItems; ++j) {
      const uint32_t x = from + tid + static_cast<uint32_t>(j) * kThreads;
      const uint32_t xc = x < to ? x : to - 1;
      k[j] = gk[xc];
      v[j] = gv[xc];
    }
#pragma unroll
    for (int j = 0; j < kMergeItems; ++j) {
      const uint32_t x = from + tid + static_cast<uint32_t>(j) * kThreads;
      if (x < to) {
        rk_s[x & kMask] = k[j];
        rv_s[x & kMask] = v[j];
      }
    }
  };
  // Tiles anchored at 16-byte aligned output positions g0; the next output
  // is always at a0 + b0.
  for (uint64_t g0 = (static_cast<uint64_t>(a0) + b0) & ~uint64_t(3); g0 < o_end; g0 += kMergeTile) {
    const uint64_t p0 = static_cast<uint64_t>(a0) + b0;  // first output of this tile's part
    const uint64_t tile_end = (g0 + kMergeTile < o_end) ? g0 + kMergeTile : o_end;
    const uint32_t n = static_cast<uint32_t>(tile_end - p0);
    const uint32_t wa = (a_lim - a0) < n ? (a_lim - a0) : n;
    const uint32_t wb = (b_lim - b0) < n ? (b_lim - b0) : n;
    fill(m.a_kv, m.a_val, a_end, a0 + wa, sa_k, sa_v);
    fill(m.b_kv, m.b_val, b_end, b0 + wb, sb_k, sb_v);
    a_end = (a0 + wa > a_end) ? a0 + wa : a_end;
    b_end = (b0 + wb > b_end) ? b0 + wb : b_end;
    __syncthreads();
    // This thread's outputs: positions p .. p + kMergeItems - 1, of which
    // those before p0 (first tile of a range only) belong to another range.
    const uint64_t p = g0 + static_cast<uint64_t>(tid) * kMergeItems;
    const uint32_t skip =
        p < p0 ? ((p0 - p) < kMergeItems ? static_cast<uint32_t>(p0 - p) : kMergeItems) : 0u;
    const uint32_t dt = p < p0 ? 0u : ((p - p0) < n ? static_cast<uint32_t>(p - p0) : n);
    uint32_t ia = ring_merge_path(sa_k, a0, wa, sb_k, b0, wb, dt, kMask);
    uint32_t ib = dt - ia;
    uint32_t rk[kMergeItems], rv[kMergeItems];
#pragma unroll
    for (int k = 0; k < kMergeItems; ++k) {
      rk[k] = 0u;
      rv[k] = 0u;
      if (static_cast<uint32_t>(k) >= skip && p + k < tile_end) {
        const uint32_t ka = ia < wa ? sa_k[(a0 + ia) & kMask] : 0u;
        const uint32_t kb = ib < wb ? sb_k[(b0 + ib) & kMask] : 0u;
        const bool take_a = ia < wa && (ib >= wb || (ka >> 1) <= (kb >> 1));
        rk[k] = take_a ? ka : kb;
        rv[k] = take_a ? sa_v[(a0 + ia) & kMask] : sb_v[(b0 + ib) & kMask];
        ia += take_a ? 1u : 0u;
        ib += take_a ? 0u : 1u;
      }
    }
    if (tid == kThreads - 1) s_split = ring_merge_path(sa_k, a0, wa, sb_k, b0, wb, n, kMask);
    if (skip == 0 && p + kMergeItems <= tile_end) {
#pragma unroll
      for (int k = 0; k < kMergeItems; k += 4) {
        *reinterpret_cast<uint4*>(m.out_kv + p + k) = make_uint4(rk[k], rk[k + 1], rk[k + 2], rk[k + 3]);
        *reinterpret_cast<uint4*>(m.out_val + p + k) = make_uint4(rv[k], rv[k + 1], rv[k + 2], rv[k + 3]);
      }
    } else {
#pragma unroll
      for (int k = 0; k < kMergeItems; ++k) {
        if (static_cast<uint32_t>(k) >= skip && p + k < tile_end) {
          m.out_kv[p + k] = rk[k];
          m.out_val[p + k] = rv[k];
        }
      }
    }
#pragma unroll
    for (int k = 0; k < kMergeItems; ++k)
      if (static_cast<uint32_t>(k) >= skip && p + k < tile_end)
        put_fence(m.out_fence, total, p + k, rk[k]);
    __syncthreads();
    const uint32_t la = s_split;
    a0 += la;
    b0 += n - la;
  }
}

// ------------------------------------------------------------ coalescer
// Step a1 for the coalescer: encodes n operations as key variables (status
// 0 for a deletion, whose value is 0) into staging[at .. at + n).  Element i
// deletes when all_delete is set or is_delete[i] != 0.
__global__ __launch_bounds__(kThreads) void k_stage(const uint32_t* keys, const uint32_t* vals,
                                                    const uint8_t* is_delete, int all_delete,
                                                    uint32_t n, uint32_t* stage_kv,
                                                    uint32_t* stage_val, uint32_t at) {
  const uint32_t i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= n) return;
  const bool del = all_delete != 0 || (is_delete != nullptr && is_delete[i] != 0);
  stage_kv[at + i] = (keys[i] << 1) | (del ? 0u : 1u);
  stage_val[at + i] = del ? 0u : vals[i];
}

__global__ __launch_bounds__(kThreads) void k_check_keys(const uint32_t* keys, uint32_t n,
                                                         uint32_t limit_bits, int encoded,
                                                         uint32_t* err) {
  const uint32_t i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= n) return;
  const uint32_t k = encoded ? (keys[i] >> 1) : keys[i];
  if ((k >> limit_bits) != 0u) atomicOr(err, 1u);
}

__global__ __launch_bounds__(kThreads) void k_fill_runs(uint32_t* a_kv, uint32_t* a_val,
                                                        uint32_t* b_kv, uint32_t* b_val,
                                                        uint32_t n) {
  const uint32_t i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= n) return;
  a_kv[i] = ((2u * i) << 1) | 1u;
  a_val[i] = i;
  b_kv[i] = ((2u * i + 1u) << 1) | 1u;
  b_val[i] = i;
}

// ------------------------------------------------------------ queries
// What bounds lookups: with ten levels (2^26 elements) 12 lines a query come
// from memory, and 2^22 queries take 1.04 ms, 6.3 TB/s of such random lines
// (1.39 ms with whole descents: then the addresser and the longer chain of
// dependent loads bound it too); with one level 212 us (244).  Five waves a
// SIMD hide the chain; at four (98 registers) ten levels take 1.10 ms.
__global__ __launch_bounds__(kQueryThreads, 5) void k_lookup(QLevels lv,
                                                             const uint32_t* q, uint32_t nq,
                                                             uint32_t* out_val,
                                                             uint8_t* out_found) {
  extern __shared__ uint32_t top[];
  load_tops<kQueryThreads / 64>(lv, top);
  for (uint64_t q0 = static_cast<uint64_t>(blockIdx.x) * kQueryThreads; q0 < nq;
       q0 += static_cast<uint64_t>(gridDim.x) * kQueryThreads) {
    // Every lane stays until the wave is done: the searches are wave-wide.
    const uint64_t i = q0 + threadIdx.x;
    const bool active = i < nq;
    const uint32_t k = active ? q[i] : 0u;
    uint32_t kq[8];
    octet_lanes(k, kq);
    uint32_t v = 0u;
    uint8_t f = 0;
    bool done = !active;
    for (int l = 0; l < lv.count; ++l) {
      if (ballot(!done) == 0) break;
      bool hit;
      const uint32_t p = octet_bound<true, false, true>(lv, top, l, k, kq, &hit);
      if (!done && hit && p < lv.v[l].len) {
        const uint32_t x = lv.v[l].kv[p], y = lv.v[l].val[p];
        if ((x >> 1) == k) {
          if (x & 1u) {
            v = y;
            f = 1;
          }
          done = true;  // the newest instance decides, tombstone or not
        }
      }
    }
    if (active) {
      out_val[i] = v;
      out_found[i] = f;
    }
  }
}

// Few lookups: a work-group takes 64 queries and deals the levels to its waves
// (up to kFewWaves, each with every kFewWaves-th level), so that the descents,
// each a chain of dependent loads from memory, run side by side instead of one
// after another; the newest level's answer is chosen at the end.  64 lookups on
// five levels take 8 us, 22.5 level after level; 2^17 on ten take 60 us, 69.
constexpr uint32_t kFewWaves = 8;
static uint32_t few_waves(int levels) {
  const uint32_t n = levels > 0 ? static_cast<uint32_t>(levels) : 1u;
  return n < kFewWaves ? n : kFewWaves;
}

__global__ __launch_bounds__(64 * kFewWaves) void k_lookup_few(QLevels lv, const uint32_t* q,
                                                               uint32_t nq, uint32_t* out_val,
                                                               uint8_t* out_found) {
  // Per wave and query: 4 l + 2 + status of the element found, and its value.
  __shared__ uint32_t s_at[kFewWaves][64], s_val[kFewWaves][64];
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wave = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
  const uint32_t waves = blockDim.x >> 6;
  const uint32_t i = blockIdx.x * 64 + lane;
  const bool active = i < nq;
  const uint32_t k = active ? q[i] : 0u;
  uint32_t kq[8];
  octet_lanes(k, kq);
  uint32_t at = ~0u, v = 0u;
  for (int l = static_cast<int>(wave); l < lv.count; l += static_cast<int>(waves)) {
    if (ballot(at == ~0u) == 0) break;
    bool hit;
    const uint32_t p = octet_bound<false, false, true>(lv, nullptr, l, k, kq, &hit);
    if (at == ~0u && hit && p < lv.v[l].len) {
      const uint32_t x = lv.v[l].kv[p], y = lv.v[l].val[p];
      if ((x >> 1) == k) {
        at = 4u * static_cast<uint32_t>(l) + 2u + (x & 1u);
        v = y;
      }
    }
  }
  if (waves > 1) {
    s_at[wave][lane] = at;
    s_val[wave][lane] = v;
    __syncthreads();
    if (wave != 0) return;
    for (uint32_t w = 1; w < waves; ++w) {
      const uint32_t a = s_at[w][lane];
      if (a < at) {  // a newer level's (the levels differ)
        at = a;
        v = s_val[w][lane];
      }
    }
  }
  if (active) {
    const bool f = at != ~0u && (at & 1u) != 0u;
    out_val[i] = f ? v : 0u;
    out_found[i] = f ? 1 : 0;
  }
}

constexpr uint32_t kNoKey = 0xFFFFFFFFu;   // above every original key (< 2^31)
constexpr uint32_t kMaxKey = 0x7FFFFFFFu;  // largest encodable original key

// First index in (c, e) whose original key differs from k, where kv[c] has
// key k: one probe for the common run of length 1, then a galloping search,
// so long runs of one key (hot keys, padded batches) cost O(log run).
__device__ __forceinline__ uint32_t skip_run(const uint32_t* kv, uint32_t c, uint32_t e,
                                             uint32_t k) {
  uint32_t lo = c + 1;  // kv[lo - 1] has key k
  if (lo >= e || (kv[lo] >> 1) != k) return lo;
  uint32_t step = 1;
  // Invariant: kv[lo] has key k.
  while (lo + step < e && (kv[lo + step] >> 1) == k) {
    lo += step;
    step <<= 1;
  }
  uint32_t hi = (lo + step < e) ? lo + step : e;  // key(hi) > k, or hi == e
  while (hi - lo > 1) {
    const uint32_t mid = lo + ((hi - lo) >> 1);
    if ((kv[mid] >> 1) == k) lo = mid;
    else hi = mid;
  }
  return hi;
}

// One level: the live keys among the candidates of [k1, k2], from p =
// lower_bound(k1) (so the candidate at p starts a key run) to the first key
// above k2 or n, whichever comes first, which goes to *e.  The first element of
// every key run is that key's newest instance, so the candidates are
// scanned in order, 16 at a time (their loads independent); a chunk that
// holds no run start lies inside one long run, which is skipped by
// galloping.
__device__ __forceinline__ uint32_t count_run_starts(const uint32_t* kv, uint32_t p, uint32_t n,
                                                     uint32_t k2, uint32_t* e) {
  uint32_t count = 0, prev = kNoKey;
  while (p < n) {
    const uint32_t m = (n - p) < 16u ? (n - p) : 16u;
    uint32_t x[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      x[i] = static_cast<uint32_t>(i) < m ? kv[p + i] : 0u;
    }
    bool any_start = false;
    uint32_t stop = m;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (static_cast<uint32_t>(i) < stop) {
        const uint32_t key = x[i] >> 1;
        if (key > k2) {
          stop = static_cast<uint32_t>(i);
        } else {
          const bool start = key != prev;
          if (start && (x[i] & 1u)) ++count;
          any_start |= start;
          prev = key;
        }
      }
    }
    if (stop < m) {
      p += stop;
      break;
    }
    p = any_start ? p + m : skip_run(kv, p + m - 1, n, prev);
  }
  *e = p < n ? p : n;
  return count;
}

constexpr int kQueryWaves = kQueryThreads / 64;

// ---- Several levels.  The candidates of a query [k1, k2] in a level run from
// lower_bound(k1) up to the first key above k2.  The eight lanes of an octet
// work on one query: they read the next eight candidates of every level (16 of
// the two largest) with the loads of all levels in flight together, and merge
// what they have read in LDS.  2^20 ranges of 16 keys over ten levels are
// counted in 533 us and emitted in 538, about 22 lines of memory a query each
// (982 and 1003 us with one lane per query and one dependent load per
// candidate); 2^15 ranges of 512 keys in 1.1 and 2.1 ms (2.0 and 30.9).
//
// A wave's LDS: the cursors of its 64 queries (level l of query i at word
// 64 l + i), then one list of kv words (and, to emit, one of values) per octet.
struct WalkLds {
  uint32_t* cur;   // [levels][64]
  uint32_t* list;  // this octet's list
  uint32_t* vals;  // its values (emission only)
};
// List entries of an octet: a multiple of 4 words (16-byte reads), an odd one,
// so that the octets' lists start on different LDS banks.
__host__ __device__ constexpr uint32_t walk_list(uint32_t levels) {
  const uint32_t quads = 2 * levels + 4;  // 8 entries a level, 16 of two
  return 4u * (quads | 1u);
}
__host__ __device__ constexpr uint32_t walk_words(uint32_t levels, bool emit) {
  return 64u * levels + 8u * walk_list(levels) * (emit ? 2u : 1u);
}
// A work-group can have the 160 KB of its CU; with 32 levels the emission that
// searches takes 117 (64 KB from 20 levels on without tops, from 15 with them).
constexpr uint32_t kLdsBytes = 160 * 1024;
static_assert(4u * (kTopWords + kQueryWaves * walk_words(kMaxLevels, true)) <= kLdsBytes &&
                  4u * (64u * kMaxLevels + 8u * kFewWaves * walk_list(kMaxLevels)) <= kLdsBytes,
              "every number of levels fits");
__device__ __forceinline__ WalkLds walk_lds(uint32_t* wave_lds, uint32_t levels, bool emit) {
  const uint32_t octet = lane_id() >> 3, len = walk_list(levels);
  WalkLds w;
  w.cur = wave_lds;
  w.list = wave_lds + 64u * levels + octet * len;
  w.vals = emit ? w.list + 8u * len : nullptr;
  return w;
}

// Orders a wave's LDS accesses before and after it for the compiler (the
// hardware applies one wave's in issue order).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The octet's bits of a wave ballot.
__device__ __forceinline__ uint32_t octet_ballot(bool p) {
  const uint64_t m = ballot(p);
  return static_cast<uint32_t>(m >> (lane_id() & 56u)) & 0xFFu;
}

// One chunk of query `qi` of the wave (the same in all lanes of an octet, as h2
// and live): fills the octet's list with every element of every level from its
// cursor on whose key is at most k2 (kv word <= h2) and below the bound that
// makes the chunk complete, in level order (newest first), each level's in its
// own order, and moves the cursors past them.  The bound is the smallest last
// key among the levels that may hold more; *bound receives it (kNoKey: the
// query ends with this chunk).  Returns the list's length.  The two largest
// levels (16 elements each) are held in registers, the others pass through the
// list, eight levels' loads in flight, and are packed there in place.
template <bool kEmit>
__device__ __forceinline__ uint32_t walk_chunk(const QLevels& lv, const WalkLds& w, uint32_t qi,
                                               uint32_t h2, bool live, uint32_t* bound) {
  constexpr int kB = 8;
  const uint32_t sub = lane_id() & 7u;
  const int small = lv.count - 2;  // levels read eight at a time
  uint32_t xw[4], aw[4], in = 0u;  // elements 8 (y & 1) .. of level small + y / 2
#pragma unroll
  for (int y = 0; y < 4; ++y) {
    const int l = small + y / 2;
    aw[y] = w.cur[l * 64 + qi] + 8u * (y & 1) + sub;
    const bool ok = live && aw[y] < lv.v[l].len;
    xw[y] = ok ? lv.v[l].kv[aw[y]] : ~0u;
    in |= ok ? 1u << y : 0u;
  }
  wave_sync();  // the previous chunk's list has been read
  uint32_t B = kNoKey;
  for (int l0 = 0; l0 < small; l0 += kB) {
    uint32_t x[kB];
    bool ok[kB];
#pragma unroll
    for (int u = 0; u < kB; ++u) {
      const int l = l0 + u < small ? l0 + u : small;
      const uint32_t at = w.cur[l * 64 + qi] + sub;
      ok[u] = live && l < small && at < lv.v[l].len;
      x[u] = ok[u] ? lv.v[l].kv[at] : ~0u;
    }
#pragma unroll
    for (int u = 0; u < kB; ++u) {
      if (l0 + u < small) {
        const uint32_t last = octet_lane<7>(ok[u] && x[u] <= h2 ? x[u] >> 1 : kNoKey);
        B = last < B ? last : B;
        w.list[(l0 + u) * 8 + sub] = x[u];
      }
    }
  }
#pragma unroll
  for (int y = 0; y < 4; ++y) {
    const bool c = ((in >> y) & 1u) != 0u && xw[y] <= h2;
    in = c ? in : in & ~(1u << y);
    if (y & 1) {
      const uint32_t last = octet_lane<7>(c ? xw[y] >> 1 : kNoKey);
      B = last < B ? last : B;
    }
  }
  // What is in is a prefix of the lanes (a level's keys ascend).
  uint32_t vw[4];
#pragma unroll
  for (int y = 0; y < 4; ++y) {
    in = (xw[y] >> 1) < B ? in : in & ~(1u << y);
    vw[y] = kEmit && ((in >> y) & 1u) != 0u ? lv.v[small + y / 2].val[aw[y]] : 0u;
  }
  uint32_t n = 0;
  auto put = [&](uint32_t x, uint32_t v, bool mine) {
    if (mine) {
      w.list[n + sub] = x;
      if (kEmit) w.vals[n + sub] = v;
    }
    n += __popc(octet_ballot(mine));
  };
  for (int l0 = 0; l0 < small; l0 += kB) {
    uint32_t x[kB], v[kB], at[kB];
    bool mine[kB];
#pragma unroll
    for (int u = 0; u < kB; ++u) {
      const int l = l0 + u < small ? l0 + u : small;
      at[u] = w.cur[l * 64 + qi] + sub;
      x[u] = w.list[(l < small ? l : 0) * 8 + sub];
      mine[u] = live && l < small && at[u] < lv.v[l].len && x[u] <= h2 && (x[u] >> 1) < B;
      v[u] = kEmit && mine[u] ? lv.v[l].val[at[u]] : 0u;
    }
    wave_sync();
#pragma unroll
    for (int u = 0; u < kB; ++u) {
      if (l0 + u < small) {
        const uint32_t n0 = n;
        put(x[u], v[u], mine[u]);
        w.cur[(l0 + u) * 64 + qi] = at[u] - sub + (n - n0);  // all eight lanes, the same
      }
    }
  }
#pragma unroll
  for (int y = 0; y < 4; y += 2) {
    const uint32_t n0 = n;
    put(xw[y], vw[y], ((in >> y) & 1u) != 0u);
    put(xw[y + 1], vw[y + 1], ((in >> (y + 1)) & 1u) != 0u);
    w.cur[(small + y / 2) * 64 + qi] = aw[y] - sub + (n - n0);
  }
  // The last quad is filled up with words above every valid one.
  if (n + sub < ((n + 3u) & ~3u)) w.list[n + sub] = ~0u;
  wave_sync();
  *bound = B;
  return n;
}

// Whether list entry i is its key's newest instance in the list and regular.
__device__ __forceinline__ bool list_valid(const uint32_t* list, uint32_t i, uint32_t x) {
  uint32_t near = ~0u;  // zero when an earlier entry has x's key
  const uint4* q = reinterpret_cast<const uint4*>(list);
  for (uint32_t e = 0; e < i; e += 4) {
    const uint4 y = q[e >> 2];
    const uint32_t y4[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
    for (uint32_t r = 0; r < 4; ++r) {
      const uint32_t d = (y4[r] ^ x) >> 1;
      near = (e + r < i && d < near) ? d : near;
    }
  }
  return near != 0u && (x & 1u) != 0u;
}

// A chunk that holds nothing below its bound B starts with a run of key B that
// fills what was read of some level.  Finds B's newest instance (*x, and its
// value with kEmit) and moves every cursor past its run.
template <bool kEmit>
__device__ __forceinline__ void walk_run(const QLevels& lv, const WalkLds& w, uint32_t qi,
                                         uint32_t B, uint32_t* x, uint32_t* v) {
  bool found = false;
  for (int l = 0; l < lv.count; ++l) {
    const uint32_t p = w.cur[l * 64 + qi], n = lv.v[l].len;
    const uint32_t y = p < n ? lv.v[l].kv[p] : 0u;
    if (p >= n || (y >> 1) != B) continue;
    if (!found) {
      found = true;
      *x = y;
      if (kEmit) *v = lv.v[l].val[p];
    }
    w.cur[l * 64 + qi] = skip_run(lv.v[l].kv, p, n, B);  // all eight lanes, the same
  }
}

// This lane's share of the live keys of query qi (the same in all lanes of an
// octet; every lane of the wave calls it).
__device__ __forceinline__ uint32_t count_walk(const QLevels& lv, const WalkLds& w, uint32_t qi,
                                               uint32_t h, bool live) {
  const uint32_t sub = lane_id() & 7u;
  uint32_t c = 0;
  while (ballot(live) != 0) {
    uint32_t B;
    const uint32_t n = walk_chunk<false>(lv, w, qi, h, live, &B);
    for (uint32_t i = sub; i < n; i += 8) c += list_valid(w.list, i, w.list[i]) ? 1u : 0u;
    if (live && B != kNoKey && n == 0) {
      uint32_t x = 0u, v = 0u;
      walk_run<false>(lv, w, qi, B, &x, &v);
      if (sub == 0) c += x & 1u;
    }
    live = live && B != kNoKey;
  }
  return c;
}

// An octet takes `per` queries (1, 2, 4 or 8): the query of a lane, counted from
// the work-group's first.  With fewer than eight, lanes per .. 7 search along
// with their octet's queries again and keep nothing.
__device__ __forceinline__ uint32_t query_slot(uint32_t per) {
  return (threadIdx.x >> 3) * per + (threadIdx.x & (per - 1u));
}

// Count pass for few queries on several levels: 64 queries a work-group, the
// levels' descents dealt to its eight waves as for few lookups, then an octet a
// query: 3000 counts on five levels take 15 us, 28 with every wave
// descending all levels; 2^17 on ten take 80 us, 118.  Stores what k_count stores.
__global__ __launch_bounds__(64 * kFewWaves) void k_count_few(QLevels lv, const uint32_t* lo,
                                                              const uint32_t* hi, uint32_t nq,
                                                              uint32_t* counts,
                                                              uint64_t* scan_status,
                                                              uint64_t scan_words,
                                                              uint32_t* bounds) {
  extern __shared__ uint32_t top[];
  if (scan_status != nullptr)
    for (uint64_t w = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x; w < scan_words;
         w += static_cast<uint64_t>(gridDim.x) * blockDim.x)
      scan_status[w] = 0ull;
  const uint32_t lane = threadIdx.x & 63, sub = lane & 7u;
  const uint32_t wave = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
  const uint32_t waves = blockDim.x >> 6, L = static_cast<uint32_t>(lv.count);
  // One set of cursors for the work-group, a list for each octet.
  WalkLds w;
  w.cur = top;
  w.list = top + 64u * L + (threadIdx.x >> 3) * walk_list(L);
  w.vals = nullptr;
  const uint32_t gi = blockIdx.x * 64 + lane;
  const uint32_t k1 = gi < nq ? lo[gi] : 1u;
  uint32_t kq[8];
  octet_lanes(k1, kq);
  for (uint32_t l = wave; l < L; l += waves) {
    const uint32_t p =
        octet_bound<false, false, false>(lv, nullptr, static_cast<int>(l), k1, kq, nullptr);
    w.cur[l * 64 + lane] = p;
    if (bounds != nullptr && gi < nq) bounds[static_cast<size_t>(l) * nq + gi] = p;
  }
  __syncthreads();
  for (uint32_t qi = threadIdx.x >> 3; qi < 64u; qi += waves * 8u) {
    const uint32_t qg = blockIdx.x * 64 + qi;
    const uint32_t k2 = qg < nq ? hi[qg] : 0u;
    const uint32_t h = ((k2 < kMaxKey ? k2 : kMaxKey) << 1) | 1u;
    const uint32_t c = octet_sum(count_walk(lv, w, qi, h, qg < nq));
    if (sub == 0 && qg < nq) counts[qg] = c;
  }
}

// Queries of few candidates over at most kN levels: a lane walks its own query, the
// levels' next elements in registers.  A level has an element while its cursor is
// below its length: every 32-bit word is the key variable of some element (all ones
// that of key 2^31 - 1), so no word can stand for none.  (Octets need a round for
// each of a wave's queries, however few candidates it has.)
// kRuns: a step passes over a key's whole run in a level, else over one element,
// so that older elements of the key take steps of their own.  Whole runs cost the
// steps 5 to 10 % where the levels lie in the L2s, and single elements the ranges
// of four keys on larger levels 4 %: a key and its tombstone in one level are
// common, and every further step of one lane is one of the whole wave.
constexpr int kNarrowLevels = 10;
constexpr uint32_t kNarrowSteps = 40;
template <int kN, bool kRuns>
struct NarrowWalk {
  uint32_t c[kN], x[kN];
  uint32_t key, last;  // the step's key, and that of the step before
  uint32_t elem, at;   // the key's newest element and its place
  const uint32_t* val;

  // From the cursors in cur (word 64 l for level l); on: the lane has a query.
  __device__ __forceinline__ void start(const QLevels& lv, const uint32_t* cur, bool on) {
    key = kNoKey;
#pragma unroll
    for (int l = 0; l < kN; ++l)  // (levels past the last have length 0)
      c[l] = l < lv.count && on ? cur[l * 64] : lv.v[l].len;
#pragma unroll
    for (int l = 0; l < kN; ++l) x[l] = c[l] < lv.v[l].len ? lv.v[l].kv[c[l]] : 0u;
  }
  // The smallest key; false when there is none up to kv word h.
  __device__ __forceinline__ bool next(const QLevels& lv, uint32_t h) {
    last = key;
    key = kNoKey;
    elem = at = 0u;
    val = nullptr;
#pragma unroll
    for (int l = 0; l < kN; ++l) {
      if (c[l] < lv.v[l].len && x[l] <= h && (x[l] >> 1) < key) {  // ties: the newer level's stays
        key = x[l] >> 1;
        elem = x[l];
        at = c[l];
        val = lv.v[l].val;
      }
    }
    return key != kNoKey;
  }
  // Whether `elem` is a live pair: a regular element and not an older one of the
  // key of the step before.
  __device__ __forceinline__ bool live() const {
    return (kRuns || key != last) && (elem & 1u) != 0u;
  }
  // Past the key's run, or one element of it, in every level that has it.
  __device__ __forceinline__ void pass(const QLevels& lv) {
#pragma unroll
    for (int l = 0; l < kN; ++l) {
      if (c[l] < lv.v[l].len && (x[l] >> 1) == key) {
        ++c[l];
        x[l] = c[l] < lv.v[l].len ? lv.v[l].kv[c[l]] : 0u;
        if (kRuns && c[l] < lv.v[l].len && (x[l] >> 1) == key) {
          c[l] = skip_run(lv.v[l].kv, c[l], lv.v[l].len, key);
          x[l] = c[l] < lv.v[l].len ? lv.v[l].kv[c[l]] : 0u;
        }
      }
    }
  }
};

// Counts the wave's queries lane by lane.  False, with nothing counted, when some
// lane's query has more than `far` candidates in the largest level (the last) or
// takes more than kNarrowSteps steps.
template <int kN>
__device__ __forceinline__ bool count_narrow(const QLevels& lv, const uint32_t* cur, uint32_t h,
                                             uint32_t far, uint32_t* count) {
  const QLevel& last = lv.v[lv.count - 1];
  const uint32_t c = cur[(lv.count - 1) * 64];
  const bool reaches = c < last.len && last.len - c > far;
  const uint32_t z = reaches ? last.kv[c + far] : 0u;
  if (ballot(reaches && z <= h) != 0) return false;
  NarrowWalk<kN, false> w;
  w.start(lv, cur, true);
  uint32_t n = 0;
  bool more = true;
  for (uint32_t i = 0; i < kNarrowSteps && ballot(more) != 0; ++i) {
    more = w.next(lv, h);
    n += more && w.live() ? 1u : 0u;
    w.pass(lv);  // (no level has kNoKey)
  }
  *count = n;
  return ballot(more) == 0;
}

// Writes pairs [o, z) of the lane's query from the cursors in cur; gives up after
// kNarrowSteps steps (many deleted keys or long runs).  Returns whether every lane
// of the wave has written all its pairs; writing them again is harmless.
template <int kN, bool kRuns>
__device__ __forceinline__ bool emit_narrow(const QLevels& lv, const uint32_t* cur, uint32_t k2,
                                            uint64_t o, uint64_t z, uint32_t* out_keys,
                                            uint32_t* out_vals) {
  const uint32_t h = ((k2 < kMaxKey ? k2 : kMaxKey) << 1) | 1u;
  NarrowWalk<kN, kRuns> w;
  w.start(lv, cur, o < z);
  for (uint32_t i = 0; i < kNarrowSteps && ballot(o < z) != 0; ++i) {
    if (!w.next(lv, h)) break;  // no query, or only after a timed-out scan
    if (o < z && w.live()) {
      out_keys[o] = w.key;
      out_vals[o] = as_global(w.val)[w.at];
      ++o;
    }
    if (o < z) w.pass(lv);
  }
  return ballot(o < z) == 0;
}

// Count pass.  With bounds non-null, each query's position in the levels is
// stored for the emission pass: with one level its candidate bounds
// [lower_bound(lo), upper_bound(hi)) (two words per query), with several its
// cursors (lower bounds), level-major (word l * nq + query).
// kMany: several occupied levels; kN != 0: waves of few candidates (`far`) count
// lane by lane.
template <bool kTop, bool kMany, int kN>
__global__ __launch_bounds__(kQueryThreads) void k_count(QLevels lv,
                                                         const uint32_t* lo, const uint32_t* hi,
                                                         uint32_t nq, uint32_t far,
                                                         uint32_t* counts, uint64_t* scan_status,
                                                         uint64_t scan_words, uint32_t* bounds) {
  extern __shared__ uint32_t top[];
  if (scan_status != nullptr)
    for (uint64_t w = static_cast<uint64_t>(blockIdx.x) * kQueryThreads + threadIdx.x;
         w < scan_words; w += static_cast<uint64_t>(gridDim.x) * kQueryThreads)
      scan_status[w] = 0ull;
  if constexpr (kTop) load_tops<kQueryWaves>(lv, top);
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, sub = lane & 7u;
  const uint32_t L = static_cast<uint32_t>(lv.count);
  WalkLds w{};
  if (kMany) w = walk_lds(top + lv.words + wave * walk_words(L, false), L, false);
  for (uint64_t q0 = static_cast<uint64_t>(blockIdx.x) * kQueryThreads; q0 < nq;
       q0 += static_cast<uint64_t>(gridDim.x) * kQueryThreads) {
    // Every lane takes part in the wave-wide descents; lanes without a query
    // search the empty range [1, 0].
    const uint64_t gi = q0 + threadIdx.x;
    const bool active = gi < nq;
    const uint32_t k1 = active ? lo[gi] : 1u, k2 = active ? hi[gi] : 0u;
    uint32_t kq[8];
    octet_lanes(k1, kq);
    if constexpr (!kMany) {
      // Both bounds by descents, so the scan reads only the candidates.
      uint32_t p = octet_bound<kTop, false, false>(lv, top, 0, k1, kq, nullptr);
      octet_lanes(k2, kq);
      uint32_t e = octet_bound<kTop, true, false>(lv, top, 0, k2, kq, nullptr);
      if (!active) continue;
      uint32_t c = 0;
      if (k1 <= k2) c = count_run_starts(lv.v[0].kv, p, e, k2, &e);
      else p = e = 0;
      if (bounds != nullptr) reinterpret_cast<uint2*>(bounds)[gi] = make_uint2(p, e);
      counts[gi] = c;
    } else {
      for (uint32_t l = 0; l < L; ++l) {
        const uint32_t p =
            octet_bound<kTop, false, false>(lv, top, static_cast<int>(l), k1, kq, nullptr);
        w.cur[l * 64 + lane] = p;
        if (bounds != nullptr && active) bounds[static_cast<size_t>(l) * nq + gi] = p;
      }
      wave_sync();
      const uint32_t h2 = ((k2 < kMaxKey ? k2 : kMaxKey) << 1) | 1u;
      uint32_t res = 0;
      bool narrow = false;
      if constexpr (kN != 0) narrow = count_narrow<kN>(lv, w.cur + lane, h2, far, &res);
      if (narrow) {
        wave_sync();
        if (active) counts[gi] = res;
        continue;
      }
      for (uint32_t r = 0; r < 8; ++r) {
        const uint32_t qi = (lane & 56u) + r;
        const uint32_t h =
            static_cast<uint32_t>(__shfl(static_cast<int>(h2), static_cast<int>(qi), 64));
        const uint32_t c = octet_sum(count_walk(lv, w, qi, h, true));
        res = sub == r ? c : res;
      }
      if (active) counts[gi] = res;
    }
  }
}

// Stage 3 of sec. IV-C / IV-D over several levels.  An octet writes its
// query's pairs at the query's offset, chunk by chunk: a valid entry's place is
// the number of valid entries of the chunk with a smaller key.  A query whose
// pairs would end beyond cap writes nothing (the caller sees
// offsets[q + 1] > cap); writes stay inside [offsets[q], offsets[q + 1]) even
// for offsets corrupted by a timed-out scan.  Cursors as the count pass stored
// them, or, with kSearch, from descents.  kN != 0: waves whose queries all have at
// most narrow_max pairs emit lane by lane.  (Without the bound of five waves a
// SIMD the lane walk takes registers from the octets': 16 pairs a query on six
// levels 345 us with it, 389 without.)
template <bool kTop, bool kSearch, int kN, bool kRuns>
__global__ __launch_bounds__(kQueryThreads, kSearch ? 1 : 5) void k_range_emit(QLevels lv,
                                                              const uint32_t* lo,
                                                              const uint32_t* hi, uint32_t nq,
                                                              uint32_t per, uint32_t narrow_max,
                                                              const uint64_t* offsets,
                                                              const uint32_t* cursors,
                                                              uint32_t* out_keys,
                                                              uint32_t* out_vals, uint64_t cap) {
  extern __shared__ uint32_t top[];
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, sub = lane & 7u;
  const uint32_t L = static_cast<uint32_t>(lv.count);
  const WalkLds w = walk_lds(top + lv.words + wave * walk_words(L, true), L, true);
  if constexpr (kSearch && kTop) load_tops<kQueryWaves>(lv, top);
  const uint64_t all = offsets[nq];
  const uint32_t block = kQueryThreads / 8 * per, slot = query_slot(per);
  for (uint64_t q0 = static_cast<uint64_t>(blockIdx.x) * block; q0 < nq;
       q0 += static_cast<uint64_t>(gridDim.x) * block) {
    const uint64_t gi = q0 + slot;
    uint64_t o = 0, z = 0;
    if (gi < nq) {
      o = offsets[gi];
      z = offsets[gi + 1];
    }
    const bool emit = z > o && z <= all && z <= cap;
    if (!emit) z = o;
    const uint32_t k1 = emit ? lo[gi] : 1u, k2 = emit ? hi[gi] : 0u;
    if constexpr (kSearch) {
      uint32_t kq[8];
      octet_lanes(k1, kq);
      for (uint32_t l = 0; l < L; ++l)
        w.cur[l * 64 + lane] =
            octet_bound<kTop, false, false>(lv, top, static_cast<int>(l), k1, kq, nullptr);
    } else {
      if (emit)
        for (uint32_t l = 0; l < L; ++l)
          w.cur[l * 64 + lane] = cursors[static_cast<size_t>(l) * nq + gi];
    }
    wave_sync();
    const uint32_t h2 = ((k2 < kMaxKey ? k2 : kMaxKey) << 1) | 1u;
    bool narrow = false;
    if constexpr (kN != 0)
      narrow = per == 8 && ballot(z - o > narrow_max) == 0 &&
               emit_narrow<kN, kRuns>(lv, w.cur + lane, k2, o, z, out_keys, out_vals);
    if (narrow) {
      wave_sync();
      continue;
    }
    for (uint32_t r = 0; r < per; ++r) {
      const int qi = static_cast<int>((lane & 56u) + r);
      const uint32_t h = static_cast<uint32_t>(__shfl(static_cast<int>(h2), qi, 64));
      uint64_t at = __shfl(o, qi, 64);
      const uint64_t end = __shfl(z, qi, 64);
      bool live = at < end;
      while (ballot(live) != 0) {
        uint32_t B;
        const uint32_t n = walk_chunk<true>(lv, w, static_cast<uint32_t>(qi), h, live, &B);
        // Mark what is not valid, from the last entries down (an entry is
        // compared with those before it), then rank the rest.
        uint64_t mine = 0;  // this lane's valid entries, bit i / 8
        uint32_t total = 0;
        for (uint32_t i0 = n & ~7u;; i0 -= 8) {
          const uint32_t i = i0 + sub;
          const uint32_t x = i < n ? w.list[i] : 0u;
          const bool ok = i < n && list_valid(w.list, i, x);
          mine |= ok ? 1ull << (i0 >> 3) : 0ull;
          total += __popc(octet_ballot(ok));
          wave_sync();
          if (i < n && !ok) w.list[i] = ~0u;
          if (i0 == 0) break;
        }
        wave_sync();
        const uint4* q4 = reinterpret_cast<const uint4*>(w.list);
        for (uint32_t i = sub; i < n; i += 8) {
          if (((mine >> (i >> 3)) & 1ull) == 0) continue;
          const uint32_t x = w.list[i];
          uint32_t rank = 0;
          for (uint32_t e = 0; e < n; e += 4) {
            const uint4 y = q4[e >> 2];
            rank += (y.x < x ? 1u : 0u) + (y.y < x ? 1u : 0u) + (y.z < x ? 1u : 0u) +
                    (y.w < x ? 1u : 0u);
          }
          if (at + rank < end) {
            out_keys[at + rank] = x >> 1;
            out_vals[at + rank] = w.vals[i];
          }
        }
        at += total;
        if (live && B != kNoKey && n == 0) {
          uint32_t x = 0u, v = 0u;
          walk_run<true>(lv, w, static_cast<uint32_t>(qi), B, &x, &v);
          if ((x & 1u) != 0u && at < end) {
            if (sub == 0) {
              out_keys[at] = B;
              out_vals[at] = v;
            }
            ++at;
          }
        }
        live = live && B != kNoKey && at < end;
      }
    }
    wave_sync();  // the cursors have been read
  }
}

// Stage 3 of sec. IV-C / IV-D with one occupied level, a wave working on
// one query at a time: the 64 lanes read 64 consecutive candidates with one
// load, mark the regular run starts (a key that differs from the candidate
// before it; the first candidate, at a lower bound, always starts a run) and
// store them at the query's offset, ranked by a ballot, so every store
// instruction writes one contiguous piece of the output.  A chunk with no
// run start lies inside one long run, which is skipped by galloping.  The
// query is done once its pairs are written.
__device__ __forceinline__ void emit_run_starts(const uint32_t* kv, const uint32_t* vv, uint32_t c,
                                                uint32_t e, uint64_t w, uint64_t z, uint32_t x,
                                                uint32_t v, uint32_t lane, uint32_t* ok,
                                                uint32_t* ov) {
  uint32_t prev = kNoKey;
  for (;;) {
    const bool in = c + lane < e;
    const uint32_t key = x >> 1;
    uint32_t pk = __shfl_up(key, 1, 64);
    if (lane == 0) pk = prev;
    const bool start = in && key != pk;
    const bool keep = start && (x & 1u);
    const uint64_t km = ballot(keep);
    const uint64_t at = w + count_below(km);
    if (keep && at < z) {
      ok[at] = key;
      ov[at] = v;
    }
    w += static_cast<uint64_t>(__popcll(km));
    const uint32_t n = (e - c) < 64u ? (e - c) : 64u;
    prev = __shfl(key, static_cast<int>(n - 1), 64);
    const bool any_start = ballot(start) != 0;
    c += n;
    if (c >= e || w >= z) break;
    if (!any_start) {
      c = skip_run(kv, c - 1, e, prev);
      if (c >= e) break;
    }
    const bool in2 = c + lane < e;
    x = in2 ? kv[c + lane] : 0u;
    v = in2 ? vv[c + lane] : 0u;
  }
}

// The wave's 64 queries are taken kU at a time, their first chunks loaded
// together.  Each query's candidate bounds come from the count pass, or,
// with kSearch, are searched here (wave-wide descents; a separate
// instantiation, so that the usual form keeps its smaller register
// footprint).  A query
// whose pairs would end beyond cap writes nothing (the caller sees
// offsets[q + 1] > cap); writes stay inside [offsets[q], offsets[q + 1])
// even for offsets corrupted by a timed-out scan.
template <bool kTop, int kU, bool kSearch>
__global__ __launch_bounds__(kQueryThreads) void k_range_emit_one(
    QLevels lv, const uint32_t* lo, const uint32_t* hi, uint32_t nq, const uint64_t* offsets,
    const uint32_t* bounds, uint32_t* out_keys, uint32_t* out_vals, uint64_t cap) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t i = blockIdx.x * kQueryThreads + threadIdx.x;
  const uint32_t* kv = lv.v[0].kv;
  const uint32_t* vv = lv.v[0].val;
  const uint32_t len = lv.v[0].len;
  uint32_t p = 0, e = 0;
  uint64_t o = 0, z = 0;
  bool emit = false;
  if (i < nq) {
    const uint64_t a = offsets[i], b = offsets[i + 1];
    if (b > a && b <= offsets[nq] && b <= cap) {
      o = a;
      z = b;
      emit = true;
    }
  }
  if constexpr (!kSearch) {
    if (emit) {
      const uint2 pe = reinterpret_cast<const uint2*>(bounds)[i];
      p = pe.x;
      e = pe.y;
    }
  } else {
    // Wave-wide descents: every lane searches (an empty range if it emits
    // nothing).
    extern __shared__ uint32_t top[];
    if constexpr (kTop) load_tops<kQueryThreads / 64>(lv, top);
    const uint32_t k1 = emit ? lo[i] : 1u, k2 = emit ? hi[i] : 0u;
    uint32_t kq[8];
    octet_lanes(k1, kq);
    p = octet_bound<kTop, false, false>(lv, top, 0, k1, kq, nullptr);
    octet_lanes(k2, kq);
    e = octet_bound<kTop, true, false>(lv, top, 0, k2, kq, nullptr);
    if (!emit || k1 > k2) p = e = 0;
  }
  e = e < len ? e : len;
  p = p < e ? p : e;
  // Every lane stays to the end: the loop below is uniform over the wave.
  for (uint32_t q0 = 0; q0 < 64; q0 += kU) {
    uint32_t qp[kU], qe[kU], x[kU], v[kU];
    uint64_t qo[kU], qz[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int src = static_cast<int>(q0) + u;
      qp[u] = __shfl(p, src, 64);
      qe[u] = __shfl(e, src, 64);
      qo[u] = __shfl(o, src, 64);
      qz[u] = __shfl(z, src, 64);
      const uint32_t at = qp[u] + lane;
      const bool in = at < qe[u];
      x[u] = in ? kv[at] : 0u;
      v[u] = in ? vv[at] : 0u;
    }
#pragma unroll
    for (int u = 0; u < kU; ++u)
      if (qp[u] < qe[u])
        emit_run_starts(kv, vv, qp[u], qe[u], qo[u], qz[u], x[u], v[u], lane, out_keys, out_vals);
  }
}

// ------------------------------------------------------------ scan
constexpr uint64_t kFlagAgg64 = 1ull << 62;
constexpr uint64_t kFlagInc64 = 2ull << 62;
constexpr uint64_t kSumMask64 = (1ull << 62) - 1;

// status[0] is the dynamic tile counter, status[1 + t] tile t's look-back
// word; all cleared beforehand by k_count.
__global__ __launch_bounds__(kThreads) void k_scan(const uint32_t* counts, uint32_t nq,
                                                   uint64_t* offsets, uint64_t* status,
                                                   uint32_t* fault) {
  __shared__ uint64_t s_w[kWaves];
  __shared__ uint32_t s_tile;
  __shared__ uint64_t s_prefix;
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid == 0) s_tile = static_cast<uint32_t>(atomicAdd(reinterpret_cast<unsigned long long*>(status), 1ull));
  __syncthreads();
  const uint32_t tile = s_tile;
  const uint64_t base = static_cast<uint64_t>(tile) * kScanTile + static_cast<uint64_t>(tid) * kScanItems;
  uint32_t v[kScanItems];
  uint64_t tsum = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    v[k] = (base + k < nq) ? counts[base + k] : 0u;
    tsum += v[k];
  }
  const uint64_t winc = wave_incl_scan64(tsum, lane);
  if (lane == 63) s_w[wave] = winc;
  __syncthreads();
  uint64_t wpre = 0, tile_total = 0;
  for (uint32_t w = 0; w < kWaves; ++w) {
    if (w < wave) wpre += s_w[w];
    tile_total += s_w[w];
  }
  const uint64_t texcl = wpre + winc - tsum;

  if (wave == 0) {
    uint64_t excl = 0;
    if (tile == 0) {
      if (lane == 0) st_dev64(&status[1], kFlagInc64 | tile_total);
    } else {
      if (lane == 0) st_dev64(&status[1 + tile], kFlagAgg64 | tile_total);
      int64_t j = static_cast<int64_t>(tile) - 1;
      uint32_t spins = 0;
      for (;;) {
        const int64_t idx = j - static_cast<int64_t>(lane);
        const uint64_t w = idx >= 0 ? ld_dev64(&status[1 + idx]) : kFlagInc64;
        const uint64_t f = w & ~kSumMask64;
        const uint64_t nr = ballot(f == 0), inc = ballot(f == kFlagInc64);
        const uint32_t first_nr = nr ? static_cast<uint32_t>(__builtin_ctzll(nr)) : 64u;
        const uint32_t first_inc = inc ? static_cast<uint32_t>(__builtin_ctzll(inc)) : 64u;
        if (first_inc < first_nr) {
          excl += wave_sum64(lane <= first_inc ? (w & kSumMask64) : 0ull);
          break;
        }
        excl += wave_sum64(lane < first_nr ? (w & kSumMask64) : 0ull);
        j -= first_nr;
        if (first_nr == 0) {
          __builtin_amdgcn_s_sleep(1);
          if (++spins == kSpinLimit) {
            if (lane == 0) atomicOr(fault, kFaultTimeout);
            break;
          }
        }
      }
      if (lane == 0) st_dev64(&status[1 + tile], kFlagInc64 | (excl + tile_total));
    }
    if (lane == 0) s_prefix = excl;
  }
  __syncthreads();
  uint64_t run = s_prefix + texcl;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (base + k < nq) offsets[base + k] = run;
    run += v[k];
  }
  const uint64_t tiles = (static_cast<uint64_t>(nq) + kScanTile - 1) / kScanTile;
  if (tile == tiles - 1 && tid == kThreads - 1) offsets[nq] = s_prefix + tile_total;
}

// ------------------------------------------------------------ order queries
// Successor: the smallest key at the levels' upper bounds of q.  Its newest
// instance is the one of the first level that holds it; nearly always a
// regular element, and the answer.  A tombstone drops the key: every level
// skips its run of it, and the smallest key of the rest is next.  The cursors
// stand in LDS (word l * kQueryThreads + thread), since an array indexed by
// the level takes 148 registers: three waves a SIMD, 439 us for 2^20 queries
// on seven levels; descending again from the dropped key takes 547.
// Few queries: 64 a work-group, the levels' descents dealt to its waves as for
// few lookups; the first wave goes on from the cursors and elements they leave:
// 500 queries on seven levels take 21 us (successor), 45 with every wave
// descending all levels; 60 000 take 45 us, 60.
template <bool kFew>
__global__ __launch_bounds__(kFew ? 64 * kFewWaves : kQueryThreads, 5) void k_successor(
    QLevels lv, const uint32_t* q, uint32_t nq, uint32_t* out_key, uint32_t* out_val,
    uint8_t* out_found) {
  constexpr uint32_t kStride = kFew ? 64 : kQueryThreads;
  extern __shared__ uint32_t top[];
  const uint32_t slot = kFew ? threadIdx.x & 63u : threadIdx.x;
  const int wave = static_cast<int>(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
  const int waves = static_cast<int>(blockDim.x >> 6);
  uint32_t* cur = top + lv.words + slot;
  uint32_t* elem = cur + static_cast<uint32_t>(lv.count) * kStride;  // few queries only
  if constexpr (!kFew) load_tops<kQueryThreads / 64>(lv, top);
  for (uint64_t q0 = static_cast<uint64_t>(blockIdx.x) * kStride; q0 < nq;
       q0 += static_cast<uint64_t>(gridDim.x) * kStride) {
    const uint64_t i = q0 + slot;
    const uint32_t k = i < nq ? q[i] : kMaxKey;
    uint32_t kq[8];
    octet_lanes(k, kq);
    uint32_t best = kNoKey, x = 0u;  // the smallest key and its newest instance
    int level = 0;
    auto take = [&](int l, uint32_t p, uint32_t y) {
      if (p < lv.v[l].len && (y >> 1) < best) {  // ties: the newer level's stays
        best = y >> 1;
        x = y;
        level = l;
      }
    };
    for (int l = kFew ? wave : 0; l < lv.count; l += kFew ? waves : 1) {
      const uint32_t p = octet_bound<!kFew, true, false>(lv, top, l, k, kq, nullptr);
      cur[l * kStride] = p;
      const uint32_t y = p < lv.v[l].len ? lv.v[l].kv[p] : 0u;
      if (kFew) elem[l * kStride] = y;
      else take(l, p, y);
    }
    if constexpr (kFew) {
      __syncthreads();
      if (wave != 0) return;  // one block of queries a work-group
      for (int l = 0; l < lv.count; ++l) take(l, cur[l * kStride], elem[l * kStride]);
    }
    if (k >= kMaxKey) best = kNoKey;
    while (best != kNoKey && (x & 1u) == 0u) {
      const uint32_t gone = best;
      best = kNoKey;
      for (int l = 0; l < lv.count; ++l) {
        const uint32_t* kv = lv.v[l].kv;
        uint32_t p = cur[l * kStride];
        if (p >= lv.v[l].len) continue;
        uint32_t y = kv[p];
        if ((y >> 1) == gone) {
          p = skip_run(kv, p, lv.v[l].len, gone);
          cur[l * kStride] = p;
          if (p >= lv.v[l].len) continue;
          y = kv[p];
        }
        take(l, p, y);
      }
    }
    if (i < nq) {
      const bool f = best != kNoKey;
      out_key[i] = f ? best : 0u;
      out_val[i] = f ? as_global(lv.v[level].val)[cur[level * kStride]] : 0u;
      out_found[i] = f ? 1 : 0;
    }
  }
}

// First element of the run of `key` that kv[c] belongs to: nearly always c itself,
// else a few elements back (a key and its tombstone), so the run is walked back by
// galloping, a long one by O(log) probes.  Searching the whole level instead, which
// one lane in a wave is enough to cause, 60 000 predecessors on three levels with a
// tenth of the keys deleted took 39.8 us, 16.5 so; 2^18 on six of 6 M 116.6 and 65.7.
__device__ __forceinline__ uint32_t run_start(const uint32_t* kv, uint32_t c, uint32_t key) {
  uint32_t hi = c;  // has the key
  if (hi == 0u || (as_global(kv)[hi - 1u] >> 1) != key) return hi;
  --hi;
  uint32_t step = 1;
  while (hi >= step && (as_global(kv)[hi - step] >> 1) == key) {
    hi -= step;
    step <<= 1;
  }
  uint32_t lo = hi >= step ? hi - step + 1u : 0u;  // nothing before it has the key
  while (lo < hi) {
    const uint32_t mid = lo + ((hi - lo) >> 1);
    if ((as_global(kv)[mid] >> 1) == key) hi = mid;
    else lo = mid + 1u;
  }
  return hi;
}

// Predecessor: the mirror walk, the largest key below the levels' lower bounds
// of q; the newest instance is the first element of its run in the first level
// that holds it.
template <bool kFew>
__global__ __launch_bounds__(kFew ? 64 * kFewWaves : kQueryThreads, 5) void k_predecessor(
    QLevels lv, const uint32_t* q, uint32_t nq, uint32_t* out_key, uint32_t* out_val,
    uint8_t* out_found) {
  constexpr uint32_t kStride = kFew ? 64 : kQueryThreads;
  extern __shared__ uint32_t top[];
  const uint32_t slot = kFew ? threadIdx.x & 63u : threadIdx.x;
  const int wave = static_cast<int>(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
  const int waves = static_cast<int>(blockDim.x >> 6);
  uint32_t* cur = top + lv.words + slot;  // the candidate is the element below
  uint32_t* elem = cur + static_cast<uint32_t>(lv.count) * kStride;  // few queries only
  if constexpr (!kFew) load_tops<kQueryThreads / 64>(lv, top);
  for (uint64_t q0 = static_cast<uint64_t>(blockIdx.x) * kStride; q0 < nq;
       q0 += static_cast<uint64_t>(gridDim.x) * kStride) {
    const uint64_t i = q0 + slot;
    const uint32_t k = i < nq ? q[i] : 0u;
    uint32_t kq[8];
    octet_lanes(k, kq);
    uint32_t best = kNoKey;  // the largest key, kNoKey for none
    int level = 0;
    auto take = [&](int l, uint32_t p, uint32_t key) {
      if (p > 0u && (best == kNoKey || key > best)) {  // ties: the newer level's stays
        best = key;
        level = l;
      }
    };
    for (int l = kFew ? wave : 0; l < lv.count; l += kFew ? waves : 1) {
      const uint32_t p = octet_bound<!kFew, false, false>(lv, top, l, k, kq, nullptr);
      cur[l * kStride] = p;
      const uint32_t key = p > 0u ? lv.v[l].kv[p - 1u] >> 1 : 0u;
      if (kFew) elem[l * kStride] = key;
      else take(l, p, key);
    }
    if constexpr (kFew) {
      __syncthreads();
      if (wave != 0) return;  // one block of queries a work-group
      for (int l = 0; l < lv.count; ++l) take(l, cur[l * kStride], elem[l * kStride]);
    }
    uint32_t at = 0u;
    while (best != kNoKey) {
      at = run_start(lv.v[level].kv, cur[level * kStride] - 1u, best);
      if ((as_global(lv.v[level].kv)[at] & 1u) != 0u) break;
      const uint32_t gone = best;
      best = kNoKey;
      for (int l = 0; l < lv.count; ++l) {
        uint32_t p = cur[l * kStride];
        if (p == 0u) continue;
        uint32_t key = lv.v[l].kv[p - 1u] >> 1;
        if (key == gone) {
          p = run_start(lv.v[l].kv, p - 1u, gone);
          cur[l * kStride] = p;
          if (p == 0u) continue;
          key = lv.v[l].kv[p - 1u] >> 1;
        }
        take(l, p, key);
      }
    }
    if (i < nq) {
      const bool f = best != kNoKey;
      out_key[i] = f ? best : 0u;
      out_val[i] = f ? as_global(lv.v[level].val)[at] : 0u;
      out_found[i] = f ? 1 : 0;
    }
  }
}

// ------------------------------------------------------------ cleanup
// Stages 2-5 of the bulk cleanup of sec. IV-D over the merged list (stage 1
// is a chain of ordinary merges).  A tile is kThreads x kCleanItems
// consecutive elements, each thread holding kCleanItems consecutive ones.
constexpr int kCleanItems = 8;
constexpr uint32_t kCleanTile = kThreads * kCleanItems;

// The thread's elements [e0, e0 + kCleanItems) of a list of n (0 past its end).
__device__ __forceinline__ void clean_load(const uint32_t* list, uint32_t n, uint32_t e0,
                                           uint32_t (&x)[kCleanItems]) {
  static_assert(kCleanItems == 8, "two 16-byte loads (the lists are 256-byte aligned)");
  if (e0 < n && n - e0 >= 8u) {  // (e0 + 8 may be 2^32)
    const uint4 a = *reinterpret_cast<const uint4*>(list + e0);
    const uint4 b = *reinterpret_cast<const uint4*>(list + e0 + 4);
    x[0] = a.x, x[1] = a.y, x[2] = a.z, x[3] = a.w;
    x[4] = b.x, x[5] = b.y, x[6] = b.z, x[7] = b.w;
  } else {
#pragma unroll
    for (int j = 0; j < kCleanItems; ++j) x[j] = e0 + j < n ? list[e0 + j] : 0u;
  }
}

// Loads the thread's elements and returns their valid flags: the first element
// of a key run, when regular (stage 2: everything else is stale).
__device__ __forceinline__ uint32_t clean_flags(const uint32_t* kv, uint32_t n, uint32_t e0,
                                                uint32_t (&x)[kCleanItems]) {
  clean_load(kv, n, e0, x);
  uint32_t prev = static_cast<uint32_t>(__shfl_up(static_cast<int>(x[kCleanItems - 1]), 1, 64)) >> 1;
  if (lane_id() == 0) prev = (e0 > 0u && e0 < n) ? (kv[e0 - 1u] >> 1) : kNoKey;
  uint32_t mask = 0u;
#pragma unroll
  for (int j = 0; j < kCleanItems; ++j) {
    if (e0 + j < n && (x[j] & 1u) && (x[j] >> 1) != prev) mask |= 1u << j;
    prev = x[j] >> 1;
  }
  return mask;
}

__global__ __launch_bounds__(kThreads) void k_clean_count(const uint32_t* kv, uint32_t n,
                                                          uint32_t* tile_cnt,
                                                          uint64_t* scan_status,
                                                          uint64_t scan_words) {
  __shared__ uint32_t tmp[kWaves];
  const uint32_t tid = threadIdx.x;
  const uint64_t gi = static_cast<uint64_t>(blockIdx.x) * kThreads + tid;
  for (uint64_t w = gi; w < scan_words; w += static_cast<uint64_t>(gridDim.x) * kThreads)
    scan_status[w] = 0ull;
  const uint32_t e0 = blockIdx.x * kCleanTile + tid * kCleanItems;
  uint32_t x[kCleanItems];
  const uint32_t c = __popc(clean_flags(kv, n, e0, x));
  const uint32_t pre = block_excl_scan(c, tmp);
  if (tid == kThreads - 1) tile_cnt[blockIdx.x] = pre + c;
}

// Position p of the redistributed list -> (level slot, index in the level).
__device__ __forceinline__ int dst_level(const LevelDst& d, uint64_t p, int l) {
  while (l + 1 < d.count && d.start[l + 1] <= p) ++l;
  return l;
}

__device__ __forceinline__ void dst_write(const LevelDst& d, int l, uint64_t p, uint32_t x,
                                          uint32_t v) {
  const uint64_t o = p - d.start[l];
  d.kv[l][o] = x;
  d.val[l][o] = v;
  put_fence(d.fence[l], d.len[l], o, x);
}

// The valid elements of a tile are gathered in LDS and written with consecutive
// lanes on consecutive positions; a tile that ends in the level it starts in
// (nearly every one) writes through uniform pointers.  Bound by memory: counting
// and scattering 63 * 2^20 elements, a tenth stale, take 237 us (5.4 TB/s), 890
// when each thread read and wrote its eight consecutive elements one by one;
// 261 * 2^16 take 66, 280.
__global__ __launch_bounds__(kThreads) void k_clean_scatter(const uint32_t* kv,
                                                            const uint32_t* val, uint32_t n,
                                                            const uint64_t* tile_off,
                                                            LevelDst d) {
  __shared__ uint32_t tmp[kWaves + 1], s_k[kCleanTile], s_v[kCleanTile];
  const uint32_t tid = threadIdx.x;
  const uint32_t e0 = blockIdx.x * kCleanTile + tid * kCleanItems;
  uint32_t x[kCleanItems], v[kCleanItems];
  clean_load(val, n, e0, v);
  const uint32_t mask = clean_flags(kv, n, e0, x);
  uint32_t at = block_excl_scan(__popc(mask), tmp);
  if (tid == kThreads - 1) tmp[kWaves] = at + __popc(mask);
#pragma unroll
  for (int j = 0; j < kCleanItems; ++j) {
    if (mask & (1u << j)) {
      s_k[at] = x[j];
      s_v[at] = v[j];
      ++at;
    }
  }
  __syncthreads();
  const uint32_t m = tmp[kWaves];
  const uint64_t p0 = tile_off[blockIdx.x];
  int l = dst_level(d, p0, 0);
  if (l + 1 >= d.count || p0 + m <= d.start[l + 1]) {
    const uint64_t o0 = p0 - d.start[l], len = d.len[l];
    uint32_t *ok = d.kv[l], *ov = d.val[l], *fence = d.fence[l];
    for (uint32_t i = tid; i < m; i += kThreads) {
      const uint32_t k = s_k[i];
      ok[o0 + i] = k;
      ov[o0 + i] = s_v[i];
      put_fence(fence, len, o0 + i, k);
    }
    return;
  }
  for (uint32_t i = tid; i < m; i += kThreads) {
    l = dst_level(d, p0 + i, l);
    dst_write(d, l, p0 + i, s_k[i], s_v[i]);
  }
}

__global__ __launch_bounds__(kThreads) void k_clean_pad(LevelDst d, uint64_t v, uint64_t total) {
  const uint64_t p = v + static_cast<uint64_t>(blockIdx.x) * kThreads + threadIdx.x;
  if (p >= total) return;
  dst_write(d, dst_level(d, p, 0), p, kPlaceboKv, 0u);
}

// Writes one zero word: clears a range call's total where a memset node on
// the stream is not wanted.
__global__ void k_zero_u64(uint64_t* p) { *p = 0ull; }

inline unsigned grid_for(uint64_t n, uint64_t per) { return static_cast<unsigned>((n + per - 1) / per); }

// lds: bytes of dynamic LDS.
template <typename Kernel, typename... Args>
hipError_t launch_lds(Kernel k, unsigned grid, unsigned block, unsigned lds, hipStream_t s,
                      const KTimer* t, Args... args) {
  if (t != nullptr && (t->start != nullptr || t->stop != nullptr))
    hipExtLaunchKernelGGL(k, dim3(grid), dim3(block), lds, s, t->start, t->stop, 0, args...);
  else
    k<<<grid, block, lds, s>>>(args...);
  return hipGetLastError();
}
template <typename Kernel, typename... Args>
hipError_t launch(Kernel k, unsigned grid, unsigned block, hipStream_t s, const KTimer* t,
                  Args... args) {
  return launch_lds(k, grid, block, 0, s, t, args...);
}

}  // namespace

// ------------------------------------------------------------ fixed scratch
// Range scratch held in the code object (the per-query counts, then the
// scan's look-back words), for callers that cannot allocate.  Every device
// that loads the library holds its own copy until the process ends.  Host
// code must never pass `scratch` itself to a kernel: on the host the name
// stands for a host-side shadow, so kernels get the address that
// hipGetSymbolAddress returns for the current device.
constexpr uint64_t kFixedStatusWords = 1 + (kFixedMaxQueries + kScanTile - 1) / kScanTile;
constexpr uint64_t kFixedWords = kFixedMaxQueries / 2 + kFixedStatusWords;
static __device__ __align__(256) uint64_t scratch[kFixedWords];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_fixed_mu;
void* g_fixed_addr[kMaxDevices] = {};
}  // namespace

hipError_t fixed_scratch(FixedScratch* out) {
  out->counts = nullptr;
  out->status = nullptr;
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_fixed_mu);
  if (g_fixed_addr[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    g_fixed_addr[dev] = p;
  }
  uint64_t* base = static_cast<uint64_t*>(g_fixed_addr[dev]);
  out->counts = reinterpret_cast<uint32_t*>(base);
  out->status = base + kFixedMaxQueries / 2;
  return hipSuccess;
}

hipError_t launch_zero_u64(uint64_t* p, hipStream_t stream) {
  return launch(k_zero_u64, 1, 1, stream, nullptr, p);
}

// ------------------------------------------------------------ launchers
size_t sort_meta_words(uint32_t b) {
  const size_t ns = grid_for(b, kSortTile);
  return static_cast<size_t>(2) * kMaxPasses * kRadix + static_cast<size_t>(kMaxPasses) * ns * kRadix +
         kMaxPasses + 4 + kSortSlots * (ns * (kTopBuckets / 2) + kTopBuckets + 4);
}

SortMeta sort_meta_carve(uint32_t* base, uint32_t b, int parity, int slot) {
  SortMeta m;
  const size_t ns = grid_for(b, kSortTile);
  m.num_sort_tiles = static_cast<uint32_t>(ns);
  m.hist = base;
  m.status = m.hist + static_cast<size_t>(2) * kMaxPasses * kRadix;
  m.tile_ctr = m.status + static_cast<size_t>(kMaxPasses) * ns * kRadix;
  m.err = m.tile_ctr + kMaxPasses;
  // Per slot: the group starts, then the bucket-size record (both 16-byte
  // aligned), then the padding element.
  uint32_t* slot_base =
      m.err + 4 + static_cast<size_t>(slot) * (ns * (kTopBuckets / 2) + kTopBuckets + 4);
  m.tile_cnt = slot_base;
  m.bucket_n = slot_base + ns * (kTopBuckets / 2);
  m.pad = m.bucket_n + kTopBuckets;
  m.parity = parity;
  return m;
}

int sort_kernel_count(const SortArgs& a) {
  if (a.path == kSortMsd) return 2;
  return 1 + a.passes;
}

// The number of 8-bit passes that sort a top-digit bucket: the key-variable
// bits below the top digit.
static int bucket_passes(const SortArgs& a) {
  return (sort_top_shift(a) - a.lo_bit + kRadixBits - 1) / kRadixBits;
}

// Tiles of a batch's scatter: its elements', without the padding's.
static uint32_t scatter_tiles(const SortArgs& a) { return grid_for(a.src.n, kSortTile); }

static ScatterArgs scatter_args(const SortArgs& a) {
  return ScatterArgs{a.src,      a.tmp_kv[0], a.tmp_val[0], a.meta.tile_cnt,  a.meta.bucket_n,
                     a.meta.pad, a.skew_out,  a.progress,   a.seq, sort_top_shift(a)};
}

hipError_t launch_scatter(const SortArgs& a, hipStream_t stream, const KTimer* t) {
  return launch(k_msd_scatter, scatter_tiles(a), kThreads, stream, t, scatter_args(a));
}

// The largest entry of a slot's bucket-size record into *out (one work-group).
__global__ __launch_bounds__(kThreads) void k_rec_max(const uint32_t* rec, uint32_t* out) {
  __shared__ uint32_t s_max[kWaves];
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint4 r = reinterpret_cast<const uint4*>(rec)[tid];
  uint32_t x = max(max(r.x, r.y), max(r.z, r.w));
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = max(x, static_cast<uint32_t>(__shfl_xor(x, o, 64)));
  if (lane == 0) s_max[wave] = x;
  __syncthreads();
  if (tid == 0) {
    uint32_t mx = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) mx = max(mx, s_max[w]);
    *out = mx;
  }
}

hipError_t launch_rec_max(const uint32_t* rec, uint32_t* out, hipStream_t stream) {
  return launch(k_rec_max, 1, kThreads, stream, nullptr, rec, out);
}

// Arguments without a group (group == 0) sort the one batch of their slot,
// scattered from element 0 of tmp_kv[0].
SortArgs grouped(SortArgs a) {
  if (a.group == 0) {
    a.group = 1;
    a.grp_cnt[0] = a.meta.tile_cnt;
    a.grp_n[0] = a.meta.bucket_n;
    a.grp_off[0] = 0;
    a.grp_real[0] = a.src.n;
    a.grp_pad[0] = a.meta.pad;
    a.pads = a.src.b - a.src.n;
    a.pad_shift = sort_top_shift(a);
  }
  return a;
}


hipError_t launch_buckets(const SortArgs& in, hipStream_t stream, const KTimer* t) {
  const SortArgs a = grouped(in);
  return launch(a.pads != 0 ? k_local_sort<true> : k_local_sort<false>, kTopBuckets, kThreads,
                stream, t, a, a.lo_bit, bucket_passes(a));
}

hipError_t launch_sort_step(const SortArgs& in, const SortArgs& sc, hipStream_t stream,
                            const KTimer* t) {
  const SortArgs bk = grouped(in);
  return launch(bk.pads != 0 ? k_sort_step<true> : k_sort_step<false>,
                scatter_tiles(sc) + kTopBuckets, kThreads, stream, t, bk, bk.lo_bit,
                bucket_passes(bk), scatter_args(sc));
}

hipError_t launch_sort(const SortArgs& a, hipStream_t stream, const KTimer* timers,
                       int* launched) {
  const uint32_t tiles = a.meta.num_sort_tiles;
  *launched = 0;
  if (a.path == kSortMsd && tiles <= static_cast<uint32_t>(kMsdMaxTiles)) {
    // Top digit: the highest 8 bits a key variable of this handle can have.
    hipError_t e = launch_scatter(a, stream, timers ? &timers[0] : nullptr);
    if (e != hipSuccess) return e;
    *launched = 1;
    e = launch_buckets(a, stream, timers ? &timers[1] : nullptr);
    if (e == hipSuccess) *launched = 2;
    return e;
  }
  if (tiles > static_cast<uint32_t>(kMsdMaxTiles)) {
    // Counts and totals live in the look-back words' region, which this path
    // does not use otherwise: at least 4 x 257 x 256 words.
    static_assert(static_cast<uint64_t>(kMaxPasses) * (kMsdMaxTiles + 1) * kRadix >=
                      static_cast<uint64_t>(kRadix) * kLsdMaxGroups + kRadix,
                  "digit counts fit the look-back region");
    const LsdGrid g = lsd_grid(a.src.b);
    uint32_t* counts = a.meta.status;
    uint32_t* totals = counts + static_cast<size_t>(kRadix) * g.groups;
    for (int p = 0; p < a.passes; ++p) {
      const LsdSrc in = p == 0 ? LsdSrc{nullptr, nullptr}
                               : LsdSrc{a.tmp_kv[(p - 1) & 1], a.tmp_val[(p - 1) & 1]};
      const bool last = p == a.passes - 1;
      const int shift = a.lo_bit + kRadixBits * p;
      // A pass is timed from its count to its scatter; the first kernel of
      // all has the histogram's timer to itself.
      const KTimer begin{timers != nullptr && p > 0 ? timers[1 + p].start : nullptr, nullptr};
      const KTimer end{timers != nullptr && p == 0 ? timers[1].start : nullptr,
                       timers != nullptr ? timers[1 + p].stop : nullptr};
      hipError_t e = launch(k_lsd_up, g.groups, kLsdThreads, stream,
                            timers != nullptr && p == 0 ? &timers[0] : &begin, a, in, shift,
                            g.tiles_per_group, counts);
      if (e != hipSuccess) return e;
      e = launch(k_lsd_scan, kRadix, kThreads, stream, nullptr, counts, g.groups, totals);
      if (e != hipSuccess) return e;
      e = launch(p == 0 ? k_lsd_down<true> : k_lsd_down<false>, g.groups, kLsdThreads, stream, &end, a, in, shift, g.tiles_per_group,
                 counts, totals, last ? a.out_kv : a.tmp_kv[p & 1],
                 last ? a.out_val : a.tmp_val[p & 1], last ? a.out_fence : nullptr);
      if (e != hipSuccess) return e;
    }
    *launched = 1 + a.passes;
    return hipSuccess;
  }
  hipError_t e = launch(k_sort_hist, tiles, kThreads, stream, timers ? &timers[0] : nullptr, a);
  if (e != hipSuccess) return e;
  *launched = 1;
  for (int p = 0; p < a.passes; ++p) {
    e = launch(k_sort_pass, tiles, kThreads, stream, timers ? &timers[1 + p] : nullptr, a, p);
    if (e != hipSuccess) return e;
    *launched += 1;
  }
  return hipSuccess;
}

template <int kItems>
hipError_t launch_merge_items(MergeArgs m, uint32_t max_blocks, hipStream_t stream,
                              const KTimer* t) {
  const uint64_t total = static_cast<uint64_t>(m.na) + m.nb;
  const uint64_t tile = static_cast<uint64_t>(kThreads) * kItems;
  const uint64_t tiles = (total + tile - 1) / tile;
  if (m.digit_mode) {
    // Work-groups over the digits: at most one per digit, and no more than
    // output tiles (a small merge takes a few work-groups of many digits).
    const uint64_t groups = tiles < kTopBuckets ? (tiles > 0 ? tiles : 1) : kTopBuckets;
    m.per_wg = static_cast<uint32_t>((kTopBuckets + groups - 1) / groups);
    return launch(k_merge<kItems>, grid_for(kTopBuckets, m.per_wg), kThreads, stream, t, m);
  }
  m.per_wg = static_cast<uint32_t>((tiles + max_blocks - 1) / max_blocks);
  return launch(k_merge<kItems>, grid_for(tiles, m.per_wg), kThreads, stream, t, m);
}

hipError_t launch_merge(const uint32_t* a_kv, const uint32_t* a_val, uint32_t na,
                        const uint32_t* b_kv, const uint32_t* b_val, uint32_t nb,
                        uint32_t* out_kv, uint32_t* out_val, uint32_t* out_fence, int variant,
                        hipStream_t stream, const KTimer* t, const MergeIndex* idx) {
  const uint64_t total = static_cast<uint64_t>(na) + nb;
  if (total == 0) return hipSuccess;
  if (variant < 0 || variant >= kMergeVariants) variant = kDefaultMergeVariant;
  MergeArgs m{};
  m.a_kv = a_kv;
  m.a_val = a_val;
  m.b_kv = b_kv;
  m.b_val = b_val;
  m.na = na;
  m.nb = nb;
  m.out_kv = out_kv;
  m.out_val = out_val;
  m.out_fence = out_fence;
  if (idx != nullptr && idx->a_dig != nullptr && idx->b_dig != nullptr) {
    m.a_dig = idx->a_dig;
    m.b_dig = idx->b_dig;
    m.out_dig = idx->out_dig;
    m.digit_mode = idx->by_digit;
  }
  const uint32_t blocks = static_cast<uint32_t>(kMergeBlocksOf[variant / 3]);
  switch (kMergeItemsOf[variant % 3]) {
    case 4: return launch_merge_items<4>(m, blocks, stream, t);
    case 16: return launch_merge_items<16>(m, blocks, stream, t);
    default: return launch_merge_items<8>(m, blocks, stream, t);
  }
}

hipError_t launch_stage(const uint32_t* keys, const uint32_t* vals, const uint8_t* is_delete,
                        int all_delete, uint32_t n, uint32_t* stage_kv, uint32_t* stage_val,
                        uint32_t at, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  return launch(k_stage, grid_for(n, kThreads), kThreads, stream, nullptr, keys, vals, is_delete,
                all_delete, n, stage_kv, stage_val, at);
}

hipError_t launch_check_keys(const uint32_t* keys, uint32_t n, uint32_t limit_bits, int encoded,
                             uint32_t* err, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  return launch(k_check_keys, grid_for(n, kThreads), kThreads, stream, nullptr, keys, n,
                limit_bits, encoded, err);
}

hipError_t launch_fill_runs(uint32_t* a_kv, uint32_t* a_val, uint32_t* b_kv, uint32_t* b_val,
                            uint32_t n, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  return launch(k_fill_runs, grid_for(n, kThreads), kThreads, stream, nullptr, a_kv, a_val, b_kv,
                b_val, n);
}

// Levels with their tops, and the grid of a query kernel that strides over the
// queries.  Up to kFewQueries the work-groups run side by side: a query's
// latency bounds the launch, so several levels are dealt to the waves of a
// work-group (k_lookup_few and the like) and the tops, whose loading would be
// part of every query's latency, are not used.  The two ways cross between
// 2^17 and 2^18 queries: lookups on ten levels take 60 us dealt and 69 with
// tops at 2^17, 111 and 96 at 2^18; counts 80 and 118, 143 and 163 (where lanes
// count alone, on small dictionaries, the lines are closer: one key on three levels
// of 0.7 M 28 and 20 at 2^17, but 16 keys 44 and 59).  Order
// queries, whose first wave works on alone, cross at half of that: successors
// on seven levels 45 and 60 at 2^16, 73 and 71 at 2^17.  Above, the grid is as large as keeps the
// loading of the tops small beside the queries (with one level 2^22 lookups
// take 212 us in 5120 work-groups, 222 in 1280).  Where nothing is dealt (one
// level counted, emission that searches) tops pay from half of kFewQueries on:
// 2^17 counts on one level take 21.6 us with them, 23.1 without.
constexpr uint32_t kFewQueries = 1u << 17;
static QLevels query_levels_for(const LevelSet& lv, uint32_t nq) {
  return query_levels(lv, nq <= kFewQueries / 2 ? 0u : kTopWords);
}
static unsigned query_grid(const QLevels& q, uint64_t nq) {
  const uint64_t g = (nq + kQueryThreads - 1) / kQueryThreads;
  const uint64_t most = 5u * 256u * (8192u / (q.words > 2048u ? q.words : 2048u));
  return static_cast<unsigned>(g < most ? g : most);
}
// Queries per octet of the several-level emission: eight, one after another, when
// that leaves 2048 waves or more (8 on each of 256 CUs), else fewer, down to one:
// the emission of 26 000 ranges on three levels set the line there.
static uint32_t queries_per_octet(uint32_t nq) {
  uint32_t per = 8;
  while (per > 1 && nq / (8u * per) < 2048u) per /= 2;
  return per;
}
// When a lane walks its query alone: whether counts may, with at most `far`
// candidates in the largest level, and up to how many pairs every query of a wave
// may have in the emission (0: never).  An octet's load instruction reads eight
// lines, a lane walk's 64, so the rule depends on where the levels lie (4 MB of L2
// hold the keys of 2^20 elements).  Octets alone and with lane walks, us: 2^20
// counts of one key on three levels of 0.7 M elements 156 and 81, of four keys 163
// and 99, of 16 (octets both) 242 and 244; of one key on eight levels of 1 M 274
// and 190, of eight 298 and 274; the ranges of these counts 221 and 139, 340 and
// 251, 551 and 552, 477 and 273, 571 and 569.  On larger levels waves of both
// kinds together cost more than either kind alone (2^18 counts of two keys on four
// levels of 48 M 70 and 77), so counts stay with the octets there; the emission
// knows its pairs and keeps to eight (2^20 ranges of one key on three levels of
// 45 M 380 and 281), up to six levels.
struct NarrowRule {
  bool count, runs;
  uint32_t far, pairs;
};
static NarrowRule narrow_rule(const LevelSet& lv) {
  uint64_t n = 0;
  for (int l = 0; l < lv.count; ++l) n += lv.len[l];
  if (lv.count > kNarrowLevels) return {false, false, 0, 0};
  return n <= (1u << 21) ? NarrowRule{true, false, 11, 12}
                         : NarrowRule{false, true, 0, lv.count <= 6 ? 8u : 0u};
}
// LDS words of the several-level walk of one work-group.
static unsigned walk_lds_words(const QLevels& q, bool emit) {
  return q.count <= 1 ? 0u : kQueryWaves * walk_words(static_cast<uint32_t>(q.count), emit);
}

hipError_t launch_lookup(const LevelSet& lv, const uint32_t* q, uint32_t nq, uint32_t* out_val,
                         uint8_t* out_found, hipStream_t stream, const KTimer* t) {
  if (nq == 0) return hipSuccess;
  if (nq <= kFewQueries)
    return launch(k_lookup_few, grid_for(nq, 64), 64 * few_waves(lv.count), stream, t,
                  query_levels(lv, 0), q, nq, out_val, out_found);
  const QLevels ql = query_levels(lv, kTopWords);
  return launch_lds(k_lookup, query_grid(ql, nq), kQueryThreads, ql.words * 4u, stream, t, ql, q,
                    nq, out_val, out_found);
}

hipError_t launch_count(const LevelSet& lv, const uint32_t* lo, const uint32_t* hi, uint32_t nq,
                        uint32_t* counts, uint64_t* scan_status, size_t scan_words,
                        uint32_t* bounds, hipStream_t stream, const KTimer* t) {
  if (nq == 0) return hipSuccess;
  if (lv.count > 1 && nq <= kFewQueries) {
    const uint32_t L = static_cast<uint32_t>(lv.count);
    return launch_lds(k_count_few, grid_for(nq, 64), 64 * kFewWaves,
                      (64u * L + 8u * kFewWaves * walk_list(L)) * 4u, stream, t,
                      query_levels(lv, 0), lo, hi, nq, counts, scan_status,
                      static_cast<uint64_t>(scan_words), bounds);
  }
  const QLevels ql = query_levels_for(lv, nq);
  const bool top = ql.words != 0;
  const NarrowRule nr = narrow_rule(lv);
  auto k = lv.count <= 1   ? (top ? k_count<true, false, 0> : k_count<false, false, 0>)
           : !nr.count     ? k_count<true, true, 0>
           : lv.count <= 3 ? k_count<true, true, 3>
           : lv.count <= 6 ? k_count<true, true, 6>
                           : k_count<true, true, kNarrowLevels>;
  const unsigned lds = (ql.words + walk_lds_words(ql, false)) * 4u;
  return launch_lds(k, query_grid(ql, nq), kQueryThreads, lds, stream, t, ql, lo, hi, nq,
                    nr.far, counts, scan_status, static_cast<uint64_t>(scan_words), bounds);
}

size_t scan_status_words(uint32_t nq) { return 1 + grid_for(nq, kScanTile); }

hipError_t launch_scan(const uint32_t* counts, uint32_t nq, uint64_t* offsets,
                       uint64_t* scan_status, uint32_t* fault, hipStream_t stream,
                       const KTimer* t) {
  if (nq == 0) return hipSuccess;
  return launch(k_scan, grid_for(nq, kScanTile), kThreads, stream, t, counts, nq, offsets,
                scan_status, fault);
}

template <typename Kernel>
static hipError_t launch_order(Kernel many, Kernel few, const LevelSet& lv, const uint32_t* q,
                               uint32_t nq, uint32_t* out_key, uint32_t* out_val,
                               uint8_t* out_found, hipStream_t stream, const KTimer* t) {
  if (nq == 0) return hipSuccess;
  const unsigned L = static_cast<unsigned>(lv.count);
  if (nq <= kFewQueries / 2)
    return launch_lds(few, grid_for(nq, 64), 64 * few_waves(lv.count), 2u * 64u * L * 4u, stream,
                      t, query_levels(lv, 0), q, nq, out_key, out_val, out_found);
  const QLevels ql = query_levels(lv, kTopWords);
  return launch_lds(many, query_grid(ql, nq), kQueryThreads, (ql.words + L * kQueryThreads) * 4u,
                    stream, t, ql, q, nq, out_key, out_val, out_found);
}

hipError_t launch_successor(const LevelSet& lv, const uint32_t* q, uint32_t nq, uint32_t* out_key,
                            uint32_t* out_val, uint8_t* out_found, hipStream_t stream,
                            const KTimer* t) {
  return launch_order(k_successor<false>, k_successor<true>, lv, q, nq, out_key, out_val, out_found,
                      stream, t);
}

hipError_t launch_predecessor(const LevelSet& lv, const uint32_t* q, uint32_t nq,
                              uint32_t* out_key, uint32_t* out_val, uint8_t* out_found,
                              hipStream_t stream, const KTimer* t) {
  return launch_order(k_predecessor<false>, k_predecessor<true>, lv, q, nq, out_key, out_val,
                      out_found, stream, t);
}

uint32_t clean_tiles(uint32_t n) { return grid_for(n, kCleanTile); }

hipError_t launch_clean_count(const uint32_t* kv, uint32_t n, uint32_t* tile_cnt,
                              uint64_t* scan_status, size_t scan_words, hipStream_t stream,
                              const KTimer* t) {
  if (n == 0) return hipSuccess;
  return launch(k_clean_count, clean_tiles(n), kThreads, stream, t, kv, n, tile_cnt, scan_status,
                static_cast<uint64_t>(scan_words));
}

hipError_t launch_clean_scatter(const uint32_t* kv, const uint32_t* val, uint32_t n,
                                const uint64_t* tile_off, const LevelDst& d, hipStream_t stream,
                                const KTimer* t) {
  if (n == 0 || d.count == 0) return hipSuccess;
  return launch(k_clean_scatter, clean_tiles(n), kThreads, stream, t, kv, val, n, tile_off, d);
}

hipError_t launch_clean_pad(const LevelDst& d, uint64_t v, uint64_t total, hipStream_t stream,
                            const KTimer* t) {
  if (total <= v || d.count == 0) return hipSuccess;
  return launch(k_clean_pad, grid_for(total - v, kThreads), kThreads, stream, t, d, v, total);
}

hipError_t launch_range_emit(const LevelSet& lv, const uint32_t* lo, const uint32_t* hi,
                             uint32_t nq, const uint64_t* offsets, const uint32_t* bounds,
                             uint32_t* out_keys, uint32_t* out_vals, uint64_t cap,
                             hipStream_t stream, const KTimer* t) {
  if (nq == 0) return hipSuccess;
  // Emission from stored bounds and emission that searches (no scratch) are
  // separate instantiations, so that the first keeps a smaller register
  // footprint and no LDS for the tops.
  const QLevels ql = bounds != nullptr ? query_levels(lv, 0) : query_levels_for(lv, nq);
  const bool top = ql.words != 0;
  const unsigned grid = grid_for(nq, kQueryThreads);
  if (lv.count <= 1)
    return launch_lds(bounds != nullptr ? k_range_emit_one<false, 4, false>
                      : top             ? k_range_emit_one<true, 4, true>
                                        : k_range_emit_one<false, 4, true>,
                      grid, kQueryThreads, ql.words * 4u, stream, t, ql, lo, hi, nq, offsets,
                      bounds, out_keys, out_vals, cap);
  const NarrowRule nr = narrow_rule(lv);
  auto k = bounds == nullptr ? (top ? k_range_emit<true, true, 0, false>
                                    : k_range_emit<false, true, 0, false>)
           : lv.count <= 3   ? (nr.runs ? k_range_emit<false, false, 3, true>
                                        : k_range_emit<false, false, 3, false>)
           : lv.count <= 6   ? (nr.runs ? k_range_emit<false, false, 6, true>
                                        : k_range_emit<false, false, 6, false>)
                             : k_range_emit<false, false, kNarrowLevels, false>;
  const unsigned lds = (ql.words + walk_lds_words(ql, true)) * 4u;
  const uint32_t per = queries_per_octet(nq);
  return launch_lds(k, grid_for(nq, kQueryThreads / 8 * per), kQueryThreads, lds, stream, t, ql,
                    lo, hi, nq, per, nr.pairs, offsets, bounds, out_keys, out_vals, cap);
}

}  // namespace lsm
