"""Padded batches in the top-digit sort, whose copies are written by the bucket
sort instead of being sorted, and the part-by-part merge of buckets larger
than LDS: levels byte for byte against the cascade oracle, with batches filled
to the edges of a tile, paddings of a group in one bucket and in different
ones, buckets sorted by rank, by LDS passes and by streaming, every fused
depth, deletions, mixed and staged batches.  Integer results, tolerance 0."""
import numpy as np
import pytest

from paper_1707_05354_amd.lsm import LSM
from _gpu import Trio, dev, dev_u8, note

pytestmark = pytest.mark.gpu


def values(rng, n):
    return rng.integers(0, 2**32, n, dtype=np.uint64).astype(np.uint32)


@pytest.mark.parametrize("group", [1, 2, 4])
@pytest.mark.parametrize("b,domain,fusion", [
    (2, 5, -1), (2049, 1 << 31, -1), (4097, 1 << 31, -1), (4097, 1 << 31, 2), (6000, 900, -1),
    (6000, 1 << 22, 0), (3000, 1 << 21, 8), (40000, 1 << 31, -1)])
def test_padded_batches(b, domain, fusion, group):
    """Domains below 2^21 put every key into one top-digit bucket: paddings of
    a group meet there, and the bucket is larger than LDS from b = 3000 on."""
    note("padded b=%d domain=%d fusion=%d group=%d" % (b, domain, fusion, group))
    rng = np.random.default_rng(b + domain + group)
    t = Trio(b)
    t.g.set_sort_path(LSM.SORT_TOP_DIGIT)
    t.g.set_fusion(fusion)
    t.g.set_grouping(group)
    fills = [1, b, 2047, 2048, 2049, b - 1, b // 2, 1, b, b - 700, 3]
    for i in range(19):
        n = max(1, min(b, fills[i % len(fills)]))
        k = rng.integers(0, domain, n, dtype=np.uint64).astype(np.uint32)
        if i % 3 == 0:
            k[-1] = domain // 2  # the same padding key again and again
        if i % 7 == 5:
            t.delete(k)
        elif i % 7 == 6:
            t.mixed(k, values(rng, n), (rng.random(n) < 0.5).astype(np.uint8))
        else:
            t.insert(k, values(rng, n))
        if i in (3, 10):
            t.check_levels()
    t.check_levels()
    q = rng.integers(0, domain, 300, dtype=np.uint64).astype(np.uint32)
    t.check_queries(np.r_[q, np.uint32(domain // 2)], q[:60], (q[:60].astype(np.uint64) + domain // 300 + 1).astype(np.uint32))
    assert t.g.stats().sorts_digit_passes == 0
    t.g.close()


@pytest.mark.parametrize("b,n", [(5000, 1), (5000, 4999), (30000, 12000)])
def test_flushed_tails(b, n):
    """The coalescer's flushed tail is a padded (staged) batch."""
    note("flushed tails b=%d n=%d" % (b, n))
    rng = np.random.default_rng(b + n)
    t = Trio(b)
    for _ in range(9):
        k = rng.integers(0, 1 << 31, n, dtype=np.uint64).astype(np.uint32)
        v, d = values(rng, n), (rng.random(n) < 0.3).astype(np.uint8)
        t.g.submit_mixed(dev(k), dev(v), dev_u8(d))
        t.g.flush()
        t.c.insert_ordered(k, np.where(d, 0, v).astype(np.uint32), (1 - d).astype(np.uint8))
        cut = np.flatnonzero(np.diff(d.astype(np.int8))) + 1
        for a, e in zip(np.r_[0, cut], np.r_[cut, n]):
            t.m.delete(k[a:e]) if d[a] else t.m.insert(k[a:e], v[a:e])
        t.check_levels()
    q = rng.integers(0, 1 << 31, 300, dtype=np.uint64).astype(np.uint32)
    t.check_queries(np.r_[q, k[-20:]], q[:50], q[:50] + np.uint32(1 << 18))
    t.g.close()


@pytest.mark.parametrize("hot", [1, 2, 5])
def test_hot_keys_in_a_large_bucket(hot):
    """Buckets larger than LDS whose levels hold long runs of `hot` keys, all
    levels fused: the merge copies runs and merges what lies between."""
    b = 7000
    note("hot keys in a bucket: %d" % hot)
    rng = np.random.default_rng(hot)
    t = Trio(b)
    t.g.set_sort_path(LSM.SORT_TOP_DIGIT)
    t.g.set_fusion(8)
    keys = rng.integers(1 << 20, 1 << 21, hot).astype(np.uint32)
    for i in range(17):
        k = rng.integers(0, 1 << 22, b, dtype=np.uint64).astype(np.uint32)
        pick = rng.random(b) < 0.7
        k[pick] = keys[rng.integers(0, hot, pick.sum())]
        t.delete(k) if i % 6 == 4 else t.insert(k, values(rng, b))
    t.check_levels()
    t.g.close()


@pytest.mark.parametrize("kind,paths", [("hot", "TTTTTT"), ("cluster", "TDDDDD"), ("spread", "TTTTTT")])
def test_path_of_large_buckets(kind, paths):
    """A bucket that outgrows LDS because of one key stays with the top-digit
    sort (T); one of many keys goes to digit passes (D)."""
    b = 1 << 15
    note("path of large buckets: %s" % kind)
    rng = np.random.default_rng(7)
    t = Trio(b)
    got = ""
    for i in range(6):
        k = rng.integers(0, 1 << 31, b, dtype=np.uint64).astype(np.uint32)
        if kind == "hot":
            k[rng.random(b) < 0.2] = 123456
        elif kind == "cluster":
            near = rng.random(b) < 0.2
            k[near] = rng.integers(0, 1 << 20, near.sum())
        before = t.g.stats().sorts_digit_passes
        t.insert(k, values(rng, b))
        t.check_levels()  # synchronises, so the next choice sees this sort
        got += "D" if t.g.stats().sorts_digit_passes > before else "T"
    assert got == paths
    t.g.close()
