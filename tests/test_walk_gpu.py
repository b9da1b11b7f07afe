"""Searches from the LDS tops and the several-level range walk at the sizes where
they can go wrong: levels whose tree parts end on and beside a block of 64 and
the largest part (2048 entries), chunks of 8 and 16 candidates a level, runs of
one key longer than a chunk, tombstones over several levels, keys at both ends
of the key space, and every number of queries an octet takes (1, 2, 4, 8).
Answers against the map oracle.  Integer results, tolerance 0."""
import numpy as np
import pytest
import torch

from _gpu import Trio, dev, host, note

pytestmark = pytest.mark.gpu


def check(t, q, lo, hi):
    q, lo, hi = (np.asarray(x, np.uint64).astype(np.uint32) for x in (q, lo, hi))
    t.check_queries(q, lo, hi)
    t.check_order(q)


def batch(rng, n, domain):
    return (rng.integers(0, domain, n, dtype=np.uint64).astype(np.uint32),
            rng.integers(0, 2**32, n, dtype=np.uint64).astype(np.uint32))


@pytest.mark.parametrize("b,R,domain", [
    (1, 31, 40), (7, 22, 60), (31, 13, 500), (64 * 32, 7, 1 << 31), (64 * 32 + 1, 7, 1 << 14),
    (2048 * 32, 3, 1 << 31), (2048 * 32 + 32, 3, 1 << 20), (65 * 32 * 32, 2, 1 << 31)])
def test_tree_sizes(b, R, domain):
    note("tree sizes b=%d R=%d" % (b, R))
    rng = np.random.default_rng(b)
    t = Trio(b)
    for i in range(R):
        k, v = batch(rng, b, domain)
        if i % 4 == 3:
            t.delete(k)
        else:
            t.insert(k, v)
    q = np.r_[rng.integers(0, domain, 400), 0, 1, domain - 1, 2**31 - 2, 2**31 - 1, 2**31, 2**32 - 1]
    a = rng.integers(0, domain, 300)
    w = max(1, 30 * domain // (b * R))
    check(t, q, np.r_[a, 0, 0, domain - 1, 2**31 - 1, 5], np.r_[a + w, 0, domain // 50, 2**32 - 1, 2**31 - 1, 4])
    t.g.close()


@pytest.mark.parametrize("nq", [1, 100, 40000, 70000, 140000])
def test_queries_per_octet(nq):
    """1, 2, 4 and 8 queries an octet, and both sides of the number of queries up
    to which the levels are dealt to the waves, against numpy on the live pairs."""
    note("queries per octet nq=%d" % nq)
    rng = np.random.default_rng(nq)
    b = 3000
    t = Trio(b)
    for i in range(13):
        k, v = batch(rng, b, 1 << 16)
        t.delete(k) if i in (5, 9) else t.insert(k, v)
    live = np.nonzero(t.m.lookup(np.arange(1 << 16, dtype=np.uint32))[1])[0].astype(np.int64)
    lo = rng.integers(0, 1 << 16, nq)
    hi = lo + rng.integers(0, 200, nq)
    a, e = np.searchsorted(live, lo), np.searchsorted(live, hi, side="right")
    got = host(t.g.count(dev(lo), dev(hi)))
    assert np.array_equal(got, e - a)
    off, keys, vals = t.g.range(dev(lo), dev(hi), cap=int((e - a).sum()))
    torch.cuda.synchronize()
    assert np.array_equal(host(off).astype(np.int64), np.r_[0, np.cumsum(e - a)])
    want = np.concatenate([live[x:y] for x, y in zip(a, e)] + [live[:0]])
    assert np.array_equal(host(keys), want)
    assert np.array_equal(host(vals), t.m.lookup(want.astype(np.uint32))[0])
    check(t, lo, lo[:100], hi[:100])
    t.g.close()


@pytest.mark.parametrize("run", [7, 8, 9, 15, 16, 17, 200])
def test_runs_across_chunks(run):
    """Runs of one key of `run` elements in every level, between single keys,
    some of them deleted last; ranges that start and end inside, at and beside
    a run."""
    note("runs of %d" % run)
    rng = np.random.default_rng(run)
    b = 2 * run + 41
    t = Trio(b)
    for i in range(15):
        k = np.r_[np.full(run, 1000), np.full(run, 1003), rng.integers(900, 1100, 41)].astype(np.uint32)
        rng.shuffle(k)
        v = rng.integers(0, 2**32, b, dtype=np.uint64).astype(np.uint32)
        if i % 5 == 4:
            t.delete(k[: run + 5])
        else:
            t.insert(k, v)
    lo = np.repeat(np.arange(895, 1010), 4)
    hi = lo + np.tile([0, 1, 4, 150], 115)
    check(t, np.arange(890, 1110), lo, hi)
    t.g.close()


@pytest.mark.parametrize("R", [2, 3, 7, 21, 63, 127])
def test_narrow_ranges(R):
    """Ranges of few pairs, many queries: widths around the number of pairs up to
    which a lane walks its own query, blocks of more deleted keys than it passes
    over, up to seven levels (six are walked so), against numpy on the live pairs."""
    note("narrow ranges R=%d" % R)
    rng = np.random.default_rng(R)
    b, top = 400, 6000
    t = Trio(b)
    for i in range(R):
        if i % 3 == 2:
            t.delete((int(rng.integers(0, top - b)) + np.arange(b if i % 2 else 30)).astype(np.uint32))
        else:
            t.insert(*batch(rng, b, top))
    live = np.nonzero(t.m.lookup(np.arange(top, dtype=np.uint32))[1])[0].astype(np.int64)
    nq = 140001
    lo = rng.integers(0, top, nq)
    lo[nq // 2:] = np.sort(lo[nq // 2:])
    density = max(1, len(live)) / top
    hi = lo + rng.integers(0, int(9 / density) + 2, nq) * (rng.random(nq) < 0.7)
    a, e = np.searchsorted(live, lo), np.searchsorted(live, hi, side="right")
    off, keys, vals = t.g.range(dev(lo), dev(hi), cap=int((e - a).sum()))
    torch.cuda.synchronize()
    assert np.array_equal(host(off).astype(np.int64), np.r_[0, np.cumsum(e - a)])
    want = np.concatenate([live[x:y] for x, y in zip(a, e)] + [live[:0]])
    assert np.array_equal(host(keys), want)
    assert np.array_equal(host(vals), t.m.lookup(want.astype(np.uint32))[0])
    t.g.close()
