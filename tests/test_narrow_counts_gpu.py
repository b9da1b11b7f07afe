"""Many counts and ranges of few candidates: a lane walks its own query where every
query of its wave is narrow, on each number of levels that has its own kernel (2
and 3, 4 to 6, 7 to 10, more) and on both sides of the dictionary size up to
which counts are walked so.  Widths around the limits (11 candidates in the
largest level, 8 and 12 pairs), runs of one key longer than a walk's steps, blocks
of deleted keys and ranges up to the largest key, against numpy on the live
pairs.  Integer results, tolerance 0."""
import numpy as np
import pytest
import torch

from paper_1707_05354_amd.lsm import LSM
from _gpu import dev, host, note

pytestmark = pytest.mark.gpu

TOP = 2**31 - 1


@pytest.mark.parametrize("b,R", [
    (300, 3), (300, 7), (300, 5), (300, 15), (300, 31), (300, 63), (300, 127), (50, 255), (50, 511), (20, 1023),
    (10, 2047), (700000, 3), (180000, 15), (90000, 31), (20000, 127), (2200, 1023)])
def test_narrow_counts_and_ranges(b, R):
    note("narrow counts b=%d R=%d" % (b, R))
    rng = np.random.default_rng(b + R)
    g = LSM(b)
    n = b * R
    base = TOP - 2 * n  # keys end at the largest
    keys, vals = [], []  # in order of insertion; value 0: deleted
    for i in range(R):
        k = base + rng.integers(0, 2 * n + 1, b)
        k[0] = TOP if i % 3 == 0 else k[0]
        if i % 5 == 1:
            k[: min(b // 2, 90)] = base + n  # a run longer than a walk's steps
        k = k.astype(np.uint32)
        if i % 4 == 3:
            block = base + int(rng.integers(0, n)) + np.arange(b)
            g.delete(dev(block))
            keys.append(block)
            vals.append(np.zeros(b, np.int64))
        else:
            v = rng.integers(1, 2**32, b, dtype=np.uint64).astype(np.uint32)
            g.insert(dev(k), dev(v))
            keys.append(k.astype(np.int64))
            vals.append(v.astype(np.int64))
    u, first = np.unique(np.concatenate(keys)[::-1], return_index=True)
    v = np.concatenate(vals)[::-1][first]  # the newest of every key
    live, val = u[v != 0], v[v != 0]
    nq = 140001
    lo = base + rng.integers(0, 2 * n + 1, nq)
    # Waves of ranges of 1, 4, 12 and 16 keys, of every width, and open ones.
    width = np.repeat([2, 8, 24, 32, 0], nq // 5 + 1)[:nq]
    hi = lo + rng.integers(0, width + 1)
    lo[-20000:] = TOP - rng.integers(0, 12, 20000)
    hi[-20000:] = rng.choice(np.array([TOP, 2**31, 2**32 - 1], np.int64), 20000)
    lo[::211] = hi[::211] + 1  # empty ranges
    hi = np.minimum(hi, 2**32 - 1)
    lo = np.minimum(lo, 2**32 - 1)
    a, e = np.searchsorted(live, lo), np.searchsorted(live, hi, side="right")
    want = np.maximum(e - a, 0)
    dlo, dhi = dev(lo), dev(hi)
    assert np.array_equal(host(g.count(dlo, dhi)), want), "counts differ"
    off, gk, gv = g.range(dlo, dhi, cap=int(want.sum()))
    torch.cuda.synchronize()
    offs = np.r_[0, np.cumsum(want)]
    assert np.array_equal(host(off).astype(np.int64), offs), "offsets differ"
    at = np.arange(offs[-1]) + np.repeat(a - offs[:-1], want)
    assert np.array_equal(host(gk).astype(np.int64), live[at]), "keys differ"
    assert np.array_equal(host(gv).astype(np.int64), val[at]), "values differ"
    g.close()
