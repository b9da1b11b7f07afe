"""Many ranges of few pairs up to the largest key, 2^31 - 1 (its key variable is
all ones), over the numbers of levels that a lane walks alone: the key live in
each level in turn with newer levels that end below it, and deleted in a newer
one.  Offsets, keys and values against the map oracle.  Integer results,
tolerance 0."""
import numpy as np
import pytest

from _gpu import Trio, dev, host, note

pytestmark = pytest.mark.gpu

TOP = 2**31 - 1


@pytest.mark.parametrize("deleted", [False, True])
@pytest.mark.parametrize("R,level", [(R, i) for R in (3, 7, 63) for i in range(R.bit_length())])
def test_narrow_ranges_at_the_largest_key(R, level, deleted):
    note("largest key: R=%d level=%d deleted=%d" % (R, level, deleted))
    rng = np.random.default_rng(100 * R + 2 * level + deleted)
    b = 50
    t = Trio(b)
    first = (R >> (level + 1)) << (level + 1)  # the level's first batch
    for i in range(R):
        k = rng.integers(TOP - 40 * b, TOP - 25, b).astype(np.uint32)
        if i == first + (1 << level) // 2:
            k[b // 2] = TOP
        if i == R - 1 and deleted:
            t.delete(np.r_[k[:3], TOP].astype(np.uint32))
        else:
            t.insert(k, rng.integers(0, 2**32, b, dtype=np.uint64).astype(np.uint32))
    nq = 140001
    lo = TOP - rng.integers(0, 30, nq)
    lo[:1000] = TOP - rng.integers(0, 40 * b, 1000)
    hi = rng.choice(np.array([TOP, TOP + 1, 2**32 - 1], np.int64), nq)
    lo, hi = lo.astype(np.uint32), hi.astype(np.uint32)
    # Waves whose ranges all hold few pairs are walked by lanes; the first
    # thousand ranges take the octets' walk.
    offs, keys, vals = t.m.range(lo, hi)
    go, gk, gv = t.g.range(dev(lo), dev(hi), cap=int(offs[-1]))
    t.g.sync()
    assert np.array_equal(host(go), offs), "offsets differ"
    assert np.array_equal(host(gk), keys), "keys differ"
    assert np.array_equal(host(gv), vals), "values differ"
    assert (keys == TOP).any() != deleted
    t.g.close()
