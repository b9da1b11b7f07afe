"""Cleanup at the edges of its tiles of 2048 elements: merged lists that end on,
before and behind a tile and inside a thread's eight elements, key runs across
threads, waves and tiles, new levels that start inside a tile, nothing valid.
Byte-exact levels against the oracle.  Integer results, tolerance 0."""
import numpy as np
import pytest

from _gpu import Trio, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,R,domain", [
    (1, 7, 1 << 20), (5, 3, 1 << 20), (255, 9, 1 << 20), (683, 3, 1 << 30), (2047, 1, 1 << 31),
    (2048, 3, 1 << 31), (2049, 5, 1 << 31), (1021, 15, 9000), (3000, 7, 40), (64, 127, 1 << 13)])
@pytest.mark.parametrize("gone", [False, True])
def test_tile_edges(b, R, domain, gone):
    note("cleanup tile edges b=%d R=%d domain=%d gone=%s" % (b, R, domain, gone))
    rng = np.random.default_rng(b + R)
    t = Trio(b)
    batches = [rng.integers(0, domain, b, dtype=np.uint64).astype(np.uint32) for _ in range(R)]
    for k in batches:
        t.insert(k, rng.integers(0, 2**32, b, dtype=np.uint64).astype(np.uint32))
    for k in batches if gone else batches[::3]:
        t.delete(k)
    t.cleanup()
    t.check_levels()
    t.g.close()
