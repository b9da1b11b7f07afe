"""The digit passes of sorts above 256 tiles of 2048 elements (chunk counts,
their scan and the chunk-wise scatter, tiles of 8192): bulk-built levels and
single batches byte for byte against the cascade oracle, at sizes around the
path's limit and its tile edges, with padding, deletions, mixed batches,
staged (encoded) batches and long runs of one key.  Integer results,
tolerance 0."""
import numpy as np
import pytest

from paper_1707_05354_amd.lsm import LSM
from _gpu import Trio, note

pytestmark = pytest.mark.gpu

LIMIT = 256 * 2048


def pairs(rng, n, domain, hot=0.0):
    k = rng.integers(0, domain, n, dtype=np.uint64).astype(np.uint32)
    if hot:
        k[rng.random(n) < hot] = domain // 3
    return k, rng.integers(0, 2**32, n, dtype=np.uint64).astype(np.uint32)


@pytest.mark.parametrize("b,n,hot", [
    (LIMIT + 1, LIMIT + 1, 0.0),          # one element over the limit
    (LIMIT + 1, 5, 0.0),                  # nearly all padding
    (65 * 8192, 65 * 8192, 0.3),          # whole tiles, a hot key
    (65 * 8192 + 1, 65 * 8192 - 8191, 0.0),  # padding across tiles
    (513 * 8192 - 1, 513 * 8192 - 1, 0.0),   # two tiles a chunk, the last chunk short
])
def test_single_batches(b, n, hot):
    note("large sort b=%d n=%d hot=%.1f" % (b, n, hot))
    rng = np.random.default_rng(b + n)
    t = Trio(b)
    k, v = pairs(rng, n, 1 << 31, hot)
    t.insert(k, v)
    t.check_levels()
    t.delete(k[: max(1, n // 2)])
    if b < 2**20:
        t.mixed(k, v, (rng.random(n) < 0.5).astype(np.uint8))
    t.check_levels()
    t.g.close()


def test_staged_batch():
    b = LIMIT + 77
    note("large sort of a staged batch b=%d" % b)
    rng = np.random.default_rng(5)
    t = Trio(b)
    k, v = pairs(rng, b, 1 << 20)
    from _gpu import dev, dev_u8
    d = (rng.random(b) < 0.4).astype(np.uint8)
    t.g.submit_mixed(dev(k), dev(v), dev_u8(d))
    t.c.insert_ordered(k, np.where(d, 0, v).astype(np.uint32), (1 - d).astype(np.uint8))
    t.merge_count_comparable = False
    t.check_levels()
    t.g.close()


@pytest.mark.parametrize("batches,tail", [(40, 0), (75, 1), (64, 16384)])
def test_bulk_levels(batches, tail):
    """b = 2^14: the largest levels of the build are above the limit, the
    smaller ones below."""
    b = 1 << 14
    note("large bulk batches=%d tail=%d" % (batches, tail))
    rng = np.random.default_rng(batches)
    t = Trio(b)
    k, v = pairs(rng, batches * b + tail, 1 << 31, 0.05)
    t.bulk(k, v)
    t.check_levels()
    t.g.close()
