"""Bulk insertions whose parts go through different sorts one after another: at
b = 2^15 on 63 batches, 49 new ones make parts of 1 batch, 32 and 16 (digit
passes with the histogram, without it, and with it again), by the digit-pass
sort chosen and by the automatic choice after clustered keys.  Levels byte for
byte against the cascade oracle.  Tolerance 0."""
import numpy as np
import pytest

from paper_1707_05354_amd.lsm import LSM
from _gpu import Trio, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r0,k", [(63, 49), (64, 49), (7, 120)])
@pytest.mark.parametrize("chosen", [True, False])
def test_parts_of_every_sort(r0, k, chosen):
    note("bulk parts: r0=%d k=%d chosen=%d" % (r0, k, chosen))
    rng = np.random.default_rng(r0 + k)
    b = 1 << 15
    t = Trio(b)
    if chosen:
        t.g.set_sort_path(LSM.SORT_DIGIT_PASSES)
    domain = 1 << 31 if chosen else 1 << 20
    for _ in range(r0):
        t.insert(rng.integers(0, domain, b).astype(np.uint32),
                 rng.integers(0, 2**32, b, dtype=np.uint64).astype(np.uint32))
    t.check_levels()  # synchronises, so the choice sees the last sort
    for _ in range(2):
        n = k * b - 5
        t.bulk(rng.integers(0, domain, n).astype(np.uint32),
               rng.integers(0, 2**32, n, dtype=np.uint64).astype(np.uint32))
        t.check_levels()
    t.g.close()
