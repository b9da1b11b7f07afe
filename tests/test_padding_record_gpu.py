"""The padding of partly filled batches does not count as a large bucket: after a
batch that sends the next one to digit passes (many keys in one bucket), partly
filled batches of spread keys go back to the top-digit sort, whichever sort
measured them.  Levels byte for byte against the cascade oracle.  Tolerance 0."""
import numpy as np
import pytest

from _gpu import Trio, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["insert", "delete", "mixed", "top"])
@pytest.mark.parametrize("n", [1, 8000, 30000])
def test_padded_batches_leave_digit_passes(kind, n):
    b = 1 << 15
    note("padding record: %s n=%d" % (kind, n))
    rng = np.random.default_rng(n)
    t = Trio(b)
    got = ""
    for i in range(6):
        size = b if i == 0 else n
        k = rng.integers(0, 1 << 20 if i == 0 else 1 << 31, size).astype(np.uint32)
        if kind == "top" and i > 0:
            k[-1] = 2**31 - 1  # the padding in the last digit
        v = rng.integers(0, 2**32, size, dtype=np.uint64).astype(np.uint32)
        before = t.g.stats().sorts_digit_passes
        if kind == "delete" and i > 0:
            t.delete(k)
        elif kind == "mixed" and i > 0:
            t.mixed(k, v, (rng.random(size) < 0.5).astype(np.uint8))
        else:
            t.insert(k, v)
        t.check_levels()  # synchronises, so the next choice sees this sort
        got += "D" if t.g.stats().sorts_digit_passes > before else "T"
    assert got == "TDTTTT"
    t.g.close()
