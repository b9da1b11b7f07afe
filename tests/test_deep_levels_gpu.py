"""Queries over 20 and 24 occupied levels (b = 1, one bulk insertion and a tail of
single updates): the several-level walks then need more LDS than 64 KiB a
work-group of four waves, with the searches' tops beside them in the
allocation-free range.  Few, more and many queries (each walk's kernels)
against numpy on the live pairs.  Integer results, tolerance 0."""
import ctypes

import numpy as np
import pytest
import torch

from paper_1707_05354_amd.lsm import LSM, LSM_OK
from _gpu import dev, host, note

pytestmark = pytest.mark.gpu

DOMAIN = 60000


def build(levels):
    rng = np.random.default_rng(levels)
    g = LSM(1)
    n = (1 << levels) - 1 - 40
    k = rng.integers(0, DOMAIN, n).astype(np.uint32)
    v = rng.integers(0, 2**32, n, dtype=np.uint64).astype(np.uint32)
    g.bulk_insert(dev(k), dev(v))
    live, val = np.zeros(DOMAIN, bool), np.zeros(DOMAIN, np.uint32)
    live[k] = True
    last = np.full(DOMAIN, -1)
    np.maximum.at(last, k, np.arange(n))
    val[live] = v[last[live]]
    for i in range(40):
        key = np.array([rng.integers(0, DOMAIN)], np.uint32)
        if i % 2:
            g.delete(dev(key))
            live[key] = False
        else:
            x = rng.integers(0, 2**32, 1, dtype=np.uint64).astype(np.uint32)
            g.insert(dev(key), dev(x))
            live[key], val[key] = True, x
    g.flush()
    assert g.occupied() == list(range(levels))
    return g, np.nonzero(live)[0].astype(np.int64), val


@pytest.mark.parametrize("levels", [20, 24])
def test_queries_on_deep_dictionaries(levels):
    note("deep dictionary: %d levels" % levels)
    g, live, val = build(levels)
    rng = np.random.default_rng(2 * levels)
    for nq in (300, 70000, 140001):
        note("deep dictionary: %d levels, %d queries" % (levels, nq))
        lo = rng.integers(0, DOMAIN, nq)
        hi = lo + rng.integers(0, 7, nq)
        lo[::97] = hi[::97] + 1  # empty ranges
        hi[::101] = 2**31 - 1 if nq == 300 else lo[::101]
        a, e = np.searchsorted(live, lo), np.searchsorted(live, hi, side="right")
        n = np.maximum(e - a, 0)
        want = np.concatenate([live[x:y] for x, y in zip(a, e)] + [live[:0]])
        offs = np.r_[0, np.cumsum(n)]
        total = int(offs[-1])
        assert np.array_equal(host(g.count(dev(lo), dev(hi))), n)
        for name in ("lsm_range", "lsm_range_async", "lsm_range_async_noalloc"):
            o = torch.zeros(nq + 1, dtype=torch.int64, device="cuda")
            k, v = (torch.zeros(total + 1, dtype=torch.int32, device="cuda") for _ in range(2))
            dlo, dhi, got = dev(lo), dev(hi), ctypes.c_uint64(0)
            args = [g._h, dlo.data_ptr(), dhi.data_ptr(), nq, o.data_ptr(), k.data_ptr(), v.data_ptr(), total]
            torch.cuda.synchronize()
            rc = getattr(g._lib, name)(*args, *([ctypes.byref(got)] if name == "lsm_range" else []))
            g.sync()
            assert rc == LSM_OK, (name, rc)
            assert np.array_equal(host(o).astype(np.int64), offs), name
            assert np.array_equal(host(k)[:total], want), name
            assert np.array_equal(host(v)[:total], val[want]), name
        q = rng.integers(0, DOMAIN + 5, nq)
        gv, gf = g.lookup(dev(q))
        sk, sv, sf = g.successor(dev(q))
        pk, pv, pf = g.predecessor(dev(q))
        torch.cuda.synchronize()
        i = np.searchsorted(live, q)
        f = (i < live.size) & (live[np.minimum(i, live.size - 1)] == q)
        assert np.array_equal(host(gf), f) and np.array_equal(host(gv), np.where(f, val[np.minimum(q, DOMAIN - 1)], 0))
        s = np.searchsorted(live, q, side="right")
        f = s < live.size
        key = live[np.minimum(s, live.size - 1)]
        assert np.array_equal(host(sf), f) and np.array_equal(host(sk), np.where(f, key, 0))
        assert np.array_equal(host(sv), np.where(f, val[key], 0))
        f = i > 0
        key = live[np.maximum(i - 1, 0)]
        assert np.array_equal(host(pf), f) and np.array_equal(host(pk), np.where(f, key, 0))
        assert np.array_equal(host(pv), np.where(f, val[key], 0))
    g.close()
