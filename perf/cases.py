"""The work that a user of this dictionary has it do, as cases that can be timed.

Every case goes through the public entry points of `paper_1707_05354_amd.lsm.LSM`
on synthetic inputs made on the GPU from a seed.  A case names what is called
(`op`) and the dictionary it is called on: `batches` update batches of `b`,
of which a share `deletes` are delete batches (keys of earlier insertions) and
a share `mixed` are mixed batches; `ragged` batches are partly filled.  Keys
are uniform in [0, 2^31) or Zipf(1.1) in [0, 2^24).

  build    an empty dictionary filled batch by batch; returns the levels
  session  a build followed by lookups, counts and ranges, as in a short script
  submit   log-normal user batches packed by the coalescer; returns the levels
  bulk     one bulk insertion (into an empty or a filled dictionary)
  lookup, count, range, order   one query call on a resident dictionary
  serve    epochs of queries and coalesced updates, then a cleanup
"""
import math

import torch

from paper_1707_05354_amd.lsm import LSM

KEY_BITS = 31
ZIPF_BITS = 24


def listed():
    return [
        # The smallest script: a dictionary of 20 small batches, a few queries
        # of each kind.  Launches and latency are all of it.
        {"name": "session_b1024", "op": "session", "b": 1024, "batches": 20, "deletes": 0.2, "nq": 4096, "hits": 8},
        # A point query from an application thread: a handful of keys.
        {"name": "lookup_64_keys", "op": "lookup", "b": 65536, "batches": 173, "deletes": 0.1, "nq": 64},
        # The paper's build: 2^26 slots in batches of 2^16, a tenth deletes.
        {"name": "build_b64k", "op": "build", "b": 65536, "batches": 1024, "deletes": 0.1},
        # Updates as they come: an odd batch size, partly filled batches,
        # insertions and deletions in the same batch.
        {"name": "build_ragged_mixed", "op": "build", "b": 50021, "batches": 75, "deletes": 0.15, "mixed": 0.25, "ragged": True},
        # Skewed keys: the same keys replaced and deleted again and again.
        {"name": "build_zipf_b32k", "op": "build", "b": 32768, "batches": 255, "deletes": 0.2, "zipf": True},
        # Lookups right after a power-of-two build: one level of 2^26.
        {"name": "lookup_1_level", "op": "lookup", "b": 65536, "batches": 1024, "deletes": 0.1, "nq": 1 << 22},
        # The other end of the same build: every level below 2^26 is full.
        {"name": "lookup_10_levels", "op": "lookup", "b": 65536, "batches": 1023, "deletes": 0.1, "nq": 1 << 22},
        # Range queries over ten levels (counts, offsets and pairs).
        {"name": "range_10_levels", "op": "range", "b": 65536, "batches": 1023, "deletes": 0.1, "nq": 1 << 20, "hits": 16},
        # Ordered access: the next and the previous key.
        {"name": "order_7_levels", "op": "order", "b": 65536, "batches": 381, "deletes": 0.1, "nq": 1 << 20},
        # Many user batches smaller than b, packed by the coalescer.
        {"name": "submit_lognormal", "op": "submit", "b": 65536, "user_batches": 512, "median": 4096},
        # Loading a data set at once, of a size that is no power of two.
        {"name": "bulk_50m", "op": "bulk", "b": 65536, "pairs": 50000001},
        # A server's cycle: six epochs of 2^18 mixed operations on 2^24
        # resident pairs (half lookups, a tenth counts and ranges each, the
        # rest coalesced insertions and deletions), then its maintenance.
        {"name": "serve_16m", "op": "serve", "b": 65536, "batches": 256, "deletes": 0.0, "epoch_ops": 1 << 18, "epochs": 6, "hits": 32},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(("session", "build", "build", "build", "submit", "bulk", "lookup", "lookup", "count",
                     "range", "range", "order", "serve"))
    deletes = round(rng.uniform(0.0, 0.3), 2)
    if op == "session":
        return {"op": op, "b": _log(rng, 200, 5000), "batches": rng.randint(3, 40), "deletes": deletes,
                "nq": _log(rng, 100, 20000), "hits": _log(rng, 2, 64)}
    if op == "build":
        b = _log(rng, 256, 1 << 19)
        zipf = rng.random() < 0.35
        r = min(1023, max(3, _log(rng, 1 << 16, 1 << (24 if zipf else 25)) // b))
        case = {"op": op, "b": b, "batches": r, "deletes": deletes}
        if zipf:
            case["zipf"] = True
        elif rng.random() < 0.3:
            case["mixed"] = round(rng.uniform(0.05, 0.5), 2)
        if rng.random() < 0.3:
            case["ragged"], case["batches"] = True, min(r, 250)
        return case
    if op == "submit":
        b = _log(rng, 4096, 1 << 17)
        return {"op": op, "b": b, "user_batches": rng.randint(20, 700), "median": _log(rng, 200, 8192)}
    if op == "bulk":
        case = {"op": op, "b": _log(rng, 4096, 1 << 17), "pairs": _log(rng, 1 << 16, 1 << 25)}
        if rng.random() < 0.4:
            case["batches"] = rng.randint(1, 30)
        return case
    if op == "serve":
        return {"op": op, "b": _log(rng, 1 << 14, 1 << 17), "batches": rng.randint(20, 128), "deletes": 0.0,
                "epoch_ops": _log(rng, 1 << 14, 1 << 18), "epochs": rng.randint(2, 6), "hits": _log(rng, 4, 64)}
    b = _log(rng, 1 << 12, 1 << 17)
    r = min(1024, max(1, _log(rng, 1 << 17, 1 << 26) // b))
    if rng.random() < 0.25:
        r = 1 << (r.bit_length() - 1)  # right after a power of two: one level
    case = {"op": op, "b": b, "batches": r, "deletes": deletes, "nq": _log(rng, 50, 1 << 22)}
    if op in ("count", "range"):
        case["hits"] = _log(rng, 1, 512)
        case["nq"] = max(50, min(case["nq"] // 4, (1 << 24) // case["hits"]))
    elif op == "order":
        case["nq"] = max(50, case["nq"] // 4)
    return case


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _ints(g, n, hi):
    return torch.randint(0, hi, (n,), generator=g, device="cuda", dtype=torch.int64)


def _values(g, n):
    return torch.randint(-(1 << 31), (1 << 31) - 1, (n,), generator=g, device="cuda", dtype=torch.int64).to(torch.int32)


def _keys(g, n, zipf):
    if not zipf:
        return _ints(g, n, (1 << KEY_BITS) - 1).to(torch.int32)
    # Ranks 1 .. 2^24 of the power law x^-1.1, by inverting its integral; the
    # first rank takes 8 % of the draws.
    u = torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    rank = (1.0 - u * (1.0 - 2.0 ** (-0.1 * ZIPF_BITS))) ** -10.0
    mask = (1 << ZIPF_BITS) - 1  # hot keys spread over the key space
    return (((rank.long().clamp_(max=mask) * 0x79B1) & mask) ^ 0x5A5A5A).to(torch.int32)


def _stream(case, g):
    """The update batches: (kind, keys, vals, delete flags), one tensor each."""
    b, r = case["b"], case["batches"]
    keys = _keys(g, b * r, case.get("zipf")).view(r, b)
    vals = _values(g, b * r).view(r, b)
    pick = torch.rand(r, generator=torch.Generator().manual_seed(r + b)).tolist()
    mixed, deletes = case.get("mixed", 0.0), case.get("deletes", 0.0)
    out, seen = [], []
    for i in range(r):
        n = b
        if case.get("ragged"):
            n = 1 + int(pick[i] * 7919 % 1.0 * b)
        k, v = keys[i, :n], vals[i, :n]
        if seen and pick[i] < deletes:
            if not case.get("zipf"):  # a skewed stream deletes by its own law
                rows = torch.tensor(seen, device="cuda")[_ints(g, n, len(seen))]
                k = keys[rows, _ints(g, n, b) if not case.get("ragged") else 0]
            out.append(("delete", k.contiguous(), None, None))
        elif pick[i] > 1.0 - mixed:
            d = (torch.rand(n, generator=g, device="cuda") < 0.3).to(torch.uint8)
            out.append(("mixed", k, v, d))
            seen.append(i)
        else:
            out.append(("insert", k, v, None))
            seen.append(i)
    return out


def _apply(g, stream):
    for kind, k, v, d in stream:
        if kind == "insert":
            g.insert(k, v)
        elif kind == "delete":
            g.delete(k)
        else:
            g.update(k, v, d)


def _handle(case):
    return LSM(case["b"], key_bits=ZIPF_BITS if case.get("zipf") else KEY_BITS)


def _lookups(g, stream, nq):
    """Half keys that were inserted, half uniform ones."""
    ins = [k for kind, k, _, _ in stream if kind != "delete"]
    rows = torch.randint(0, len(ins), (min(64, len(ins)),), generator=torch.Generator().manual_seed(nq)).tolist()
    pool = torch.cat([ins[i] for i in rows])
    hit = pool[_ints(g, nq, pool.numel())]
    return torch.where(torch.rand(nq, generator=g, device="cuda") < 0.5, hit, _keys(g, nq, False))


def _bounds(g, case, nq):
    """Query bounds that expect case["hits"] resident keys."""
    width = max(1, int(case["hits"] * (1 << KEY_BITS) / (case["b"] * case["batches"])))
    width = min(width, 1 << 30)
    lo = _ints(g, nq, (1 << KEY_BITS) - width)
    return lo.to(torch.int32), (lo + (width - 1)).to(torch.int32)


def _pair_buffers(case, nq):
    """Offsets, keys and values of a range call, kept by the program: room for
    twice the expected pairs, zero behind the pairs that a call writes."""
    cap = 2 * case["hits"] * nq + 4096
    new = lambda n, t: torch.zeros(n, dtype=t, device="cuda")  # noqa: E731
    return new(nq + 1, torch.int64), new(cap, torch.int32), new(cap, torch.int32)


def _user_batches(case, g):
    n = case["user_batches"]
    z = torch.randn(n, generator=torch.Generator().manual_seed(n))
    sizes = torch.exp(math.log(case["median"]) + z).round().clamp(16, 65536).long().tolist()
    keys, vals = _keys(g, sum(sizes), False), _values(g, sum(sizes))
    out, at = [], 0
    for i, s in enumerate(sizes):
        k = keys[at:at + s]
        if i % 10 == 9:  # every tenth deletes keys of earlier user batches
            k = keys[_ints(g, s, at)]
        out.append((k, vals[at:at + s], i % 10 == 9))
        at += s
    return out


def prepare(case, seed):
    g, op = _gen(seed), case["op"]
    s = {"case": case, "lsm": _handle(case)}
    if op in ("build", "session"):
        s["stream"] = _stream(case, g)
    if op == "session":
        s["q"] = _lookups(g, s["stream"], case["nq"])
        s["lo"], s["hi"] = _bounds(g, case, max(1, case["nq"] // 4))
        s["pairs"] = _pair_buffers(case, s["lo"].numel())
    elif op == "submit":
        s["users"] = _user_batches(case, g)
    elif op == "bulk":
        s["keys"], s["vals"] = _keys(g, case["pairs"], False), _values(g, case["pairs"])
        s["stream"] = _stream(case, g) if case.get("batches") else []
    elif op in ("lookup", "count", "range", "order", "serve"):
        s["stream"] = _stream(case, g)
        _apply(s["lsm"], s["stream"])
        s["lsm"].flush()
        if op in ("lookup", "order"):
            s["q"] = _lookups(g, s["stream"], case["nq"])
        elif op != "serve":
            s["lo"], s["hi"] = _bounds(g, case, case["nq"])
            s["pairs"] = _pair_buffers(case, case["nq"])
        else:
            s["epochs"] = [_epoch(case, g, s["stream"]) for _ in range(case["epochs"])]
        del s["stream"]
    return s


def _epoch(case, g, stream):
    ops = case["epoch_ops"]
    nl, nc, nu = ops // 2, max(1, ops // 10), max(1, 3 * ops // 10)
    e = {"q": _lookups(g, stream, nl)}
    e["clo"], e["chi"] = _bounds(g, case, nc)
    e["rlo"], e["rhi"] = _bounds(g, case, nc)
    d = (torch.rand(nu, generator=g, device="cuda") < 1 / 6).to(torch.uint8)
    old = stream[0][1][_ints(g, nu, case["b"])]
    e["uk"], e["uv"], e["ud"] = torch.where(d != 0, old, _keys(g, nu, False)), _values(g, nu), d
    new = lambda n, t: torch.zeros(n, dtype=t, device="cuda")  # noqa: E731
    e["out"] = {"vals": new(nl, torch.int32), "found": new(nl, torch.uint8), "counts": new(nc, torch.int32),
                "pairs": _pair_buffers(case, nc)}
    return e


def _levels(g):
    return [g.level(i) for i in g.occupied()]


def _range(s):
    offsets, keys, vals = s["pairs"]
    total = s["lsm"].range_raw(s["lo"], s["hi"], offsets, keys, vals, keys.numel())
    return offsets, keys, vals, total


def run(s):
    g, op = s["lsm"], s["case"]["op"]
    if op == "lookup":
        return g.lookup(s["q"])
    if op == "count":
        return g.count(s["lo"], s["hi"])
    if op == "range":
        return _range(s)
    if op == "order":
        return {"next": g.successor(s["q"]), "previous": g.predecessor(s["q"])}
    if op == "serve":
        for e in s["epochs"]:
            o = e["out"]
            g.lookup(e["q"], out=(o["vals"], o["found"]))
            g.count(e["clo"], e["chi"], out=o["counts"])
            g.range_async(e["rlo"], e["rhi"], *o["pairs"], o["pairs"][1].numel())
            g.submit_mixed(e["uk"], e["uv"], e["ud"])
            g.flush()
        live = g.cleanup()
        return {"live": live, "epochs": [e["out"] for e in s["epochs"]], "levels": _levels(g)}
    g.clear()
    if op == "submit":
        for k, v, delete in s["users"]:
            g.submit(k, None if delete else v, delete=delete)
        g.flush()
        return _levels(g)
    _apply(g, s["stream"])
    if op == "bulk":
        g.bulk_insert(s["keys"], s["vals"])
        return _levels(g)
    if op == "build":
        g.flush()
        return _levels(g)
    return {"lookup": g.lookup(s["q"]), "count": g.count(s["lo"], s["hi"]),
            "range": _range(s), "levels": _levels(g)}


# -------------------------------------------------------------------- work
LINE = 128  # a random access to a level costs one line of memory


def _probe_bytes(case, nq):
    """What nq queries read of the resident pairs: a line in every level that
    they cannot skip, and no more than all pairs once."""
    levels = bin(case["batches"]).count("1")
    return min(8 * case["b"] * case["batches"], LINE * levels * nq)


def work(case):
    """A pair read once and written once where pairs go in; for queries, their
    own inputs and outputs and the lines of the levels that they touch."""
    op = case["op"]
    pairs = case["b"] * case.get("batches", 0)
    if op == "build":
        byts = 16 * pairs
    elif op == "submit":
        byts = 16 * case["median"] * 1.6 * case["user_batches"]
    elif op == "bulk":
        byts = 16 * (case["pairs"] + pairs)
    elif op == "session":
        nr = max(1, case["nq"] // 4)
        byts = 16 * pairs + 9 * case["nq"] + nr * (28 + 8 * case["hits"]) + _probe_bytes(case, case["nq"] + 2 * nr)
    elif op == "serve":
        ops = case["epoch_ops"]
        epoch = ops // 2 * 9 + ops // 10 * (28 + 8 * case["hits"]) + 3 * ops // 10 * 17 + _probe_bytes(case, 7 * ops // 10)
        byts = case["epochs"] * epoch + 16 * pairs
    else:
        per = {"lookup": 9, "count": 12, "range": 16 + 8 * case.get("hits", 0), "order": 26}[op]
        byts = case["nq"] * per + _probe_bytes(case, case["nq"])
    return {"bytes": float(byts), "flops": 0.0}


# ------------------------------------------------------------------- exact
def _padded(k, v, status, b):
    """One batch as its level holds it: newest position first, filled up to b
    with copies of its last element, which are its newest."""
    pad = b - k.numel()
    if pad:
        k, v, status = (torch.cat([x, x[-1:].expand(pad)]) for x in (k, v, status))
    return k.flip(0), v.flip(0), status.flip(0)


def _exact_levels(batches, b, first=0):
    """The levels that the batches (newest-first triples of b elements) make:
    level i holds the batches of its bit of the count, sorted by key, newest
    first among equal keys."""
    r = len(batches)
    out = []
    for i in range(r.bit_length()):
        if (r >> i) & 1:
            lo = (r >> (i + 1)) << (i + 1)
            part = batches[lo:lo + (1 << i)][::-1]
            k, v, st = (torch.cat([p[x] for p in part]) for x in range(3))
            order = torch.sort(k, stable=True).indices
            out.append(((k[order] * 2 + st[order]).to(torch.int32), v[order]))
    return out


def _exact_batches(stream, b):
    out = []
    for kind, k, v, d in stream:
        k = k.long()
        if kind == "insert":
            t = _padded(k, v, torch.ones_like(k), b)
        elif kind == "delete":
            t = _padded(k, torch.zeros_like(k, dtype=torch.int32), torch.zeros_like(k), b)
        else:
            st = 1 - d.long()
            t = _padded(k, torch.where(d != 0, torch.zeros_like(v), v), st, b)
            order = torch.sort(t[2], stable=True).indices  # tombstones of a mixed batch first
            t = tuple(x[order] for x in t)
        out.append(t)
    return out


def _exact_live(batches):
    """Keys (64 bits, ascending) and values of the live pairs."""
    k, v, st = (torch.cat([p[x] for p in batches[::-1]]) for x in range(3))
    k, order = torch.sort(k, stable=True)
    first = torch.ones_like(k, dtype=torch.bool)
    first[1:] = k[1:] != k[:-1]
    keep = first & (st[order] == 1)
    return k[keep], v[order][keep]


def _exact_lookup(k, v, q):
    i = torch.searchsorted(k, q.long()).clamp_(max=k.numel() - 1)
    found = k[i] == q.long()
    return torch.where(found, v[i], torch.zeros_like(v[i])), found.to(torch.uint8)


def _exact_range(k, v, lo, hi, cap):
    a, e = torch.searchsorted(k, lo.long()), torch.searchsorted(k, hi.long(), right=True)
    offsets = torch.cat([a.new_zeros(1), torch.cumsum(e - a, 0)])
    total = int(offsets[-1])
    at = torch.arange(total, device="cuda") + torch.repeat_interleave(a - offsets[:-1], e - a)
    keys, vals = v.new_zeros(cap), v.new_zeros(cap)
    keys[:total], vals[:total] = k[at].to(torch.int32), v[at]
    return offsets, keys, vals, total


def exact(case, seed):
    """run()'s answer by 64-bit sorts and searches of torch; a serve case's
    epochs each change the pairs that the next one sees, and get none."""
    g, op = _gen(seed), case["op"]
    b = case["b"]
    if op == "serve":
        return None
    if op == "submit":
        users = _user_batches(case, g)
        k = torch.cat([x[0] for x in users]).long()
        st = torch.cat([torch.full_like(x[0], 0 if x[2] else 1) for x in users]).long()
        v = torch.cat([torch.zeros_like(x[1]) if x[2] else x[1] for x in users])
        return _exact_levels([_padded(k[i:i + b], v[i:i + b], st[i:i + b], b) for i in range(0, k.numel(), b)], b)
    if op == "bulk":
        k, v = _keys(g, case["pairs"], False).long(), _values(g, case["pairs"])
        stream = _stream(case, g) if case.get("batches") else []
        new = [_padded(k[i:i + b], v[i:i + b], torch.ones_like(k[i:i + b]), b) for i in range(0, k.numel(), b)]
        return _exact_levels(_exact_batches(stream, b) + new, b)
    stream = _stream(case, g)
    batches = _exact_batches(stream, b)
    if op == "build":
        return _exact_levels(batches, b)
    k, v = _exact_live(batches)
    if op == "session":
        q = _lookups(g, stream, case["nq"])
        lo, hi = _bounds(g, case, max(1, case["nq"] // 4))
        pairs = _exact_range(k, v, lo, hi, _pair_buffers(case, lo.numel())[1].numel())
        return {"lookup": _exact_lookup(k, v, q), "count": pairs[0].diff().to(torch.int32), "range": pairs,
                "levels": _exact_levels(batches, b)}
    if op in ("count", "range"):
        pairs = _exact_range(k, v, *_bounds(g, case, case["nq"]), _pair_buffers(case, case["nq"])[1].numel())
        return pairs if op == "range" else pairs[0].diff().to(torch.int32)
    q = _lookups(g, stream, case["nq"])
    if op == "lookup":
        return _exact_lookup(k, v, q)
    out = {}
    for name, i in (("next", torch.searchsorted(k, q.long(), right=True)), ("previous", torch.searchsorted(k, q.long()) - 1)):
        found = (i >= 0) & (i < k.numel())
        i = i.clamp(0, k.numel() - 1)
        zero = torch.zeros_like(v[i])
        out[name] = (torch.where(found, k[i].to(torch.int32), zero), torch.where(found, v[i], zero), found.to(torch.uint8))
    return out
