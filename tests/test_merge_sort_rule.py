"""The rank rule of the merge sort, in Python: tiles sorted by runs, then runs
merged 16 at a time, every element placed by the counts of smaller keys in the
other runs of its own system, against a stable sort by (system, key, slot).

Same arithmetic as the kernels, with tiles of 64 and first runs of 4 so that
small inputs pass several merge levels; systems of every size between them
(empty, one particle, straddling tiles and groups of tiles), many equal keys."""
import random

import pytest

TILE, RUN, FAN = 64, 4, 16


def _system(offs, q):
    r = 0
    for i in range(len(offs) - 1):
        if offs[i] <= q:
            r = i
    return offs[r], offs[r + 1]


def _search(keys, k, lo, hi, upper, steps):
    for _ in range(steps):
        if lo < hi:
            mid = (lo + hi) >> 1
            if keys[mid] < k or (upper and keys[mid] == k):
                lo = mid + 1
            else:
                hi = mid
    assert lo >= hi, "search did not end"
    return lo


def _lds_merge4(keys, ids, n, seg, run):
    ko, io = [0] * TILE, [None] * TILE
    for p in range(n):
        s0, s1 = seg(p)
        g0, m = p - p % (4 * run), (p // run) & 3
        at = max(s0, g0) + p - max(s0, g0 + m * run)
        for u in range(3):
            j = u + (1 if u >= m else 0)
            lo = max(s0, g0 + j * run)
            hi = max(lo, min(s1, g0 + j * run + run))
            at += _search(keys, keys[p], lo, hi, u < m, run.bit_length()) - lo
        assert io[at] is None
        ko[at], io[at] = keys[p], ids[p]
    return ko, io


def _sort_tile(keys, offs, b):
    n = min(TILE, len(keys) - b)

    def seg(p):
        s, e = _system(offs, b + p)
        return max(s - b, 0), min(e - b, TILE)

    ka = keys[b:b + n] + [0] * (TILE - n)
    kb, ib = [0] * TILE, [None] * TILE
    for p in range(n):
        s0, s1 = seg(p)
        w0 = p - p % RUN
        a, e = max(s0, w0), min(s1, w0 + RUN)
        at = a + sum(ka[j] < ka[p] or (ka[j] == ka[p] and j < p) for j in range(a, min(e, n)))
        kb[at], ib[at] = ka[p], p
    for run in (RUN, 4 * RUN):
        kb, ib = _lds_merge4(kb, ib, n, seg, run)
    return kb[:n], [b + i for i in ib[:n]]


def _merge(keys, slots, offs, R):
    n = len(keys)
    ko, so = [None] * n, [None] * n
    for q in range(n):
        off0, off1 = _system(offs, q)
        o = off0 & ~(TILE - 1)
        run = (q - o) // R
        m = run & (FAN - 1)
        g0 = o + (run - m) * R
        at = max(off0, g0) + q - max(off0, g0 + m * R)
        for h in range(0, FAN, 8):
            if h > 0 and g0 + h * R >= off1:
                break
            part = []
            for u in range(8):
                a = g0 + (h + u) * R
                lo = min(off1, max(off0, a))
                part.append((lo, lo if h + u == m else max(lo, min(off1, a + R)), h + u < m))
            steps = max(hi - lo for lo, hi, _ in part).bit_length()
            at += sum(_search(keys, keys[q], lo, hi, up, steps) - lo for lo, hi, up in part)
        assert ko[at] is None
        ko[at], so[at] = keys[q], slots[q]
    return ko, so


@pytest.mark.parametrize("seed", range(40))
def test_ranks_are_the_stable_order(seed):
    rng = random.Random(seed)
    offs = [0]
    for _ in range(rng.choice([1, 1, 2, 5, 9])):
        offs.append(offs[-1] + rng.choice([0, 1, 3, 17, 64, 65, 100, 300, 1500]))
    n = offs[-1]
    keys = [rng.randrange(rng.choice([3, 50, 10 ** 6])) for _ in range(n)]
    order = [i for r in range(len(offs) - 1)
             for i in sorted(range(offs[r], offs[r + 1]), key=lambda i: (keys[i], i))]
    k, s = [], []
    for b in range(0, n, TILE):
        kt, st = _sort_tile(keys, offs, b)
        k += kt
        s += st
    largest = max(offs[i + 1] - offs[i] for i in range(len(offs) - 1))
    reach = n if len(offs) == 2 else largest + TILE - 1
    R = TILE
    while R < reach:
        k, s = _merge(k, s, offs, R)
        R *= FAN
    assert s == order
