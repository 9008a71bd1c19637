"""The decode planner's two ways of cutting a sequence: equal parts, and items filled to the longest equal
part.  Compared with equal parts (restated here) over small page tables of every mixture of widths."""
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_2605_17170_amd import tkv

C2, C4 = 6, 7


def _cost(a, lo, hi):
    return C2 * max(0, min(hi, a) - lo) + C4 * max(0, hi - max(lo, a))


def _equal_parts(p2, p4, target):
    """(number of items, pages of the longest, cost of the heaviest) of the cut into equal parts, per sequence."""
    cost = [C2 * a + C4 * b for a, b in zip(p2, p4)]
    count = lambda bound: sum(min(a + b, -(-c // bound)) for a, b, c in zip(p2, p4, cost) if c)  # noqa: E731
    bound = next((x for x in range(1, max(1, sum(cost))) if count(x) <= target), max(1, sum(cost)))
    n_all, longest, heaviest = 0, 0, 0
    for a, b, c in zip(p2, p4, cost):
        if not c:
            continue
        n = min(a + b, -(-c // bound))
        begin = 0
        for k in range(n):
            goal = c * (k + 1) // n
            end = goal // C2 if goal < C2 * a else a + (goal - C2 * a) // C4
            end = a + b if k == n - 1 else min(max(end, begin + 1), a + b - (n - 1 - k))
            longest = max(longest, end - begin)
            heaviest = max(heaviest, _cost(a, begin, end))
            begin = end
        n_all += n
    return n_all, longest, heaviest


def _plan(heads, p2, p4, target, n2=None, n4=None, axis=tkv.TKV_KEYS_PER_TOKEN):
    n2 = (64 * p2).astype(np.int32) if n2 is None else n2
    n4 = (64 * p4).astype(np.int32) if n4 is None else n4
    ip = np.concatenate([[0], np.cumsum(p2 + p4)]).astype(np.int32)
    return tkv.tkv_plan_decode(tkv.tkv_desc.make(heads, 4096, 4096, int2_key_axis=axis), ip, n2, n4, target)


def _check(items, sip, heads, p2, p4, target, axis=tkv.TKV_KEYS_PER_TOKEN):
    """The items cover the pages in order; none has more pages than the longest equal part, none costs more than the heaviest
    (where that has four pages or more).  True if they are full.  (Plans whose parts of one or two pages get a page more are not for
    this function: test_plan_pairs.py.)"""
    n_equal, longest, heaviest = _equal_parts(p2.tolist(), p4.tolist(), target)
    n2, n4, per_token = p2.sum(), p4.sum(), axis == tkv.TKV_KEYS_PER_TOKEN
    roomy = per_token or 5 * sum(-(-(p2 + p4) // max(1, longest))) <= 4 * target
    full = target * heads <= 3072 and (longest == 2 or (longest == 3 and n4 <= 4 * n2 and roomy) or
                                       (longest == 4 and per_token and 3 * n4 <= 2 * n2))
    most = C4 * longest if longest <= 3 else heaviest
    assert items.shape[0] <= n_equal if full else items.shape[0] == n_equal
    items = items[np.argsort(items[:, 3])]
    for b in range(p2.size):
        own = items[sip[b]:sip[b + 1]]
        assert np.all(own[:, 0] == b)
        if p2[b] + p4[b] == 0:
            assert own.shape[0] == 0
            continue
        assert own[0, 1] == 0 and own[-1, 2] == p2[b] + p4[b] and np.all(own[1:, 1] == own[:-1, 2])
        for last, (_, lo, hi, _) in zip([False] * (len(own) - 1) + [True], own):
            assert 0 < hi - lo <= longest and _cost(p2[b], lo, hi) <= most
            assert not full or last or hi - lo == longest or _cost(p2[b], lo, hi + 1) > most    # a page more: too much
    return full


@pytest.mark.parametrize("target", [1, 3, 8, 20, 45])
def test_items_are_full_and_no_longer_than_the_longest_equal_part(target):
    rng = np.random.default_rng(target)
    kinds = set()
    for trial in range(120):
        heads = 3 if trial % 2 else 1 + 3072 // target       # more items than run at once: equal parts
        batch = int(rng.integers(1, 7))
        p2, p4 = rng.integers(0, rng.integers(1, 40), (2, batch))
        if trial % 3 == 0:
            p4[:] = 0
        if trial % 3 == 1:
            p2[:] = 0
        n2, n4 = (np.maximum(0, 64 * p - rng.integers(0, 64, batch)).astype(np.int32) for p in (p2, p4))
        p2, p4 = -(-n2 // 64), -(-n4 // 64)
        items, sip = _plan(heads, p2, p4, target, n2, n4)
        kinds.add(_check(items, sip, heads, p2, p4, target))
    assert target < 8 or kinds == {True, False}


# Equal parts of exactly six pages, nearly all of six, thirteen; then the lines of the rule: two to five pages, INT4 shares
# on both sides of two and four fifths, both key schemes.
SHAPES = [(8, [288] * 8, [0] * 8, 0), (8, [240] * 8, [8] * 8, 0), (8, [240] * 8, [48] * 8, 0), (8, [610] * 8, [0] * 8, 0)]
SHAPES += [(h, [round(x * 3072 / h / 5 * (20 - s) / 20)] * 5, [round(x * 3072 / h / 5 * s / 20)] * 5, axis)
           for h in (1, 8) for x in (1.05, 2.3, 2.6, 3.1, 4.3) for s in (0, 7, 9, 15, 17, 20) for axis in (tkv.TKV_KEYS_PER_TOKEN, tkv.TKV_KEYS_PER_CHANNEL)]


@pytest.mark.parametrize("heads,p2,p4,axis", SHAPES, ids=["%d heads, %d + %d pages, axis %d" % (h, a[0], b[0], k) for h, a, b, k in SHAPES])
def test_plan_at_the_lines_of_the_rule(heads, p2, p4, axis):
    p2, p4 = np.array(p2), np.array(p4)
    target = 3072 // heads
    items, sip = _plan(heads, p2, p4, target, axis=axis)
    _check(items, sip, heads, p2, p4, target, axis)


_NO_MEMORY = """
import ctypes as C, resource
import numpy as np
from paper_2605_17170_amd import tkv
batch = 16 << 20
zero, out, item = np.zeros(batch + 1, np.int32), np.ones(batch + 1, np.int32), np.empty(4, np.int32)
L, desc = tkv.lib(), tkv.tkv_desc.make(1, 8, 8)
def plan(n, indptr, n2, capacity):
    p = lambda a: C.c_void_p(a.ctypes.data)
    return L.tkv_plan_decode(C.byref(desc), n, p(indptr), p(n2), p(zero), 8, p(item), capacity, p(out))
assert plan(2, zero, zero, 1) == 0
size = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (size + (16 << 20), resource.RLIM_INFINITY))
assert plan(batch, zero, zero, 1) == 0 and not out.any()
print("planned")
"""


def test_plan_over_many_sequences_needs_no_memory():
    """A C entry lets no exception out: what the cut into parts needs does not grow with the batch."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    run = subprocess.run([sys.executable, "-c", _NO_MEMORY], cwd=root, capture_output=True, text=True, timeout=100)
    assert run.returncode == 0 and run.stdout.strip() == "planned", run.stderr[-500:]
