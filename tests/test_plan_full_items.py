"""The decode planner's two ways of cutting a sequence: equal parts, and items filled to the cost of the longest equal
part.  Compared with equal parts (restated here) over small page tables of every mixture of widths."""
import numpy as np
import pytest

from paper_2605_17170_amd import tkv

C2, C4 = 6, 7


def _equal_parts(p2, p4, target):
    """(number of items, cost of the heaviest) of the cut into equal parts, per sequence."""
    cost = [C2 * a + C4 * b for a, b in zip(p2, p4)]
    count = lambda bound: sum(min(a + b, -(-c // bound)) for a, b, c in zip(p2, p4, cost) if c)  # noqa: E731
    bound = next((x for x in range(1, max(1, sum(cost))) if count(x) <= target), max(1, sum(cost)))
    n_all, most = 0, 0
    for a, b, c in zip(p2, p4, cost):
        if not c:
            continue
        n = min(a + b, -(-c // bound))
        begin = 0
        for k in range(n):
            goal = c * (k + 1) // n
            end = goal // C2 if goal < C2 * a else a + (goal - C2 * a) // C4
            end = a + b if k == n - 1 else min(max(end, begin + 1), a + b - (n - 1 - k))
            most = max(most, C2 * max(0, min(end, a) - begin) + C4 * (end - max(begin, a) if end > a else 0))
            begin = end
        n_all += n
    return n_all, most


@pytest.mark.parametrize("target", [1, 3, 8, 20, 45])
def test_items_are_full_and_no_longer_than_the_longest_equal_part(target):
    rng = np.random.default_rng(target)
    for trial in range(120):
        heads = 3 if trial % 2 else 1 + 3072 // target       # more items than run at once: equal parts
        d = tkv.tkv_desc.make(heads, 4096, 4096)
        batch = int(rng.integers(1, 7))
        p2, p4 = rng.integers(0, rng.integers(1, 40), (2, batch))
        if trial % 3 == 0:
            p4[:] = 0
        if trial % 3 == 1:
            p2[:] = 0
        n2, n4 = (np.maximum(0, 64 * p - rng.integers(0, 64, batch)).astype(np.int32) for p in (p2, p4))
        p2, p4 = -(-n2 // 64), -(-n4 // 64)
        ip = np.concatenate([[0], np.cumsum(p2 + p4)]).astype(np.int32)
        items, sip = tkv.tkv_plan_decode(d, ip, n2, n4, target)
        n_equal, heaviest = _equal_parts(p2.tolist(), p4.tolist(), target)
        full = C4 < heaviest <= 16 * C4 and target * heads <= 3072
        most = -(-heaviest // C4) * C4 if full else heaviest
        assert items.shape[0] <= n_equal if full else items.shape[0] == n_equal
        items = items[np.argsort(items[:, 3])]
        for b in range(batch):
            own = items[sip[b]:sip[b + 1]]
            assert np.all(own[:, 0] == b)
            if p2[b] + p4[b] == 0:
                assert own.shape[0] == 0
                continue
            assert own[0, 1] == 0 and own[-1, 2] == p2[b] + p4[b] and np.all(own[1:, 1] == own[:-1, 2])
            cost = [C2 * max(0, min(hi, p2[b]) - lo) + C4 * max(0, hi - max(lo, p2[b])) for _, lo, hi, _ in own]
            assert min(cost) > 0 and max(cost) <= most
            if full:      # a page more would have been too much
                for (_, lo, hi, _), c in zip(own[:-1], cost[:-1]):
                    assert c + (C2 if hi < p2[b] else C4) > most
