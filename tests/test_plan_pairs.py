"""The decode planner's rule for parts of one or two pages: a page more above 2048 (page, kv head) records per page, up to the 3072
wavefronts that the device holds at once."""
import numpy as np
import pytest

from paper_2605_17170_amd import tkv


def _plan(heads, p2, p4, target, axis):
    n2, n4 = (64 * np.array(p, np.int32) for p in (p2, p4))
    ip = np.concatenate([[0], np.cumsum(np.add(p2, p4))]).astype(np.int32)
    return tkv.tkv_plan_decode(tkv.tkv_desc.make(heads, 4096, 4096, int2_key_axis=axis), ip, n2, n4, target)


# (kv heads, INT2 pages, INT4 pages, target items, pages of an item)
CASES = [
    (8, [256], [0], 384, 1), (8, [257], [0], 384, 2), (8, [384], [0], 384, 2),           # 2048, 2056, 3072 records
    (1, [1000, 48], [1000, 0], 3072, 1), (1, [1000, 49], [1000, 0], 3072, 2), (1, [0, 0, 7], [3001, 1, 63], 3072, 2),
    (4, [3] * 90 + [0], [4] * 90 + [1], 768, 2),                                          # an odd page at every end, pairs of both widths
    (3, [1] * 900, [0] * 900, 1024, 1),                                                   # a page each: nothing to pair
    (8, [300], [0], 385, 1), (8, [300], [0], 1000, 1),                                    # more items asked for than run at once
    (8, [512], [0], 384, 2), (8, [513], [0], 384, 3), (8, [400], [368], 384, 3),          # 4096, 4104, 6144 records
    (1, [1000, 1097], [1000, 1000], 3072, 3), (2, [1, 2, 500], [700, 1, 900], 1536, 3),   # odd ends
]


@pytest.mark.parametrize("axis", [tkv.TKV_KEYS_PER_TOKEN, tkv.TKV_KEYS_PER_CHANNEL])
@pytest.mark.parametrize("heads,p2,p4,target,size", CASES)
def test_short_parts_get_a_page_more(heads, p2, p4, target, size, axis):
    items, sip = _plan(heads, p2, p4, target, axis)
    want = [(b, a, min(a + size, x + y)) for b, (x, y) in enumerate(zip(p2, p4)) for a in range(0, x + y, size)]
    assert [tuple(i[:3]) for i in items[np.argsort(items[:, 3])].tolist()] == want
    assert sip.tolist() == [sum(w[0] < b for w in want) for b in range(len(p2) + 1)]
