"""Pages that receive some of their 64 tokens: the slots that arrive change, nothing else does.  Patterns at the edges of
what the kernel distinguishes: a wavefront's 16 slots, the four tokens of a quad, a block of 32, one token short of a page."""
import numpy as np
import pytest
import torch

from paper_2605_17170_amd import harness, tkv

pytestmark = pytest.mark.gpu

PATTERNS = {
    "first": [0], "last": [63], "quad edges": [3, 4, 15, 16], "one wavefront": range(16, 32), "block edges": [31, 32],
    "one block": range(32, 64), "all but one": [s for s in range(64) if s != 37], "all": range(64), "every fourth": range(2, 64, 4),
}


@pytest.fixture(scope="module")
def G():
    import gpu_common
    return gpu_common


@pytest.mark.parametrize("heads", [1, 3])
def test_only_the_slots_that_arrive_change(G, heads):
    from oracle import tkv_oracle as orc
    n = len(PATTERNS)
    desc = tkv.tkv_desc.make(heads, n, n)
    rng = np.random.default_rng(heads)
    pool = rng.integers(0, 256, tkv.tkv_pool_bytes(desc)).astype(np.uint8)    # what the pages held before
    bmap = np.zeros(2 * n, np.uint8)
    pages, rows, slots, bits = [], [], [], []
    for page in rng.permutation(2 * n):
        row = np.full(64, -1, np.int32)
        for s in list(PATTERNS.values())[page % n]:
            row[s] = len(slots)
            slots.append(int(page) * 64 + s)
            bits.append(2 if page < n else 4)
        pages.append(page)
        rows.append(row)
    slots, bits = np.array(slots, np.int64), np.array(bits, np.uint8)
    order = rng.permutation(slots.size)                                       # the tokens lie in another order
    where = np.empty(slots.size, np.int32)
    where[order] = np.arange(slots.size, dtype=np.int32)
    work_src = np.stack([np.where(r >= 0, where[np.maximum(r, 0)], r) for r in rows]).astype(np.int32)
    slots, bits = slots[order], bits[order]
    _, K, V, _ = G.random_case(60 + heads, [slots.size], heads, heads)
    want_pool, want_map = pool.copy(), bmap.copy()
    orc.pack_pool(want_pool, want_map, heads, n, n, slots, bits, orc.quantize(K, bits), orc.quantize(V, bits))
    dev = lambda a: torch.from_numpy(a).to(G.DEV)  # noqa: E731
    d_pool, d_map, status = dev(pool), dev(bmap), torch.zeros(1, dtype=torch.int32, device=G.DEV)
    tkv.tkv_quantize_append(desc, d_pool, d_map, harness.bf16_tensor(K, G.DEV), harness.bf16_tensor(V, G.DEV), dev(bits),
                            dev(np.array(pages, np.int32)), dev(work_src), status)
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    assert np.array_equal(d_map.cpu().numpy(), want_map)
    diff = np.nonzero(d_pool.cpu().numpy() != want_pool)[0]
    assert diff.size == 0, "pool bytes differ at %s" % diff[:8].tolist()
