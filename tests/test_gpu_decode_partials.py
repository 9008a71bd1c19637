"""Decode with as many items and query heads as fill the device (more than 17408 rows of partials), and fewer: hand-made item lists in
any order with items without pages and malformed ones, what each item leaves in the workspace, a query head of NaN; both key schemes.
Against the oracle, or against the same call without what must not matter."""
import numpy as np
import pytest
import torch

from paper_2605_17170_amd import harness, tkv

pytestmark = pytest.mark.gpu

LENS = [1, 64, 65, 400, 0, 130, 900, 37, 2000, 256, 700, 3000, 5, 1500, 600, 64, 1300, 449]


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import gpu_common
    return gpu_common


def _lists(pages, per, n_items, order, rng):
    """Items of `per` pages, filled up with items without pages to n_items, in sequence order / the planner's / at random."""
    cuts = [[(a, min(p, a + per)) for a in range(0, p, per)] for p in pages]
    while sum(map(len, cuts)) < n_items:
        b = int(rng.integers(0, len(cuts)))
        cuts[b].insert(int(rng.integers(0, len(cuts[b]) + 1)), (3, 3))
    sip = np.concatenate([[0], np.cumsum([len(c) for c in cuts])]).astype(np.int32)
    items = np.array([(b, lo, hi, sip[b] + k) for b, c in enumerate(cuts) for k, (lo, hi) in enumerate(c)], np.int32)
    assert len(items) == n_items
    if order == "random":
        items = items[rng.permutation(n_items)]
    if order == "runs":      # runs of three items of a sequence, the sequences in turn
        turn = np.array([k // 3 for c in cuts for k in range(len(c))])
        items = items[np.argsort(turn, kind="stable")]
    return np.ascontiguousarray(items), sip


@pytest.mark.parametrize("channel_keys", [False, True])
@pytest.mark.parametrize("n_items,order", [(273, "sequence"), (274, "runs"), (275, "random"), (384, "random")])
def test_item_lists_in_any_order(G, n_items, order, channel_keys):
    q, K, V, seq_bits = G.random_case(n_items, LENS, 64, 8)
    if channel_keys:
        cache, ref = G.kc_check_append(seq_bits, K, V, 8)
    else:
        cache, ref = G.check_append(seq_bits, K, V, 8)
    try:
        want = G.kc_decode_ref(q, ref, LENS) if channel_keys else G.decode_ref(q, *ref, LENS)
        pages = np.diff(cache.page_indptr).tolist()
        assert sum(pages) <= 270 and n_items * 64 > 17408
        items, sip = _lists(pages, 1, n_items, order, np.random.default_rng(n_items))
        cache._plan = (torch.from_numpy(items).to(G.DEV), torch.from_numpy(sip).to(G.DEV), items, sip)
        ws = cache.workspace(64)
        outs = []
        for _ in range(3):
            ws.view(torch.float32).fill_(float("nan"))     # what an earlier call left there must not reach the output
            out = cache.decode(harness.bf16_tensor(q, G.DEV), workspace=ws)
            torch.cuda.synchronize()
            outs.append(out.cpu().numpy())
        assert int(cache.status.item()) == 0
        G.assert_close(outs[0], want, "%d items, %s" % (n_items, order))
        assert not outs[0][LENS.index(0)].any()
        assert all(np.array_equal(outs[0], o) for o in outs[1:])
        # an item that names no sequence adds nothing, and its neighbours are whole
        bad = items.copy()
        k = int(np.nonzero((items[:, 0] == 11) & (items[:, 1] < items[:, 2]))[0][0])
        bad[k, 0] = len(LENS)
        cache._plan = (torch.from_numpy(bad).to(G.DEV), cache._plan[1], bad, sip)
        ws.view(torch.float32).fill_(float("nan"))
        out = cache.decode(harness.bf16_tensor(q, G.DEV), workspace=ws)
        torch.cuda.synchronize()
        assert int(cache.status.item()) == tkv.TKV_STATUS_BAD_ITEM
        out, keep = out.cpu().numpy(), np.arange(len(LENS)) != 11
        assert np.isfinite(out).all()
        G.assert_close(out[keep], want[keep], "the other sequences")
    finally:
        cache.close()


# (lengths, query heads, kv heads, items at least): 17408 rows of partials, more, on one kv head too, and more wavefronts than run at once
LARGE = [([1500] * 4, 64, 8, 272), ([700, 9000, 300, 300], 64, 8, 384), ([20000], 8, 1, 3072), ([4096] * 6, 64, 8, 384)]


def _large(G, lens, hq, hkv, target, channel_keys):
    q, K, V, seq_bits = G.random_case(sum(lens) + hq, lens, hq, hkv)
    axis = tkv.TKV_KEYS_PER_CHANNEL if channel_keys else tkv.TKV_KEYS_PER_TOKEN
    cache = harness.PagedCache(hkv, seq_bits, G.DEV, key_axis=axis)
    cache.append(harness.bf16_tensor(K, G.DEV), harness.bf16_tensor(V, G.DEV))
    # single pages, filled up with items without pages to the number asked for
    items, sip = _lists(np.diff(cache.page_indptr).tolist(), 1, max(target, int(cache.page_indptr[-1])), "sequence", np.random.default_rng(1))
    cache._plan = (torch.from_numpy(items).to(G.DEV), torch.from_numpy(sip).to(G.DEV), items, sip)
    return cache, harness.bf16_tensor(q, G.DEV)


@pytest.mark.parametrize("channel_keys", [False, True])
@pytest.mark.parametrize("lens,hq,hkv,target", LARGE, ids=lambda v: None if isinstance(v, list) else str(v))
def test_a_head_of_nan_stays_nan(G, lens, hq, hkv, target, channel_keys):
    """A query head without a number in it has no attention: NaN in every channel of its output, in launches of any size.  The other
    heads and sequences are what they are without it, bit for bit."""
    cache, q = _large(G, lens, hq, hkv, target, channel_keys)
    try:
        want = cache.decode(q).cpu().numpy()
        assert np.isfinite(want).all()
        poisoned = q.clone()
        poisoned[len(lens) // 2, 3] = float("nan")
        got = cache.decode(poisoned).cpu().numpy()
        assert np.isnan(got[len(lens) // 2, 3]).all()
        got[len(lens) // 2, 3] = want[len(lens) // 2, 3]
        assert np.array_equal(got, want)
    finally:
        cache.close()


@pytest.mark.parametrize("channel_keys", [False, True])
@pytest.mark.parametrize("lens,hq,hkv,target", LARGE, ids=lambda v: None if isinstance(v, list) else str(v))
def test_every_item_leaves_its_partial(G, lens, hq, hkv, target, channel_keys):
    """What tkv_decode_split writes: (m, l, acc) of every item and query head in the item's own slot, whatever the size of the launch;
    and tkv_decode_reduce merges them by nothing but the counts it is given."""
    cache, q = _large(G, lens, hq, hkv, target, channel_keys)
    try:
        items, n = cache._plan[2], len(cache._plan[2])
        want = cache.decode(q).cpu().numpy()
        ws = cache.workspace(hq)
        ws.view(torch.float32).fill_(float("nan"))
        cache.decode_split(q, ws)
        f = ws.view(torch.float32).cpu().numpy()
        acc, ml = f[:n * hq * 128].reshape(n, hq, 128), f[n * hq * 128:n * hq * 130].reshape(n, hq, 2)
        empty = np.zeros(n, bool)
        empty[items[:, 3]] = items[:, 1] >= items[:, 2]
        assert np.isfinite(acc).all() and np.isneginf(ml[empty, :, 0]).all() and not ml[empty, :, 1].any() and not acc[empty].any()
        assert np.isfinite(ml[~empty]).all() and (ml[~empty, :, 1] > 0).all()
        for axis in (tkv.TKV_KEYS_PER_TOKEN, tkv.TKV_KEYS_PER_CHANNEL):
            out = torch.full(want.shape, float("nan"), device=G.DEV)
            tkv.tkv_decode_reduce(tkv.tkv_desc.make(hkv, cache.P2, cache.P4, int2_key_axis=axis), cache._plan[1], n, out, ws)
            assert np.array_equal(out.cpu().numpy(), want)
    finally:
        cache.close()
