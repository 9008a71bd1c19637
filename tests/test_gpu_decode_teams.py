"""Decode with as many items and query heads as make workgroups of four items share one partial per sequence (more than 17408
rows of partials): hand-made item lists in which a workgroup holds one to four sequences in any order, items without pages, lists that
end inside a workgroup, malformed items, both key schemes.  Against the oracle."""
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
    if order == "runs":      # runs of three items of a sequence, the sequences in turn: every workgroup meets two
        turn = np.array([k // 3 for c in cuts for k in range(len(c))])
        items = items[np.argsort(turn, kind="stable")]
    return np.ascontiguousarray(items), sip


@pytest.mark.parametrize("channel_keys", [False, True])
@pytest.mark.parametrize("n_items,order", [(273, "sequence"), (274, "runs"), (275, "random"), (384, "random")])
def test_items_of_a_workgroup_share_a_partial(G, n_items, order, channel_keys):
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
        # an item that names no sequence adds nothing, and its neighbours in the workgroup are whole
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
