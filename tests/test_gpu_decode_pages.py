"""The decode kernel walks an item's pages from a list of 64 it holds in registers, asks for nothing behind the last
page, and finds its q operands per (kv head, query heads per kv head): items of one page up to several lists, with the
switch from INT2 to INT4 pages at the edges of a list."""
import numpy as np
import pytest
import torch

from paper_2605_17170_amd import harness, tkv

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import gpu_common
    return gpu_common


def _case(G, seed, pages2, pages4, last, hq, hkv):
    """One sequence with that many pages of either width, the last page of each holding `last` tokens."""
    n2, n4 = (max(0, 64 * p - 64 + last) if p else 0 for p in (pages2, pages4))
    q, K, V, _ = G.random_case(seed, [n2 + n4], hq, hkv)
    return q, K, V, [np.concatenate([np.full(n2, 2, np.uint8), np.full(n4, 4, np.uint8)])]


@pytest.mark.parametrize("pages2,pages4", [(1, 0), (0, 1), (63, 1), (64, 0), (64, 1), (65, 0), (1, 64), (0, 65), (100, 29), (40, 100)])
@pytest.mark.parametrize("hq,hkv", [(8, 1), (3, 3)])
def test_one_item_over_several_lists_of_pages(G, pages2, pages4, hq, hkv):
    q, K, V, seq_bits = _case(G, 71 + pages2, pages2, pages4, 17, hq, hkv)
    cache, (Kq, Vq) = G.check_append(seq_bits, K, V, hkv, fill=0x7C)
    try:
        ref = G.decode_ref(q, Kq, Vq, [seq_bits[0].size])
        for target in (1, 2):
            G.assert_close(G.gpu_decode(cache, q, target), ref, "%d + %d pages, %d items" % (pages2, pages4, target))
    finally:
        cache.close()


@pytest.mark.parametrize("pages2,pages4", [(1, 0), (64, 1), (65, 2), (70, 70)])
def test_one_item_over_several_lists_of_pages_channel_keys(G, pages2, pages4):
    q, K, V, seq_bits = _case(G, 90 + pages2, pages2, pages4, 32, 16, 2)
    cache, ref = G.kc_check_append(seq_bits, K, V, 2)
    try:
        G.assert_close(G.gpu_decode(cache, q, 1), G.kc_decode_ref(q, ref, [seq_bits[0].size]), "%d + %d pages" % (pages2, pages4))
    finally:
        cache.close()


@pytest.mark.parametrize("at,bad", [(0, -1), (0, 1 << 20), (69, 1 << 20), (129, -5), (63, None), (64, None)])
def test_a_page_id_outside_its_pool_is_flagged_and_skipped(G, at, bad):
    """bad = None: a page of the other pool."""
    from oracle import tkv_oracle as orc
    q, K, V, seq_bits = _case(G, 101, 100, 30, 64, 4, 1)
    cache, (Kq, Vq) = G.check_append(seq_bits, K, V, 1)
    try:
        cache.plan_decode(1)
        ids = cache.page_ids.copy()
        lost = ids[at]
        ids[at] = bad if bad is not None else (cache.P2 if at < 100 else 0)
        cache.d_page_ids = torch.from_numpy(ids).to(G.DEV)
        out = cache.decode(harness.bf16_tensor(q, G.DEV))
        torch.cuda.synchronize()
        assert int(cache.status.item()) == (tkv.TKV_STATUS_PAGE_RANGE if bad is not None else tkv.TKV_STATUS_BITMAP_MISMATCH)
        keep = np.nonzero(cache.slot_ids // 64 != lost)[0]
        ref = G.decode_ref(q, tuple(a[keep] for a in Kq), tuple(a[keep] for a in Vq), [keep.size])
        G.assert_close(out.cpu().numpy(), ref, "without page %d of the list" % at)
    finally:
        cache.close()


@pytest.mark.parametrize("axis", [tkv.TKV_KEYS_PER_TOKEN, tkv.TKV_KEYS_PER_CHANNEL])
@pytest.mark.parametrize("bits", [0x0000, 0x7fc0, 0xffc1, 0x7f80, 0x0001, 0x0080], ids=["zero", "nan", "-nan", "inf", "subnormal", "smallest"])
def test_one_odd_head_leaves_the_others_alone(G, bits, axis):
    """The heads of a kv head share a power of two found from their exponents: a head of zeros, NaN, infinities or tiny
    numbers must not change what the others give."""
    q, K, V, seq_bits = G.random_case(103, [300], 8, 1)
    q[0, 3, ::5] = bits
    if bits in (0x0000, 0x0001, 0x0080):
        q[0, 3, :] = bits
    if axis == tkv.TKV_KEYS_PER_CHANNEL:
        cache, kc = G.kc_check_append(seq_bits, K, V, 1)
    else:
        cache, (Kq, Vq) = G.check_append(seq_bits, K, V, 1)
    try:
        out = G.gpu_decode(cache, q, 2)
        finite = bits not in (0x7fc0, 0xffc1, 0x7f80)
        if not finite:
            q[0, 3, :] = 0
        ref = G.kc_decode_ref(q, kc, [300]) if axis == tkv.TKV_KEYS_PER_CHANNEL else G.decode_ref(q, Kq, Vq, [300])
        heads = [h for h in range(8) if finite or h != 3]
        G.assert_close(out[:, heads], ref[:, heads], "q head of %#06x" % bits)
    finally:
        cache.close()


@pytest.mark.parametrize("axis", [tkv.TKV_KEYS_PER_TOKEN, tkv.TKV_KEYS_PER_CHANNEL])
@pytest.mark.parametrize("claimed,first", [(1, 0), (63, 0), (64, 0), (65, 0), (70, 0), (128, 0), (130, 5), (200, 136), (200, 137), (70, 70)])
@pytest.mark.parametrize("named", [-1, 0], ids=["nothing", "an-int4-page"])
def test_int2_tokens_without_an_int2_pool_take_nothing_from_the_int4_pages(G, named, claimed, first, axis):
    """The table counts `claimed` INT2 pages, the pool has none: they are flagged, and the item attends over all its INT4
    pages, however many list positions lie between its first one and the first INT4 page."""
    q, K, V, seq_bits = _case(G, 107, 0, 6, 17, 8, 2)
    cache, (Kq, Vq) = G.check_append(seq_bits, K, V, 2)
    try:
        assert cache.P2 == 1   # an unused page in front of the INT4 pages: the same memory without it is a pool of INT4 pages only
        desc = tkv.tkv_desc.make(2, 0, cache.P4, int2_key_axis=axis)
        pool, bit_map = cache.pool[tkv.tkv_pool_bytes(cache.desc) - tkv.tkv_pool_bytes(desc):], cache.bit_map[1:]
        ids = np.concatenate([np.full(claimed, named), cache.page_ids - 1])
        dev = lambda *v: torch.tensor(v, dtype=torch.int32, device=G.DEV)
        items = torch.tensor([[0, first, ids.size, 0]], dtype=torch.int32, device=G.DEV)
        out = torch.empty((1, 8, 128), device=G.DEV)
        workspace = torch.empty(tkv.tkv_decode_workspace_bytes(desc, 1, 8), dtype=torch.uint8, device=G.DEV)
        tkv.tkv_decode_attention(desc, pool, bit_map, harness.bf16_tensor(q, G.DEV), dev(0, ids.size), dev(*ids.tolist()), dev(64 * claimed),
                                 dev(seq_bits[0].size), items, dev(0, 1), G.SM, out, workspace, cache.status)
        torch.cuda.synchronize()
        flags = tkv.TKV_STATUS_PAGE_RANGE | (tkv.TKV_STATUS_BITMAP_MISMATCH if named == 0 else 0)
        assert int(cache.status.item()) == (flags if first < claimed else 0)
        G.assert_close(out.cpu().numpy(), G.decode_ref(q, Kq, Vq, [seq_bits[0].size]), "behind %d INT2 pages" % (claimed - first))
    finally:
        cache.close()
