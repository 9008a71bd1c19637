"""A launch is cut where the grid ends: append at 524 280 pages and 32 767 kv heads, gather at 262 136 pages and 65 535 kv
heads, the decode kernel folds its items at 65 535 and the merge of hundreds of items its workgroups at 2^22.  Lists just above those limits, little of them in use: what lies
around each cut is where it belongs, and nothing else is touched."""
import numpy as np
import pytest
import torch

from paper_2605_17170_amd import harness, tkv

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import gpu_common
    return gpu_common


def test_append_and_gather_beyond_the_pages_of_a_launch(G):
    from oracle import tkv_oracle as orc
    n = 8 * 65535 + 5
    places = np.array([0, 262135, 262136, 262143, 524271, 524272, 524279, 524280, n - 1])     # in the work list
    lens = np.array([64, 3, 64, 1, 64, 5, 64, 64, 2])
    T = int(lens.sum())
    _, K, V, _ = G.random_case(301, [T], 1, 1)
    bits = np.full(T, 2, np.uint8)
    rng = np.random.default_rng(301)
    pages = rng.permutation(n).astype(np.int32)
    at = np.concatenate([np.stack([np.full(m, k), np.sort(rng.permutation(64)[:m])], 1) for k, m in enumerate(lens)])   # (place, slot) of the tokens
    work = torch.full((n, 64), -1, dtype=torch.int32, device=G.DEV)
    rows = np.full((places.size, 64), -1, np.int32)
    rows[at[:, 0], at[:, 1]] = np.arange(T)
    work[torch.from_numpy(places).to(G.DEV)] = torch.from_numpy(rows).to(G.DEV)
    desc = tkv.tkv_desc.make(1, n, 1)
    pool = torch.zeros(tkv.tkv_pool_bytes(desc), dtype=torch.uint8, device=G.DEV)
    bmap = torch.zeros(n + 1, dtype=torch.uint8, device=G.DEV)
    status = torch.zeros(1, dtype=torch.int32, device=G.DEV)
    d_pages = torch.from_numpy(pages).to(G.DEV)
    tkv.tkv_quantize_append(desc, pool, bmap, harness.bf16_tensor(K, G.DEV), harness.bf16_tensor(V, G.DEV), torch.from_numpy(bits).to(G.DEV),
                            d_pages, work, status)
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    Kq, Vq = orc.quantize(K, bits), orc.quantize(V, bits)
    want, want_map = np.zeros(places.size * 6144 + 10240, np.uint8), np.zeros(places.size + 1, np.uint8)
    orc.pack_pool(want, want_map, 1, places.size, 1, at[:, 0] * 64 + at[:, 1], bits, Kq, Vq)
    mine = torch.from_numpy(pages[places].astype(np.int64)).to(G.DEV)
    records = pool[:n * 6144].view(n, 6144)
    assert np.array_equal(records[mine].cpu().numpy().reshape(-1), want[:places.size * 6144])
    assert np.array_equal(bmap[mine].cpu().numpy(), want_map[:places.size])
    records[mine] = 0
    bmap[mine] = 0
    assert int(torch.count_nonzero(pool)) == 0 and int(torch.count_nonzero(bmap)) == 0, "another page was written"
    records[mine] = torch.from_numpy(want[:places.size * 6144].reshape(-1, 6144)).to(G.DEV)
    bmap.fill_(2)
    out = [torch.full((T + 1, 1, 128), float("nan"), dtype=torch.float16, device=G.DEV) for _ in range(2)]
    tkv.tkv_gather_dequant(desc, pool, bmap, d_pages, work, out[0], out[1], status)
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    for got, q in zip(out, (Kq, Vq)):
        assert np.array_equal(got[:T].cpu().numpy().view(np.uint16), orc.dequantize_f16(*q)) and bool(torch.isnan(got[T]).all())


def test_append_and_gather_beyond_the_heads_of_a_launch(G):
    from oracle import tkv_oracle as orc
    heads, few = 65537, 7                                       # head h holds what head h % 7 of the oracle holds
    bits = np.array([2, 4, 2, 4, 2], np.uint8)
    _, K, V, _ = G.random_case(302, [5], few, few)
    slots = np.array([3, 64 + 17, 40, 64 + 63, 0], np.int64)
    Kq, Vq = orc.quantize(K, bits), orc.quantize(V, bits)
    want, want_map = np.zeros(few * (6144 + 10240), np.uint8), np.zeros(2, np.uint8)
    orc.pack_pool(want, want_map, few, 1, 1, slots, bits, Kq, Vq)
    dev = lambda a: torch.from_numpy(a).to(G.DEV)  # noqa: E731
    which = torch.arange(heads, device=G.DEV) % few
    desc = tkv.tkv_desc.make(heads, 1, 1)
    pool = torch.zeros(tkv.tkv_pool_bytes(desc), dtype=torch.uint8, device=G.DEV)
    bmap, status = torch.zeros(2, dtype=torch.uint8, device=G.DEV), torch.zeros(1, dtype=torch.int32, device=G.DEV)
    work_src = np.full((2, 64), -1, np.int32)
    work_src.reshape(-1)[slots] = np.arange(5)
    d_pages, d_src = dev(np.array([0, 1], np.int32)), dev(work_src)
    tkv.tkv_quantize_append(desc, pool, bmap, *(harness.bf16_tensor(x, G.DEV)[:, which].contiguous() for x in (K, V)), dev(bits), d_pages, d_src, status)
    torch.cuda.synchronize()
    assert int(status.item()) == 0 and np.array_equal(bmap.cpu().numpy(), want_map)
    cut, cut_few = heads * 6144, few * 6144
    assert torch.equal(pool[:cut].view(heads, 6144), dev(want[:cut_few].reshape(few, 6144))[which])
    assert torch.equal(pool[cut:].view(heads, 10240), dev(want[cut_few:].reshape(few, 10240))[which])
    out = [torch.full((6, heads, 128), float("nan"), dtype=torch.float16, device=G.DEV) for _ in range(2)]
    tkv.tkv_gather_dequant(desc, pool, bmap, d_pages, d_src, out[0], out[1], status)
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    for got, q in zip(out, (Kq, Vq)):
        assert torch.equal(got[:5].view(torch.int16), dev(orc.dequantize_f16(*q).view(np.int16))[:, which]) and bool(torch.isnan(got[5]).all())


def test_decode_beyond_65535_items(G):
    from oracle import tkv_oracle as orc
    batch = 65535 + 6                                           # one item each, all on one page, of 1 .. 64 tokens
    _, K, V, _ = G.random_case(303, [64], 1, 1)
    cache, (Kq, Vq) = G.check_append([np.full(64, 2, np.uint8)], K, V, 1)
    try:
        n2 = (np.arange(batch) % 64 + 1).astype(np.int32)
        indptr, n4 = np.arange(batch + 1, dtype=np.int32), np.zeros(batch, np.int32)
        items, slots = tkv.tkv_plan_decode(cache.desc, indptr, n2, n4, 1)
        assert items.shape[0] == batch
        g = torch.Generator(device=G.DEV)
        g.manual_seed(303)
        q = torch.randn((batch, 2, 128), device=G.DEV, generator=g).to(torch.bfloat16)
        dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(G.DEV)  # noqa: E731
        out = torch.full((batch, 2, 128), float("nan"), dtype=torch.float32, device=G.DEV)
        ws = torch.empty(tkv.tkv_decode_workspace_bytes(cache.desc, batch, 2), dtype=torch.uint8, device=G.DEV)
        ids = np.full(batch, cache.page_ids[0], np.int32)
        tkv.tkv_decode_attention(cache.desc, cache.pool, cache.bit_map, q, dev(indptr), dev(ids), dev(n2), dev(n4), dev(items), dev(slots),
                                 G.SM, out, ws, cache.status)
        torch.cuda.synchronize()
        assert int(cache.status.item()) == 0
        k, v = (dev(orc.dequantize(*x)[:, 0].astype(np.float64)) for x in (Kq, Vq))
        s = G.SM * (q.double().view(-1, 128) @ k.t().contiguous()).view(batch, 2, 64)
        s = s.masked_fill(torch.arange(64, device=G.DEV)[None, None] >= dev(n2)[:, None, None], float("-inf"))
        ref = (torch.softmax(s, -1).view(-1, 64) @ v).view(batch, 2, 128)
        G.assert_close(out.cpu().numpy(), ref.cpu().numpy(), "%d items" % batch)
    finally:
        cache.close()


@pytest.mark.parametrize("heads", [131072, 131080])   # up to 2^17 the merge kernel of few items, above it the one of hundreds
def test_merge_beyond_the_workgroups_of_a_launch(heads):
    """Four workgroups of 512 threads for each of 16 x 131080 heads are more than 2^32 threads."""
    counts = [1, 3] + [0] * 13 + [2]
    n = sum(counts)
    desc = tkv.tkv_desc.make(heads // 8, 1, 1)
    g = torch.Generator(device="cuda")
    g.manual_seed(304)
    ws = torch.empty(tkv.tkv_decode_workspace_bytes(desc, n, heads) // 4, device="cuda")
    acc, ml = ws[:n * heads * 128].view(n, heads, 128), ws[n * heads * 128:].view(n, heads, 2)
    acc.normal_(generator=g)
    ml[..., 0].normal_(generator=g)
    ml[..., 1].uniform_(1, 300, generator=g)
    out = torch.full((len(counts), heads, 128), float("nan"), device="cuda")
    indptr = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    tkv.tkv_decode_reduce(desc, torch.from_numpy(indptr).cuda(), n, out, ws.view(torch.uint8))
    torch.cuda.synchronize()
    for b, (i0, i1) in enumerate(zip(indptr, indptr[1:])):
        if i0 == i1:
            assert int(torch.count_nonzero(out[b])) == 0
            continue
        m, l = ml[i0:i1, :, 0].double(), ml[i0:i1, :, 1].double()
        w = torch.exp2(m - m.max(0).values)
        num = (w[..., None] * acc[i0:i1].double()).sum(0)
        mag = (w[..., None] * acc[i0:i1].double().abs()).sum(0)
        den = (w * l).sum(0)[:, None]
        # a weight is good to 2^-22, sums of three terms and the division to a few ulps of the magnitudes added
        assert bool(((out[b].double() - num / den).abs() <= 2.0 ** -20 * mag / den).all()), "sequence %d" % b
