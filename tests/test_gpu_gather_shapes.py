"""The gather's grid counts pages in eights and does K before V: work lists around a multiple of eight pages, one head and
several, both key schemes, rows that nobody asked for left alone."""
import numpy as np
import pytest
import torch

from paper_2605_17170_amd import harness, tkv

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import gpu_common
    return gpu_common


@pytest.mark.parametrize("pages2,pages4", [(1, 0), (0, 7), (3, 5), (4, 5), (16, 1)])
@pytest.mark.parametrize("heads,axis", [(1, tkv.TKV_KEYS_PER_TOKEN), (5, tkv.TKV_KEYS_PER_TOKEN), (2, tkv.TKV_KEYS_PER_CHANNEL)])
def test_pages_around_a_multiple_of_eight(G, pages2, pages4, heads, axis):
    from oracle import tkv_oracle as orc
    bits = np.concatenate([np.full(64 * pages2, 2, np.uint8), np.full(64 * pages4, 4, np.uint8)])
    bits = np.random.default_rng(pages2).permutation(bits.reshape(-1, 32)).reshape(-1)
    _, K, V, _ = G.random_case(80 + pages4, [bits.size], heads, heads)
    if axis == tkv.TKV_KEYS_PER_CHANNEL:
        cache, (_, Kq, Vq, tok, bs, bz) = G.kc_check_append([bits], K, V, heads)
    else:
        cache, (Kq, Vq) = G.check_append([bits], K, V, heads)
    try:
        src = cache.work_src.copy()
        src[(src % 5) == 3] = -1                      # some rows are not wanted
        cache.d_work_src = torch.from_numpy(src).to(G.DEV)
        out = [torch.full((bits.size, heads, 128), float("nan"), dtype=torch.float16, device=G.DEV) for _ in range(2)]
        cache.gather(*out)
        torch.cuda.synchronize()
        assert int(cache.status.item()) == 0
        skipped = np.arange(bits.size) % 5 == 3
        gK, gV = (o.cpu().numpy() for o in out)
        assert np.all(np.isnan(gK[skipped])) and np.all(np.isnan(gV[skipped]))
        wK = orc.f64_to_f16(G.kc_dequantized(Kq, Vq, tok, bs, bz)[0]) if axis == tkv.TKV_KEYS_PER_CHANNEL else orc.dequantize_f16(*Kq)
        assert np.array_equal(gK[~skipped].view(np.uint16), wK[~skipped])
        assert np.array_equal(gV[~skipped].view(np.uint16), orc.dequantize_f16(*Vq)[~skipped])
    finally:
        cache.close()
