"""Source rows of an append: slots that name a row outside the input (any 32-bit number) get nothing and read nothing, and inputs
around the sizes at which the launcher changes its loads and its occupancy give the same bytes."""
import numpy as np
import pytest
import torch

from paper_2605_17170_amd import tkv

pytestmark = pytest.mark.gpu

INT32_MAX, INT32_MIN = (1 << 31) - 1, -(1 << 31)


def _append(K, V, bits, pages, src, n2, n4, keys):
    desc = tkv.tkv_desc.make(1, n2, n4, int2_key_axis=keys)
    pool = torch.full((tkv.tkv_pool_bytes(desc),), 0x5A, dtype=torch.uint8, device="cuda")
    bmap = torch.zeros(n2 + n4, dtype=torch.uint8, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    tkv.tkv_quantize_append(desc, pool, bmap, K, V, bits, torch.from_numpy(pages).cuda(), torch.from_numpy(src).cuda(), status)
    torch.cuda.synchronize()
    return pool.cpu().numpy(), bmap.cpu().numpy(), int(status)


def _rows(n, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn((n, 1, 128), device="cuda", generator=g).to(torch.bfloat16)


@pytest.mark.parametrize("n_tokens", [1, 65])
def test_slots_without_a_source_change_nothing(n_tokens):
    K, V = _rows(n_tokens, 1), _rows(n_tokens, 2)
    bits = torch.full((n_tokens,), 4, dtype=torch.uint8, device="cuda")
    src = np.full((2, 64), -1, np.int32)
    src[0, :6] = [n_tokens, n_tokens + 1, INT32_MAX, INT32_MIN, -1, -64]
    src[1, 5], src[1, 6], src[1, 40] = n_tokens - 1, n_tokens, 0
    pages = np.array([0, 1], np.int32)
    pool, bmap, status = _append(K, V, bits, pages, src, 0, 2, tkv.TKV_KEYS_PER_TOKEN)
    assert status == 0 and bmap.tolist() == [0, 4]
    first = tkv.tkv_record_bytes(4)
    assert (pool[:first] == 0x5A).all()
    clean = np.where((src >= 0) & (src < n_tokens), src, -1).astype(np.int32)
    again, _, _ = _append(K, V, bits, pages, clean, 0, 2, tkv.TKV_KEYS_PER_TOKEN)
    assert np.array_equal(pool, again)
    assert (pool[first:] != 0x5A).any()


@pytest.mark.parametrize("keys", [tkv.TKV_KEYS_PER_TOKEN, tkv.TKV_KEYS_PER_CHANNEL])
@pytest.mark.parametrize("mib", [64, 320, 768])
def test_large_inputs_give_the_bytes_of_small_ones(mib, keys):
    """The rows of a few pages, out of an input just at and just above the size where the launcher changes over."""
    at = (mib << 20) // 512
    few = 4 * 64 + 32
    K, V = _rows(few, 3), _rows(few, 4)
    widths = np.repeat(np.uint8([2, 4, 2, 4]), 64)
    bits = torch.from_numpy(np.concatenate([widths, np.full(32, 4, np.uint8)])).cuda()
    src = np.full((5, 64), -1, np.int32)
    src[:4] = np.arange(256).reshape(4, 64)
    src[4, :32] = np.arange(256, few)
    pages = np.array([0, 2, 1, 3, 4], np.int32)
    want = _append(K, V, bits, pages, src, 2, 3, keys)
    for n in (at, at + 1):
        bigK, bigV = torch.zeros((n, 1, 128), dtype=torch.bfloat16, device="cuda"), torch.zeros((n, 1, 128), dtype=torch.bfloat16, device="cuda")
        big_bits = torch.zeros(n, dtype=torch.uint8, device="cuda")
        first = n - few
        bigK[first:], bigV[first:], big_bits[first:] = K, V, bits
        got = _append(bigK, bigV, big_bits, pages, np.where(src >= 0, src + first, -1).astype(np.int32), 2, 3, keys)
        assert want[2] == got[2] == 0 and np.array_equal(want[1], got[1]) and np.array_equal(want[0], got[0])
