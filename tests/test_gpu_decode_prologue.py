"""The q operands of the decode kernel are made by the lane that loaded the channels: every (head, channel) of q has to reach
its place, for every head ratio, with items that start with either width and items that cross from INT2 to INT4."""
import numpy as np
import pytest
import torch

from paper_2605_17170_amd import tkv
from paper_2605_17170_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import gpu_common
    return gpu_common


def _bf16(x):
    return torch.from_numpy(np.ascontiguousarray(x, np.float32)).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)


@pytest.mark.parametrize("axis", [tkv.TKV_KEYS_PER_TOKEN, tkv.TKV_KEYS_PER_CHANNEL])
@pytest.mark.parametrize("ratio", [1, 2, 4, 8])
def test_every_channel_of_q_meets_its_key(G, ratio, axis):
    """One channel of q per query is non-zero and the keys differ in every channel: a channel, head or group in the wrong place
    changes the logits by as much as they differ.  Over the passes every head meets every channel with items of INT2 pages, of
    INT4 pages, and of both."""
    rng = np.random.default_rng(ratio)
    hkv, batch, n = 2, 16, 224
    width = [np.full(n, 2, np.uint8), np.full(n, 4, np.uint8), np.repeat(np.uint8([2, 4]), n // 2), np.repeat(np.uint8([2, 4]), [96, n - 96])]
    bits = [width[b % 4] for b in range(batch)]
    K, V = _bf16(rng.normal(size=(batch * n, hkv, 128))), _bf16(rng.normal(size=(batch * n, hkv, 128)))
    if axis == tkv.TKV_KEYS_PER_CHANNEL:
        bits = [np.concatenate([b[b == 2][:(b == 2).sum() // 32 * 32], b[b == 4], np.full((b == 2).sum() % 32, 4, np.uint8)]) for b in bits]
        cache, kc = G.kc_check_append(bits, K, V, hkv)
    else:
        cache, (Kq, Vq) = G.check_append(bits, K, V, hkv)
    # logits below 2^6 in 32 bits, weights of 22 bits, |out| <= max |V|: 2^-16 of it is generous and far below the effect
    tol = float(np.abs(wl.bf16_bits_to_f32(V)).max()) * 2.0 ** -16
    met = np.zeros((4, hkv * ratio, 128), bool)
    try:
        for shift in range(32):
            q = np.zeros((batch, hkv * ratio, 128), np.float32)
            for i, (b, h) in enumerate(np.ndindex(batch, hkv * ratio)):
                c = (4 * shift + b // 4 + 9 * h) % 128   # the four sequences of a kind take four channels
                q[b, h, c] = 8.0 * (1 + h % 3) * (-1) ** i
                met[b % 4, h, c] = True
            q = _bf16(q)
            out = G.gpu_decode(cache, q, batch)
            ref = G.kc_decode_ref(q, kc, [n] * batch) if axis == tkv.TKV_KEYS_PER_CHANNEL else G.decode_ref(q, Kq, Vq, [n] * batch)
            assert float(np.abs(out - ref).max()) <= tol, "pass %d" % shift
    finally:
        cache.close()
    assert met.all()
