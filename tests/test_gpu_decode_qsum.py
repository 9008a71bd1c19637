"""The zero-point term of a key group is its zero-point times the sum of q over the group's channels, and that sum is good to
32 bits: keys that are one number per group (scale 0, so the zero-point is all there is) against q whose large numbers cancel
or belong to another head."""
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


def _q(kind, rng):
    """[1, 8, 128].  The large numbers come in pairs that cancel in the first addition, so 32-bit sums lose nothing."""
    q = np.sign(rng.normal(size=(8, 64, 2))) * 2.0 ** rng.uniform(-5, -3, (8, 64, 2))
    large = 2.0 ** rng.uniform(20, 22, (8, 64))
    pairs = np.arange(64) % 8 == 5                       # two of the sixteen pairs of a group
    heads = slice(0, 8) if kind == "in a group" else slice(2, 3)
    for k in (0, 1):
        q[heads, pairs, k] = (1 - 2 * k) * large[heads][:, pairs]
    return _bf16(q.reshape(1, 8, 128))


@pytest.mark.parametrize("axis", [tkv.TKV_KEYS_PER_TOKEN, tkv.TKV_KEYS_PER_CHANNEL])
@pytest.mark.parametrize("kind", ["in a group", "between heads"])
def test_group_sums_of_q_keep_32_bits(G, kind, axis):
    rng = np.random.default_rng(211)
    n = 200
    q = _q(kind, rng)
    z = np.sign(rng.normal(size=(n, 1, 4, 1))) * 2.0 ** rng.integers(2, 7, (n, 1, 4, 1))
    K = _bf16(np.broadcast_to(z, (n, 1, 4, 32)).reshape(n, 1, 128))
    V = _bf16(rng.normal(size=(n, 1, 128)))
    # per-channel keys have their zero-points inside the product for INT2 pages: the sums serve the INT4 pages
    bits = [np.full(n, 4, np.uint8) if axis == tkv.TKV_KEYS_PER_CHANNEL else np.repeat(np.uint8([2, 4, 2, 4]), n // 4)]
    if axis == tkv.TKV_KEYS_PER_CHANNEL:
        cache, kc = G.kc_check_append(bits, K, V, 1)
        ref = G.kc_decode_ref(q, kc, [n])
    else:
        cache, (Kq, Vq) = G.check_append(bits, K, V, 1)
        ref = G.decode_ref(q, Kq, Vq, [n])
    try:
        out = G.gpu_decode(cache, q, 2)
    finally:
        cache.close()
    # 32-bit logits: good to 2^-21 of the largest sum of terms; weights and products to 2^-19 in all; |out| <= max |V|
    sums = wl.bf16_bits_to_f32(q).astype(np.float64).reshape(8, 4, 32).sum(-1)
    terms = G.SM * np.abs(sums[None] * z.reshape(n, 1, 4)).sum(-1).max()
    tol = float(np.abs(wl.bf16_bits_to_f32(V)).max()) * (terms * 2.0 ** -21 + 2.0 ** -19)
    err = float(np.abs(out - ref).max())
    print("  terms %.2f, error %.2e, tolerance %.2e" % (terms, err, tol), flush=True)
    assert terms > 1 and err <= tol
