"""tkv_decode_reduce on made-up partials: item counts at the edges of the two kernels (alone / shared between wavefronts, batches
of 32, the switch at 128 items per sequence on average, by equal and by skewed counts), both lane widths, skewed and empty sequences,
empty items."""
import numpy as np
import pytest
import torch

from paper_2605_17170_amd import tkv

pytestmark = pytest.mark.gpu


def _case(counts, hq, seed):
    rng = np.random.default_rng(seed)
    n = int(sum(counts))
    acc = rng.normal(size=(n, hq, 128)).astype(np.float32)
    m = rng.normal(size=(n, hq)).astype(np.float32) * 4
    l = rng.uniform(1, 300, (n, hq)).astype(np.float32)
    empty = rng.random((n, hq)) < 0.1
    acc[empty], m[empty], l[empty] = 0.0, -np.inf, 0.0
    return acc, m, l


def _reference(acc, m, l, counts):
    outs, mags, at = [], [], 0
    for c in counts:
        a, mm, ll = (x[at:at + c].astype(np.float64) for x in (acc, m, l))
        at += c
        if c == 0 or not np.isfinite(mm).any():
            outs.append(np.zeros(acc.shape[1:]))
            mags.append(np.zeros(acc.shape[1:]))
            continue
        top = mm.max(0)
        w = np.exp2(mm - np.where(np.isfinite(top), top, 0.0))
        den = (w * ll).sum(0)
        den = np.where(den > 0, den, np.inf)[:, None]
        outs.append((w[:, :, None] * a).sum(0) / den)
        mags.append((w[:, :, None] * np.abs(a)).sum(0) / den)
    return np.stack(outs), np.stack(mags)


def _run(acc, m, l, counts, hq, tail=0):
    """`tail` partials of NaN lie behind the last item."""
    n = acc.shape[0]
    desc = tkv.tkv_desc.make(1, 4, 4) if hq <= 8 else tkv.tkv_desc.make(hq // 8, 4, 4)
    need = tkv.tkv_decode_workspace_bytes(desc, n, hq)
    ws = torch.full((max(16, need) // 4 + tail * hq * 130,), float("nan"), device="cuda")
    ws[:acc.size] = torch.from_numpy(acc.reshape(-1)).cuda()
    ws[acc.size:acc.size + 2 * m.size] = torch.from_numpy(np.stack([m, l], -1).reshape(-1)).cuda()
    sip = torch.from_numpy(np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)).cuda()
    out = torch.full((len(counts), hq, 128), float("nan"), device="cuda")
    tkv.tkv_decode_reduce(desc, sip, n, out, ws.view(torch.uint8))
    torch.cuda.synchronize()
    return out.cpu().numpy()


COUNTS = [[1], [24], [25], [26, 0, 3], [31, 32, 33], [96, 97], [128], [129, 1, 0], [4 * 32 + 1], [255], [256], [257], [1, 1, 1, 700], [0, 0], [600, 40],
          [200, 56], [200, 57], [1, 509, 1, 1], [1, 510, 1, 1]]


@pytest.mark.parametrize("counts, hq", [(c, h) for c in COUNTS for h in (1, 8, 64, 256) if sum(c) * h <= 80000],   # (host memory)
                         ids=lambda v: "-".join(map(str, v)) if isinstance(v, list) else str(v))
def test_merge_of_partials(counts, hq):
    acc, m, l = _case(counts, hq, sum(counts) + hq)
    got = _run(acc, m, l, counts, hq, tail=40)
    ref, mag = _reference(acc, m, l, counts)
    # a weight is good to 2^-22 (difference of two numbers below 2^5, exp2 to an ulp), a sum of n terms to n / 2 more ulps in
    # any order, numerator and denominator alike
    tol = (2.0 ** -21 + max(counts) * 2.0 ** -23) * mag + 1e-30
    assert np.isfinite(got).all()
    assert (np.abs(got - ref) <= tol).all()


def test_other_sequences_do_not_matter():
    """Neither the NaN of the next sequence nor an infinite one of its own reaches further than it should."""
    counts, hq = [5, 40, 5, 40], 8
    acc, m, l = _case(counts, hq, 3)
    ref, _ = _reference(acc, m, l, counts)
    acc[5:45] = np.nan
    acc[45 + 2, 3, 7] = np.inf
    m[45 + 2, 3], l[45 + 2, 3] = 1.0, 2.0
    got = _run(acc, m, l, counts, hq)
    assert np.isnan(got[1]).any() and np.isposinf(got[2, 3, 7])
    assert np.allclose(got[0], ref[0], rtol=1e-4, atol=1e-6) and np.allclose(got[3], ref[3], rtol=1e-4, atol=1e-6)
    rest = np.ones((hq, 128), bool)
    rest[3] = False
    assert np.allclose(got[2][rest], ref[2][rest], rtol=1e-4, atol=1e-6) and np.isfinite(got[2]).sum() == hq * 128 - 1
