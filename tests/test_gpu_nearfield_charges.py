"""The near-field sum with charges at the ends of their range: infinite and NaN
ones, and ones so small or so large that scaled terms would leave FP32's normal
range. Against sums in 64 bits over the pairs themselves. Points lie in the
middle of the cube, where the 2 x 2 x 2 boxes of level 2 are all neighbors, so
every source counts for every receiver."""
import os

import numpy as np
import pytest

import parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1301_1704_amd as F
    if not os.path.exists(F.LIB_PATH):
        from paper_1301_1704_amd import _compile
        _compile.build()
    F._lib()
    return F


def _points(n, seed):
    return np.ascontiguousarray(0.26 + 0.48 * np.random.RandomState(seed).rand(n, 3), np.float32)


def _sums(src, recv, q):
    """phi and sum |q| / r in 64 bits, pairs at distance zero left out."""
    phi, mag = np.empty(len(recv)), np.empty(len(recv))
    x, q = src.astype(np.float64), q.astype(np.float64)
    for i, y in enumerate(recv.astype(np.float64)):
        r = np.sqrt(np.sum((x - y) ** 2, axis=1))
        on = r > 0
        t = q[on] / r[on]
        phi[i], mag[i] = np.sum(t), np.sum(np.abs(t))
    return phi, mag


def _run(F, src, recv, q, no_alloc):
    import torch
    g = F.build(parity.to_gpu(src), None if recv is None else parity.to_gpu(recv), max_level=2)
    phi, _ = g.near_field(torch.from_numpy(q).cuda(), no_alloc=no_alloc)
    torch.cuda.synchronize()
    got = phi.cpu().numpy()
    g.free()
    return got


# sources and receivers a box: walks and tiles, short lists and long
SHAPES = [(5, 5), (40, 300), (1500, 2), (1500, 700)]


@pytest.mark.parametrize("no_alloc", [False, True])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("n,m", SHAPES)
def test_charge_that_is_not_finite_spoils_other_pairs_only(F, n, m, value, no_alloc):
    src = _points(n, 1)
    q = np.random.RandomState(2).uniform(-1, 1, n).astype(np.float32)
    at = n // 2
    q[at] = value
    recv = _points(m, 3)
    recv[m // 3] = src[at]  # its only pair with that source is left out
    with np.errstate(invalid="ignore"):
        ref, mag = _sums(src, recv, q)
    got = _run(F, src, recv, q, no_alloc).astype(np.float64)
    assert np.isfinite(ref[m // 3]) and np.isfinite(ref).sum() == 1
    assert abs(got[m // 3] - ref[m // 3]) <= (n + 8) * 2.0 ** -24 * mag[m // 3]
    rest = np.arange(m) != m // 3
    assert np.array_equal(got[rest], ref[rest], equal_nan=True)
    if n == m:  # shared: every receiver is a source
        got = _run(F, src, None, q, no_alloc).astype(np.float64)
        with np.errstate(invalid="ignore"):
            ref, mag = _sums(src, src, q)
        assert np.isfinite(got).sum() == 1
        assert abs(got[at] - ref[at]) <= (n + 8) * 2.0 ** -24 * mag[at]


@pytest.mark.parametrize("no_alloc", [False, True])
@pytest.mark.parametrize("scale", [4e-38, 1e-36, 1e-30, 2.0 ** -80.5, 2.0 ** -80, 1.0, 2.0 ** 59,
                                   2.0 ** 59.75, 1e30, 3e35, 1e37])
@pytest.mark.parametrize("n,m", SHAPES)
def test_charges_of_any_size_keep_their_bits(F, n, m, scale, no_alloc):
    """Every term and sum is a normal number, so the bound is the plain one. (A
    term scaled by 4096 would be subnormal at the small end, a charge so scaled
    infinite at the large one.)"""
    src, recv = _points(n, 4), _points(m, 5)
    # the largest sums stay in range: terms of 2 to 100 times the charge here
    top = scale if scale < 1e30 else scale / n
    q = (top * np.random.RandomState(6).uniform(1, 1.5, n)).astype(np.float32)
    ref, mag = _sums(src, recv, q)
    got = _run(F, src, recv, q, no_alloc).astype(np.float64)
    assert np.all(np.abs(got - ref) <= (n + 8) * 2.0 ** -24 * mag)
