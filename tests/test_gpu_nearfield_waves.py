"""GPU parity of the near-field sum for every number of receivers a wave takes
(4 below 65536 receivers, then 8, 16, 32 and, from 524288, 64): both sides of
each switch, boxes around half a wave and a whole one with lists on both sides of
1024 points, and waves whose 64 boxes have more runs than the staging space
holds. Every sum and the pair count against the FP64 oracle; the tolerance is
that of test_gpu_nearfield.py, from the FP32 arithmetic:
|phi - phi64| <= (n + 8) * 2^-24 * sum |q| / r with n at most 27 times the
largest source box."""
import os
import sys

import numpy as np
import pytest

import parity
from paper_1301_1704_amd import inputs as I

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


def _grid(nx, ny, nz):
    z, y, x = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    return np.stack([x.ravel(), y.ravel(), z.ravel()], axis=1)


def _in_boxes(boxes, counts, level, seed):
    """counts[i] points in box boxes[i] (integer coordinates), shuffled."""
    r = np.random.RandomState(seed)
    b = np.repeat(np.asarray(boxes, np.float64), counts, axis=0)
    p = (b + 0.05 + 0.9 * r.rand(*b.shape)) / (1 << level)
    return np.ascontiguousarray(p[r.permutation(len(p))].astype(np.float32))


def _check(F, oracle_lib, src, recv, L, least, most):
    import torch
    m = len(src if recv is None else recv)
    assert least <= m <= most, m
    q = I.uniform_points(710, len(src))[:, 0] - np.float32(0.5)
    g = F.build(parity.to_gpu(src), None if recv is None else parity.to_gpu(recv), max_level=L)
    phi, cnt = g.near_field(torch.from_numpy(np.ascontiguousarray(q)).cuda(), count_pairs=True)
    torch.cuda.synchronize()
    o = oracle_lib.OracleTree(src, recv, key_bits=64, max_level=L)
    ref, a = o.near_field(q)
    got = phi.cpu().numpy().astype(np.float64)
    n = 27 * o.max_occupancy(0, o.depth)
    assert np.all(np.abs(got - ref) <= (n + 8) * 2.0 ** -24 * a)
    off, ent = o.list(2, L)
    per_src = np.diff(o.begin(0, L).astype(np.int64))
    cs = np.concatenate([[0], np.cumsum(per_src[ent])])
    per_box = cs[off[1:].astype(np.int64)] - cs[off[:-1].astype(np.int64)]
    assert int(cnt.item()) == int(np.sum(per_box * np.diff(o.begin(1, L).astype(np.int64))))
    g.free()
    o.close()


@pytest.mark.parametrize("m", [65535, 65536, 131071, 131072, 262143, 262144, 524287, 524288,
                               524351])
def test_both_sides_of_each_switch(F, oracle_lib, m):
    print(m, file=sys.__stderr__, flush=True)
    _check(F, oracle_lib, I.uniform_points(701, 60000),
           I.cluster_points(702, m, I.cluster_centres(703), 0.2), 5, m, m)


# receivers a wave, the counts that select it
WAVES = {8: (65536, 131071), 16: (131072, 262143), 32: (262144, 524287), 64: (524288, 1 << 30)}


@pytest.mark.parametrize("W", list(WAVES))
def test_boxes_around_half_and_whole_waves(F, oracle_lib, W):
    """Boxes of 1, W / 2 and W receivers, one more and one less, beside boxes of
    37 sources (27 of them: 999) in one half of the cube and of 38 (1026) in the
    other."""
    print(W, file=sys.__stderr__, flush=True)
    low, h = _grid(13, 32, 17), W // 2
    high = low + np.array([16, 0, 0])
    counts = np.resize([1, h - 1, h, h + 1, W - 1, W, W + 1], len(low))
    src = _in_boxes(np.concatenate([low, high]), np.repeat([37, 38], len(low)), 5, 704)
    recv = _in_boxes(np.concatenate([low, high]), np.concatenate([counts, counts[::-1]]), 5, 705)
    _check(F, oracle_lib, src, recv, 5, *WAVES[W])


@pytest.mark.parametrize("side,least", [(41, 65536), (52, 131072), (65, 262144), (82, 524288)])
def test_one_point_a_box(F, oracle_lib, side, least):
    """As many boxes as receivers, each with 27 entries in nine runs or more."""
    print(side, file=sys.__stderr__, flush=True)
    pts = _in_boxes(_grid(side, side, side), np.ones(side ** 3, np.int64), 7, 706)
    _check(F, oracle_lib, pts, None, 7, least, 2 * least - 1)
