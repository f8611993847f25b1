"""GPU parity of the list kernels where their paths change: two pairs of
receiver parents per wave (levels of at least 2^16 parents) with odd parent
counts, sparse deep levels (most boxes have one child), full lists (189 E4
entries, the staging buffer flushed inside a parent), and the batched form
with sets that end above the batch's deepest level. Bit for bit against the
CPU oracle."""
import os
import sys

import numpy as np
import pytest

import brute
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


def _subset(points, n, seed):
    return np.ascontiguousarray(points[np.random.RandomState(seed).permutation(len(points))[:n]])


CASES = {
    "sparse_deep_shared": lambda: (I.uniform_points(61, 70001), None, 9, 64),
    "sparse_deep_wide_keys": lambda: (I.uniform_points(62, 66003), None, 12, 64),
    "sparse_separate": lambda: (I.uniform_points(63, 90001), I.uniform_points(64, 65537), 8, 32),
    "full_lists": lambda: (brute.slab_points(7, 32), None, 7, 64),
    "nearly_full_lists": lambda: (_subset(brute.slab_points(7, 32), 500003, 5), None, 7, 64),
    "half_full_separate": lambda: (_subset(brute.slab_points(7, 32), 300007, 6),
                                   _subset(brute.slab_points(7, 32), 260001, 7), 7, 64),
}


@pytest.mark.parametrize("name", list(CASES))
def test_lists_of_large_levels(F, oracle_lib, name):
    import torch
    print(name, file=sys.__stderr__, flush=True)
    src, recv, L, kb = CASES[name]()
    g = F.build(parity.to_gpu(src), None if recv is None else parity.to_gpu(recv), max_level=L,
                key_bits=kb)
    torch.cuda.synchronize()
    o = oracle_lib.OracleTree(src, recv, key_bits=kb, max_level=L, with_lists=False)
    parity.compare_tables(g, o, kb)
    parity.compare_lists_chunked(g, o)
    g.free()


def test_batch_lists_of_large_levels(F, oracle_lib):
    """Level 6 of three sets has 3 x 2^15 possible parents; a fourth set ends
    at level 4, a fifth at level 2."""
    import torch
    sets = [I.uniform_points(71, 50001), I.uniform_points(72, 70003),
            I.cluster_points(73, 9001, I.cluster_centres(9), 0.05), I.uniform_points(74, 90007),
            I.uniform_points(75, 33)]
    levels = [6, 6, 4, 6, 2]
    off = np.zeros(len(sets) + 1, np.uint64)
    off[1:] = np.cumsum([len(s) for s in sets])
    x = parity.to_gpu(np.concatenate(sets))
    b = F.Batch(off, np.asarray(levels, np.uint8))
    for capture in (False, True, True):
        b.launch(x, capture=capture)
        b.wait()
        for i, (pts, L) in enumerate(zip(sets, levels)):
            o = oracle_lib.OracleTree(pts, None, key_bits=64, max_level=L)
            t = b.tree(i)
            parity.compare_tables(t, o, 64)
            parity.compare_lists(t, o)
        torch.cuda.synchronize()
    b.free()


@pytest.mark.parametrize("sizes,levels", [
    ((3000, 9000, 40), (9, 3, 9)),        # records in the sorted elements' space and E4 lists
    ((20000, 20000, 2), (8, 4, 12)),      # few deep boxes: also in the set-relative offsets
    ((9, 5, 7), (12, 11, 20)),            # key and index apart
    ((1, 1), (2, 3)),
])
def test_batch_records_in_borrowed_space(F, oracle_lib, sizes, levels):
    """Batches of more boxes than points: the list kernels' records use space
    of buffers written later. Replays with other points each time."""
    import torch
    off = np.zeros(len(sizes) + 1, np.uint64)
    off[1:] = np.cumsum(sizes)
    b = F.Batch(off, np.asarray(levels, np.uint8))
    x = torch.empty((int(off[-1]), 3), dtype=torch.float32, device="cuda")
    for k, capture in enumerate((False, True, True)):
        sets = [I.uniform_points(400 + 10 * k + i, n) for i, n in enumerate(sizes)]
        x.copy_(torch.from_numpy(np.concatenate(sets)))
        torch.cuda.synchronize()
        b.launch(x, capture=capture)
        b.wait()
        for i, (pts, L) in enumerate(zip(sets, levels)):
            o = oracle_lib.OracleTree(pts, None, key_bits=64, max_level=L)
            t = b.tree(i)
            parity.compare_tables(t, o, 64)
            parity.compare_lists(t, o)
        torch.cuda.synchronize()
    b.free()
