"""GPU parity of the lists of deep, sparse trees of few points, where the scan of
a level's counts is part of the fill before it or a launch of its own, by the
number of parents. Bit for bit against the CPU oracle."""
import os
import sys

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


@pytest.mark.parametrize("n,m,L", [(799, 0, 7), (800, 0, 7), (801, 800, 8), (700, 801, 9),
                                   (4096, 0, 8), (4097, 0, 6), (3000, 4096, 21)])
def test_sparse_levels_match_oracle(F, oracle_lib, n, m, L):
    """Many levels of as many boxes as points: scanned by the fill before them up to
    800 parents and 4096 boxes, apart past that."""
    import torch
    print(n, m, L, file=sys.__stderr__, flush=True)
    src = I.uniform_points(311, n)
    recv = I.uniform_points(312, m) if m else None
    g = F.build(parity.to_gpu(src), None if recv is None else parity.to_gpu(recv), max_level=L)
    torch.cuda.synchronize()
    o = oracle_lib.OracleTree(src, recv, key_bits=64, max_level=L)
    parity.compare_tables(g, o, 64)
    parity.compare_lists(g, o)
    g.free()
    o.close()
