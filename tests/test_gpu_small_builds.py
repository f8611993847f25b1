"""GPU parity of the builds whose launches are merged: the one-block sort (up
to 8192 points, packed keys) at the edges of its three block shapes and past
it, digit offsets straight from key generation's rows and table counts scanned
in place (up to 64 blocks, 131072 points), the table blocks of 1024 and of 512
threads (up to and past 1048576 points), the sort tiles of 2048, 4096 and 8192
elements (up to 2^18, 2^20 and past it, packed and not), the passes over whole
points (past 2^20 points: two and three passes), level 2 in one block and the coarse
levels' scans inside the fill. Bit for bit against the CPU oracle."""
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


# sources, receivers (0: shared), level, key bits, cluster size
CASES = [(1, 0, 2, 32, 0), (1, 1, 5, 64, 0), (2, 63, 3, 32, 0), (2048, 0, 3, 32, 0),
         (2049, 2047, 4, 64, 0), (4096, 0, 5, 32, 0), (4097, 4095, 2, 32, 0),
         (8192, 0, 10, 32, 0), (8193, 8191, 4, 32, 0), (8192, 8193, 9, 64, 4),
         (5000, 0, 12, 64, 0), (131072, 0, 4, 32, 0), (131073, 131072, 6, 32, 0),
         (131073, 5, 6, 64, 16), (30000, 30000, 10, 32, 40),
         (1048576, 1048577, 7, 64, 0), (262144, 262145, 5, 32, 0),
         (262145, 262144, 11, 64, 64), (1048577, 1048576, 11, 64, 256),
         (1048577, 1048576, 5, 32, 0), (2000003, 1500001, 8, 64, 0)]


@pytest.mark.parametrize("n,m,L,kb,s", CASES)
def test_small_build_matches_oracle(F, oracle_lib, n, m, L, kb, s):
    import torch
    print(n, m, L, kb, s, file=sys.__stderr__, flush=True)
    src = I.uniform_points(301, n)
    recv = I.cluster_points(302, m, I.cluster_centres(9), 0.2) if m else None
    if n > 3000:  # many copies of one point: runs longer than a wave's items
        src[1::3] = src[0]
    g = F.build(parity.to_gpu(src), None if recv is None else parity.to_gpu(recv), max_level=L,
                key_bits=kb, cluster_s=s)
    torch.cuda.synchronize()
    o = oracle_lib.OracleTree(src, recv, key_bits=kb, max_level=L, cluster_s=s)
    assert g.depth == o.depth
    parity.compare_tables(g, o, kb)
    parity.compare_lists(g, o)
    g.free()
    o.close()


@pytest.mark.parametrize("n", [8192, 1048577])
def test_points_out_of_range_are_refused(F, n):
    for at in (0, n // 2 + 3, n - 1):
        p = I.uniform_points(303, n)
        p[at, 1] = 1.0
        with pytest.raises(F.FmmdsError):
            F.build(parity.to_gpu(p), None, max_level=4, key_bits=32)
