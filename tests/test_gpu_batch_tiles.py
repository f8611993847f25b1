"""GPU parity of the batched sort with each tile size fixed in turn, for keys
that go with their index in one element (at most 32 bits of set and level) and
for wider ones, whose index is kept apart: sets of one point, and of a point
fewer and more than a tile of 8192, beside one of many tiles. Every set against
the CPU oracle, bit for bit, eagerly and through a graph."""
import os

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


SIZES = [1, 8191, 8192, 8193, 1, 50000, 2047, 2049]


@pytest.mark.parametrize("items", [8, 12, 16, 32])
@pytest.mark.parametrize("levels", [[2, 4, 5, 6, 7, 6, 3, 9], [2, 4, 5, 11, 13, 6, 3, 20]],
                         ids=["narrow", "wide"])
def test_fixed_tile_size_matches_oracle(F, oracle_lib, monkeypatch, levels, items):
    monkeypatch.setenv("FMMDS_BATCH_SORT_ITEMS", str(items))
    pts = [I.sphere_cluster_points(850 + i, 851, n) for i, n in enumerate(SIZES)]
    off = np.concatenate([[0], np.cumsum(SIZES)]).astype(np.uint64)
    b = F.Batch(off, np.asarray(levels, np.uint8))
    assert b.sort_items == items
    x = parity.to_gpu(np.concatenate(pts))
    for capture in (False, True, True):
        b.launch(x, capture=capture)
        b.wait()
        assert b.sort_items == items
        for i, p in enumerate(pts):
            o = oracle_lib.OracleTree(p, None, key_bits=64, max_level=levels[i])
            parity.compare_tables(b.tree(i), o, 64)
            parity.compare_lists(b.tree(i), o)
            o.close()
    b.free()
