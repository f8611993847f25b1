"""GPU parity of batches whose list kernels' records lie in the space of the
set-relative tables: sets of very different depth, shallow ones with most of the
boxes, eagerly and through a graph whose every replay writes that space twice.
Every set against the CPU oracle, bit for bit."""
import os

import numpy as np
import pytest

import parity
from paper_1301_1704_amd import inputs as I
from test_batch_footprint import SHAPES

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


@pytest.mark.parametrize("sizes,levels,most", SHAPES + [([1, 70000, 300], [2, 7, 12], 0)])
def test_deep_and_shallow_sets_match_oracle(F, oracle_lib, sizes, levels, most):
    import torch
    pts = [I.sphere_cluster_points(870 + i, 871, n) for i, n in enumerate(sizes)]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint64)
    b = F.Batch(off, np.asarray(levels, np.uint8))
    x = parity.to_gpu(np.concatenate(pts))
    for k, capture in enumerate((False, True, True, True)):
        if k == 2:  # other points in the same buffer
            pts = [I.uniform_points(880 + i, n) for i, n in enumerate(sizes)]
            x.copy_(torch.from_numpy(np.concatenate(pts)))
            torch.cuda.synchronize()
        b.launch(x, capture=capture)
        b.wait()
        for i, p in enumerate(pts):
            o = oracle_lib.OracleTree(p, None, key_bits=64, max_level=levels[i])
            parity.compare_tables(b.tree(i), o, 64)
            parity.compare_lists(b.tree(i), o)
            o.close()
        torch.randn(1000, device="cuda").sum()
    b.free()
