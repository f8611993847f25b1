"""The fixed scratch of the near-field sum takes every call that the header says
fits: 16 bytes a source, and 8 bytes per 9 receivers and 256, each rounded up to
256 bytes, in FMMDS_NEAR_FIELD_STATIC_BYTES. Receiver counts whose waves are
the smallest (up to 65535) and so need the most room for each."""
import os

import numpy as np
import pytest

import parity
from paper_1301_1704_amd import inputs as I

pytestmark = pytest.mark.gpu

STATIC_BYTES = 64 << 20


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


@pytest.mark.parametrize("n_recv", [1, 2561, 65535, 65536, 300000])
def test_largest_call_that_fits_is_taken(F, n_recv):
    import torch
    work = -(-(n_recv // 9 + 1) * 8 // 256) * 256 + 256
    n_src = (STATIC_BYTES - work) // 256 * 16
    rng = np.random.RandomState(7)
    pts = rng.random_sample((n_src + 1, 3)).astype(np.float32) * np.float32(0.999)
    recv = parity.to_gpu(I.uniform_points(8, n_recv))
    g = F.build(parity.to_gpu(pts[:n_src]), recv, max_level=6)
    a, na = g.near_field(count_pairs=True, no_alloc=True)
    b, nb = g.near_field(count_pairs=True)
    torch.cuda.synchronize()
    assert torch.equal(a, b) and int(na.item()) == int(nb.item()) > 0
    g.free()
    g = F.build(parity.to_gpu(pts), recv, max_level=6)
    with pytest.raises(F.FmmdsError) as e:
        g.near_field(no_alloc=True)
    assert e.value.status == F.ERR_TOO_LARGE
    g.free()
