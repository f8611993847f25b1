"""Box types on a device with too little memory left for the work lists of every
level, but enough for one level's: the same types."""
import os

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


@pytest.mark.parametrize("l_par", [3, 5])
def test_one_level_at_a_time(F, l_par):
    import torch
    n, L = 1500000, 16
    g = F.build(parity.to_gpu(I.uniform_points(891, n)), None, max_level=L, key_bits=64)
    owner = g.partition(l_par, 7)
    want, sizes = g.box_types(l_par, owner, 3)
    torch.cuda.synchronize()
    lists = [4 * g.n_boxes(1, l) for l in range(l_par - 1, L + 1)]
    assert sum(lists) > 40 << 20 and max(lists) < 8 << 20
    again = torch.empty_like(want)  # (its block, and the call's, come from torch's cache)
    del again
    F.trim()
    torch.cuda.synchronize()
    filler = []
    try:
        while True:  # down to less than the lists of all levels take
            free = torch.cuda.mem_get_info()[0]
            if free < 36 << 20:
                break
            try:
                filler.append(torch.empty(max((free - (24 << 20)) // 2, 4 << 20),
                                          dtype=torch.uint8, device="cuda"))
            except torch.cuda.OutOfMemoryError:
                break
        before = F.cache_info()["misses"]
        got, _ = g.box_types(l_par, owner, 3)
        torch.cuda.synchronize()
        print("left", free, "allocations", F.cache_info()["misses"] - before)
        assert F.cache_info()["misses"] - before == 2  # the first was refused
    finally:
        del filler
        torch.cuda.empty_cache()
    assert torch.equal(got, want) and len(set(want.tolist())) >= 3
    g.free()
    F.trim()
