"""The algorithmic bytes that the profiler reports for the list kernels and the
records they read, against the same sums over the tree's own counts: every array
that a launch needs, once in and once out."""
import os

import pytest

import parity
from paper_1301_1704_amd import inputs as I

pytestmark = pytest.mark.gpu

SCAN_SMALL, SCAN_PARENTS = 4096, 800  # such levels are scanned by the fill above


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


def _expected(t, n, m, L, kb):
    src = [t.n_boxes(0, l) for l in range(L + 1)]
    rcv = [t.n_boxes(1, l) for l in range(L + 1)]
    e2 = [0, 0] + [t.neighbors(l)[3] for l in range(2, L + 1)]
    e4 = [0, 0] + [t.interactions(l)[3] for l in range(2, L + 1)]
    cap = [min(m, 8 ** l) for l in range(L + 1)]
    # level 2 counted and scanned at once: both sides' records in, offsets out
    out = {"list_count": 8 * rcv[1] + 8 * src[1] + 8 * rcv[2] + 8, "scan_counts": 0,
           "list_fill": 0, "level": 0}
    for l in range(2, L + 1):
        b = 8 * rcv[l - 1] + (16 if l < L else 8) * src[l - 1]  # records
        if l > 2:
            b += 4 * (rcv[l - 1] + 1) + 4 * e2[l - 1]  # the parents' lists
        b += 8 * rcv[l - 1] + 4 * (e2[l] + e4[l])  # where to, and the entries
        if l < L:
            b += 8 * rcv[l] + 8 * rcv[l + 1]  # the receivers' records, the next counts
            scan = 16 * rcv[l + 1] + 8
            if cap[l + 1] <= SCAN_SMALL and cap[l - 1] <= SCAN_PARENTS:
                b += scan
            else:
                out["scan_counts"] += scan
        out["list_fill"] += b
    for c in ([src] if rcv is src or t.shared else [src, rcv]):
        out["level"] += sum(4 * (c[l] + 1) + (kb // 8) * c[l + 1] for l in range(L))
        out["level"] += sum(16 * c[l] for l in range(1, L - 1)) + 8 * c[L - 1]
    return out


@pytest.mark.parametrize("n,m,L,kb", [(30000, 0, 5, 32), (3000, 5000, 3, 64), (200000, 90000, 8, 64),
                                      (20000, 0, 2, 32), (800, 0, 7, 32), (801, 4000, 8, 64)])
def test_list_bytes(F, n, m, L, kb):
    import torch
    s = parity.to_gpu(I.sphere_cluster_points(861, 862, n))
    r = parity.to_gpu(I.uniform_points(863, m)) if m else None
    F.profile_enable(True)
    F.profile_reset()
    t = F.build(s, r, max_level=L, key_bits=kb)
    got = F.profile_read()
    F.profile_enable(False)
    torch.cuda.synchronize()
    for name, want in _expected(t, n, m or n, L, kb).items():
        assert got.get(name, {"bytes": 0})["bytes"] == want, name
    t.free()
