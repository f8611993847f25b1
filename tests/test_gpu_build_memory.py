"""Builds through an allocator of the caller's with a bound: the temporaries may
take more where there is room (the sort moves whole points, the list kernels'
records of every level stand at once), but a build that the least memory allows
is made, and gives the same tree. The bound is that least memory to the byte:
the outputs, one mask byte a box, and the blocks counted in `_least` below."""
import ctypes as C
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


class Bounded:
    """Device memory of torch's, at most `limit` bytes of it at once."""

    def __init__(self, F, limit=None):
        import torch
        self.live, self.peak, self.limit, self.refused, self.blocks = 0, 0, limit, 0, {}

        def alloc(ctx, nbytes, stream):
            if self.limit is not None and self.live + nbytes > self.limit:
                self.refused += 1
                return None
            p = torch.cuda.caching_allocator_alloc(int(nbytes), stream=stream or 0)
            self.blocks[p] = nbytes
            self.live += nbytes
            self.peak = max(self.peak, self.live)
            return p

        def release(ctx, ptr, nbytes, stream):
            assert self.blocks.pop(ptr) == nbytes
            self.live -= nbytes
            torch.cuda.caching_allocator_delete(ptr)

        self.alloc, self.release = F.ALLOC_FN(alloc), F.RELEASE_FN(release)

    def build(self, F, src, recv, L, kb, prev=None, cluster=0):
        opt = F.Options(kb, cluster, L, 0, None, self.alloc, self.release, None)
        out = C.POINTER(F.TreeStruct)()
        r = None if recv is None else recv.data_ptr()
        if prev is None:
            st = F._lib().fmmds_build(src.data_ptr(), src.shape[0], r,
                                      0 if recv is None else recv.shape[0], C.byref(opt),
                                      C.byref(out))
        else:
            st = F._lib().fmmds_rebuild(prev._h, src.data_ptr(), r, 1, C.byref(opt), C.byref(out))
        return st, (F.Tree(out, self) if st == F.OK else None)


def _r(b, a=256):
    return -(-max(b, 1) // a) * a


def _least(sizes, L, boxes, rebuild):
    """Temporaries in bytes: sizes: the sets' points; boxes: receiver boxes of
    the fullest level."""
    packed = 3 * L <= 32
    n_pass, big = -(-3 * L // 8), max(sizes)
    words = tickets = rest = 0
    for n in sizes:
        ib = 1 if n <= 2 else (n - 1).bit_length()
        np_ = -(-(3 * L + ib) // 8) if rebuild else n_pass
        tile = 8192 if packed and not rebuild else 4096
        words += np_ * -(-n // tile) * 256 + 2 * -(-n // 2048)
        tickets += np_ + 2 + L
        rest += _r(-(-n // 2048) * n_pass * 1024)  # digit counts
        rest += _r(2 * (L + 1) * -(-n // 2048) * 4)  # box starts
        rest += sum(_r(min(n, 8 ** l)) for l in range(L))  # masks
    rest += _r(768 + 2 * 16384 + _r(tickets * 4) + words * 8)
    rest += len(sizes) * 2 * _r(8 * big)  # sort elements
    if rebuild or not packed:
        rest += len(sizes) * 2 * _r(4 * big)
    if rebuild:
        rest += 2 * (_r(8 * big) + _r(4 * big))
        if len(sizes) == 2:
            rest += 2 * (_r(8 * sizes[1]) + _r(4 * sizes[1])) + _r(8 * big) + _r(4 * big)
    return rest + _r(2 * _r(boxes, 4) * 4)


# sources, receivers (0: shared), level, key bits, rebuild: points as records in
# three and in four passes, records of many levels, both, small sort tiles
CASES = [(1500000, 0, 7, 32, False), (1200000, 1300000, 8, 64, False), (5000000, 0, 9, 32, False),
         (300000, 0, 13, 64, False), (200000, 150000, 21, 64, False), (400000, 300000, 10, 32, False),
         (250000, 0, 4, 32, False), (250000, 200000, 12, 64, True), (200000, 0, 5, 64, True)]


@pytest.mark.parametrize("n,m,L,kb,rebuild", CASES)
def test_build_in_the_least_memory(F, n, m, L, kb, rebuild):
    import torch
    src = I.sphere_cluster_points(801, 802, n)
    recv = I.uniform_points(803, m) if m else None
    s, r = parity.to_gpu(src), None if recv is None else parity.to_gpu(recv)
    prev = None
    if rebuild:
        prev = F.build(s, r, max_level=L, key_bits=kb)
        torch.cuda.synchronize()
        move = np.random.RandomState(9)
        xs = [np.clip(prev.host_sorted_xyz(k) + move.normal(0, 0.01, (c, 3)), 0, 0.999).astype(
            np.float32) for k, c in ((0, n), (1, m or n))]
        s, r = parity.to_gpu(xs[0]), parity.to_gpu(xs[1]) if m else None
    roomy = Bounded(F)
    st, want = roomy.build(F, s, r, L, kb, prev)
    assert st == F.OK
    torch.cuda.synchronize()
    boxes = max(want.n_boxes(1, l) for l in range(2, L + 1)) if rebuild else min(m or n, 8 ** L)
    least = roomy.live + _least([n, m] if m else [n], L, boxes, rebuild)
    assert roomy.peak > least, (roomy.peak, least)  # (or the case shows nothing)
    tight = Bounded(F, least)
    st, got = tight.build(F, s, r, L, kb, prev)
    assert st == F.OK and tight.refused > 0 and tight.peak <= least
    torch.cuda.synchronize()
    for k in (0, 1):
        assert np.array_equal(got.host_perm(k), want.host_perm(k))
        assert got.host_sorted_xyz(k).tobytes() == want.host_sorted_xyz(k).tobytes()
        for l in range(L + 1):
            assert np.array_equal(got.host_keys(k, l), want.host_keys(k, l))
            assert np.array_equal(got.host_begin(k, l), want.host_begin(k, l))
            if l:
                assert np.array_equal(got.host_parent(k, l), want.host_parent(k, l))
            if l < L:
                assert np.array_equal(got.host_child(k, l), want.host_child(k, l))
    for l in range(2, L + 1):
        for kind in (2, 4):
            for a, b in zip(got.host_list(kind, l), want.host_list(kind, l)):
                assert a.tobytes() == b.tobytes(), (kind, l)
    got.free()
    assert tight.live == 0
    none = Bounded(F, roomy.live // 2)
    st, got = none.build(F, s, r, L, kb, prev)
    assert st == F.ERR_NOMEM and got is None and none.live == 0
    want.free()
    assert roomy.live == 0
    if prev:
        prev.free()


@pytest.mark.parametrize("n,m,L,cluster", [(300000, 200000, 14, 4), (300000, 0, 16, 40)])
def test_depth_rule_in_less_memory(F, n, m, L, cluster):
    """The same with lists that stop above the finest level of the tables: a byte
    less than the first try takes."""
    import torch
    s = parity.to_gpu(I.sphere_cluster_points(804, 805, n))
    r = parity.to_gpu(I.uniform_points(806, m)) if m else None
    roomy = Bounded(F)
    st, want = roomy.build(F, s, r, L, 64, cluster=cluster)
    assert st == F.OK and want.depth < L
    tight = Bounded(F, roomy.peak - 1)
    st, got = tight.build(F, s, r, L, 64, cluster=cluster)
    torch.cuda.synchronize()
    assert st == F.OK and tight.refused > 0 and got.depth == want.depth
    for l in range(2, got.depth + 1):
        for kind in (2, 4):
            for a, b in zip(got.host_list(kind, l), want.host_list(kind, l)):
                assert a.tobytes() == b.tobytes(), (kind, l)
    got.free()
    want.free()


def test_one_set_of_four_passes_sorts_elements(F):
    """Nothing is gained there by moving whole points: 16 bytes a point, not 32."""
    import torch
    n, L = 5000000, 9
    b = Bounded(F)
    st, t = b.build(F, parity.to_gpu(I.uniform_points(807, n)), None, L, 32)
    torch.cuda.synchronize()
    assert st == F.OK
    records = sum(min(n, 8 ** l) for l in range(1, L))
    assert records > n  # (a block of their own, 16 bytes each, in place of masks)
    masks = sum(_r(min(n, 8 ** l)) for l in range(L))
    scans = 256 + sum(16 * -(-min(n, 8 ** l) // 16384) for l in range(2, L + 1))
    assert b.peak - b.live <= _least([n], L, n, False) - masks + _r(16 * records) + _r(scans)
    t.free()
