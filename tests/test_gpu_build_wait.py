"""What a build does while it waits on the host for its list sizes."""
import hashlib
import os
import threading
import time

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


def test_waiting_build_leaves_the_core_to_others(F):
    """A build behind a quarter of a second of other work on its stream, on one
    core that a second thread wants too: the wait is offered to that thread, so
    the building thread uses well under the half that it would get by polling."""
    import torch
    x = parity.to_gpu(I.uniform_points(601, 20000))
    for _ in range(2):
        F.build(x, None, max_level=4).free()
    torch.cuda._sleep(1000)
    torch.cuda.synchronize()
    cpus = os.sched_getaffinity(0)
    stop = threading.Event()
    data = bytes(1 << 20)

    def busy():  # (hashing releases the interpreter lock)
        while not stop.is_set():
            hashlib.sha256(data).digest()

    other = threading.Thread(target=busy)
    try:
        os.sched_setaffinity(0, {min(cpus)})
        other.start()
        torch.cuda._sleep(600_000_000)
        w0, c0 = time.perf_counter(), time.thread_time()
        t = F.build(x, None, max_level=4)
        wall, cpu = time.perf_counter() - w0, time.thread_time() - c0
    finally:
        stop.set()
        other.join()
        os.sched_setaffinity(0, cpus)
    torch.cuda.synchronize()
    t.free()
    assert wall > 0.05, wall  # it did wait
    assert cpu < 0.25 * wall, (cpu, wall)


@pytest.mark.parametrize("entry", ["build", "build_shared", "build_dense", "rebuild"])
def test_build_on_a_capturing_stream_is_refused(F, entry):
    """A stream under capture runs nothing, so a build could only wait for ever:
    the call returns an error before it records anything, the capture goes on and
    its graph replays, and the next build is whole."""
    import torch
    x, y = parity.to_gpu(I.uniform_points(602, 30000)), parity.to_gpu(I.uniform_points(603, 20000))
    prev = F.build(x, y, max_level=5)
    torch.cuda.synchronize()
    call = {"build": lambda s: F.build(x, y, max_level=5, stream=s),
            "build_shared": lambda s: F.build(x, None, max_level=5, stream=s),
            "build_dense": lambda s: F.build_dense(x, y, max_level=5, stream=s),
            "rebuild": lambda s: F.rebuild(prev, x, y, in_prev_order=True, stream=s)}[entry]
    v = torch.zeros(1000, device="cuda")
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        g.capture_begin()
        v.add_(1.0)
        with pytest.raises(F.FmmdsError) as e:
            call(s)
        v.add_(1.0)
        g.capture_end()
    assert e.value.status == F.ERR_DEVICE
    for k in range(3):
        g.replay()
        torch.cuda.synchronize()
        assert torch.all(v == 2.0 * (k + 1))
        t = F.build(x, y, max_level=5)
        torch.cuda.synchronize()
        for l in range(2, 6):
            for kind in (2, 4):
                for a, b in zip(t.host_list(kind, l), prev.host_list(kind, l)):
                    assert a.tobytes() == b.tobytes()
        t.free()
    prev.free()
