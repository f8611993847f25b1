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
