"""No kernel needs scratch memory. The runtime takes it from the device when a
kernel first runs on a queue, so a kernel that spills a register ends its queue
(out of resources) on a device that the library's cache and its user have filled."""
import concurrent.futures as cf
import os
import re
import subprocess

import pytest

from paper_1301_1704_amd import _compile


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{(source, kernel): bytes of scratch per lane} from the compiled code's metadata."""
    if not os.path.exists(_compile.HIPCC):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("asm")

    def one(src):
        out = str(d / (os.path.basename(src) + ".s"))
        subprocess.check_call([_compile.HIPCC, *_compile.HIP_FLAGS, "--cuda-device-only", "-S",
                               src, "-o", out], stderr=subprocess.DEVNULL)
        text = open(out).read()
        meta = text[text.rindex("amdhsa.kernels:"):]
        names = re.findall(r"^ +\.name: +(_Z\S+)", meta, re.M)
        sizes = re.findall(r"^ +\.private_segment_fixed_size: (\d+)", meta, re.M)
        assert len(names) == len(sizes), src
        return {(os.path.basename(src), n): int(b) for n, b in zip(names, sizes)}

    got = {}
    with cf.ThreadPoolExecutor(4) as ex:
        for r in ex.map(one, _compile.sources()):
            got.update(r)
    return got


def test_no_kernel_needs_scratch(kernels):
    assert len(kernels) > 60
    bad = {k: b for k, b in kernels.items() if b}
    assert not bad, bad
