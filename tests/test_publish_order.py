"""The order in which the list kernels hand results to a reader that does not
wait for the kernel to end, read from the compiled device code: the host polls
a flag in pinned memory, so the words before it have to be released to the
system (caches written back, then every store waited for) ahead of it."""
import os
import re
import subprocess

import pytest

from paper_1301_1704_amd import _compile


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    if not os.path.exists(_compile.HIPCC):
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("asm") / "lists.s")
    subprocess.check_call([_compile.HIPCC, *_compile.HIP_FLAGS, "--cuda-device-only", "-S",
                           os.path.join(_compile.CSRC, "lists.hip"), "-o", out],
                          stderr=subprocess.DEVNULL)
    return open(out).read()


def _kernel(asm, name):
    m = re.search(r"^_ZN5fmmds\d+" + name + r"\w*:(.*?)^\.Lfunc_end", asm, re.M | re.S)
    assert m, name
    return [x.split(";")[0].strip() for x in m.group(1).splitlines()]


@pytest.mark.parametrize("name", ["k_publish", "k_list_first", "k_list_fill_scan",
                                  "k_scan_counts2"])
def test_flag_is_stored_after_a_release_to_the_system(asm, name):
    ops = [x for x in _kernel(asm, name)
           if re.match(r"(global|flat)_store.* sc0 sc1$|buffer_wbl2 sc0 sc1$|s_waitcnt .*vmcnt\(0\)", x)]
    stores = [i for i, x in enumerate(ops) if "_store" in x]
    assert len(stores) == 2, ops  # the words (in a loop) and the flag
    between = ops[stores[0] + 1:stores[1]]
    assert between and between[0] == "buffer_wbl2 sc0 sc1", ops
    assert "s_waitcnt" in between[1], ops


def test_last_block_acquires_what_the_others_released(asm):
    """The block that counts itself last scans the counts that the others wrote:
    the counter is an acquire and a release across the chip."""
    ops = [x for x in _kernel(asm, "k_list_fill_scan")
           if re.match(r"s_barrier|buffer_wbl2 sc1$|buffer_inv sc1$|global_atomic_add|"
                       r"s_waitcnt .*vmcnt\(0\)", x)]
    at = [i for i, x in enumerate(ops) if x.startswith("global_atomic_add")]
    assert len(at) == 1, ops
    before, after = ops[:at[0]], ops[at[0] + 1:]
    while before[-1].startswith("s_waitcnt"):
        before.pop()
    assert before[-1] == "buffer_wbl2 sc1" and before[-2] == "s_barrier", ops
    assert after[0].startswith("s_waitcnt") and after[1] == "buffer_inv sc1", ops
