"""The list kernels' records take no device memory of a batch's own: footprints of
shapes whose deep levels have more boxes than any dead buffer of the build has
room for, at most what they were with one mask byte a box instead (the values
here). Host only; the same shapes are built on the GPU in
test_gpu_batch_records.py."""
import pytest

import paper_1301_1704_amd as F

SHAPES = [([43245, 8], [6, 15], 100663296), ([6187, 20, 6], [4, 14, 18], 8388608),
          ([1, 12084], [18, 4], 8388608), ([13, 7793], [11, 5], 14680064),
          ([2, 182], [18, 3], 499712), ([3, 216], [17, 5], 954368),
          ([18, 7225, 11], [6, 5, 17], 16777216)]


@pytest.mark.parametrize("sizes,levels,most", SHAPES)
def test_footprint_of_deep_and_shallow_sets(sizes, levels, most):
    off = [sum(sizes[:i]) for i in range(len(sizes) + 1)]
    assert F.batch_footprint(off, levels) <= most
