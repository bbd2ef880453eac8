"""GroupNorm where its statistics kernels' slabs and chunks can go wrong: a
group in a fraction of a 16-byte vector and across several, one token, one
token in the last chunk, more chunks than lanes merge at once, groups that no
slab holds, the widest rows, and more bands than lanes per group."""

import numpy as np
import pytest

from tests import test_gpu_norms as norms

pytestmark = pytest.mark.gpu

CASES = [
    (1, 1, 320, 32, 0, False),      # one token, ten channels a group
    (2, 17, 320, 32, 1, True),      # chunks of six, six and five tokens
    (1, 129, 960, 32, 0, True),     # thirty channels a group, four groups a slab
    (1, 4097, 1920, 32, 1, False),  # sixty a group, 32 chunks of 129 tokens, the last of 98
    (3, 515, 2560, 32, 0, True),    # the widest rows
    (1, 300, 48, 48, 0, False),     # one channel a group
    (1, 200, 1032, 3, 0, True),     # 344 channels a group: no slab
    (1, 77, 320, 1, 1, False),      # one group: no slab
    (1, 40000, 8, 2, 0, True),      # one vector a row
    (1, 70000, 256, 2, 1, False),   # 16 rows a thread, 274 chunks of 256 tokens
    (2, 64, 2560, 256, 0, True),    # one lane a group, three bands each
    (1, 241, 640, 32, 0, False),    # a last chunk of one token
    (16, 130, 256, 256, 0, True),   # 256 groups a slab: one lane sums each
    (16, 130, 256, 128, 1, False),  # two lanes
    (1, 50, 24, 8, 0, True),        # three channels a group: lanes step over ten rows and two channels
    (1, 100, 504, 2, 0, False),     # one group of 252 channels and no whole vectors: rows
    (1, 300, 496, 2, 1, True),      # one group of 248 channels a slab, 64 lanes
    (2, 3, 2560, 256, 0, False),    # fewer tokens than rows side by side
    (1, 8, 8, 8, 1, True),          # one vector, eight groups
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_group_norm_slabs(case):
    norms.test_group_norm_matches_oracle(*case)
