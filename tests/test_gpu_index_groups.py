"""The two-phase hash where its lane groups, rounds and strides turn over, bit for bit."""
import numpy as np
import pytest

import oracle.index as X
from gpu_util import log
from test_gpu_index import _gpu, _gpu_hash  # noqa: F401

pytestmark = pytest.mark.gpu


# segment sizes around the lane-group sizes (16 bytes per lane, groups of 1 to 64) and a round of
# 64 lanes, more segments than the largest grid covers at once, more than 8 x 1,024 to merge
@pytest.mark.parametrize("n,s", [(8500001, 16), (100003, 32), (50001, 144), (70000, 512), (70001, 528), (40000, 1024),
                                 (40009, 1040), (99999, 4112), (300000, 65520), (16 * 1024, 16), (16 * 1025 - 3, 16)])
def test_index_hash_groups(n, s):
    log(f"index hash n={n} s={s}")
    data = np.random.default_rng(n + s).integers(0, 256, size=n, dtype=np.uint8)
    data[: n // 2] |= 0xF0  # large units: the widest sums
    data = data.tobytes()
    H, segs = _gpu_hash(data, s)
    ref = X.segment_hashes(data, s)
    assert segs == ref
    assert H == X.hash_func2(ref, n)


def test_index_hash_all_ones():
    data = b"\xff" * (65536 * 2 + 48)
    H, segs = _gpu_hash(data, 65536)
    assert segs == X.segment_hashes(data, 65536) and H == X.two_phase_hash(data, 65536)
