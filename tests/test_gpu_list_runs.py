"""The voxel lists at the edges of their inner forms, voxel by voxel against the
oracle: the longest segments of the fixed-point forms and one more."""

import numpy as np
import pytest

from tests.test_gpu_list import assert_parity

pytestmark = pytest.mark.gpu

def axis_aligned_mix(rng, lengths):
    """Segments of these axis lengths: a third along an axis, the rest with two
    shorter axes, in every sign."""
    n = len(lengths)
    lengths = np.asarray(lengths)
    d = rng.integers(0, lengths[:, None] + 1, (n, 3))
    d[::3] = 0
    d[np.arange(n), rng.integers(0, 3, n)] = lengths
    d *= rng.choice([-1, 1], (n, 3))
    p0 = np.clip(rng.integers(-300, 301, (n, 3)) - d // 2, np.maximum(-32768, -32768 - d),
                 np.minimum(32767, 32767 - d))
    return np.concatenate([p0, p0 + d], 1).astype(np.int32)


@pytest.mark.parametrize("longest", [3899, 3900, 3901])
@pytest.mark.parametrize("n", [7, 1025])
def test_list_fixed_point_bound(longest, n):
    rng = np.random.default_rng(longest * 7 + n)
    lengths = rng.integers(0, 60, n)
    lengths[rng.integers(0, n, 3)] = longest
    assert_parity(axis_aligned_mix(rng, lengths))
