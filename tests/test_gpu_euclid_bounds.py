"""Euclidean lists with lengths about the longest of the fixed-point forms, on
slopes that no axis shares, among short segments enough that every kernel of the
lists takes them (GPU, voxel by voxel against the oracle)."""

import math

import numpy as np
import pytest

from tests.test_gpu_euclid import assert_list
from tests.test_gpu_list_runs import axis_aligned_mix

pytestmark = pytest.mark.gpu


def of_length(rng, n):
    """A segment of Euclidean N = n exactly, with three different slopes."""
    while True:
        v = rng.standard_normal(3)
        d = np.rint(v / np.linalg.norm(v) * (n + 0.5)).astype(np.int64)
        if math.isqrt(int((d * d).sum())) == n and len(set(abs(d))) == 3 and abs(d).min() > 0:
            p0 = np.clip(-(d // 2) + rng.integers(-40, 41, 3), np.maximum(-32768, -32768 - d), np.minimum(32767, 32767 - d))
            return np.concatenate([p0, p0 + d])


@pytest.mark.parametrize("n", [700, 16_385, 66_000, 270_000])
@pytest.mark.parametrize("longest", [[32765, 32766, 32767], [32767, 32768, 32769], [9, 23169, 30011, 32767, 40001]])
def test_longest(n, longest):
    rng = np.random.default_rng(n + longest[0])
    segs = axis_aligned_mix(rng, rng.integers(0, 14, n))
    at = rng.choice(n, 4 * len(longest), replace=False)
    for i, length in zip(at, longest * 4):
        segs[i] = of_length(rng, length)
    assert_list(segs)
