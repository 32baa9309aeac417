"""Small bit-volume calls whose segments lie in a few of the workgroups' runs of
words (a drawing in one slice, along one row, in a corner), which are cut anew by
the work in them (GPU, word by word against the oracle)."""

import numpy as np
import pytest

from tests.test_gpu_slabs import check

pytestmark = pytest.mark.gpu


def gathered(dims, n, kind, seed):
    """n segments in a part of the volume, every 50th anywhere if "astray"."""
    rng = np.random.default_rng(seed)
    d = np.array(dims)
    p = rng.integers(0, d, (n, 2, 3))
    at = d // 3
    if kind in ("slice", "astray"):
        p[:, :, 2] = at[2]
    elif kind == "slices":
        p[:, :, 2] = at[2] + p[:, :, 2] % min(3, d[2] - at[2])
    elif kind == "side":
        p[:, :, 1] = at[1]
    elif kind == "rows":
        p[:, :, 2], p[:, :, 1] = at[2], at[1] + p[:, :, 1] % min(2, d[1] - at[1])
    elif kind == "end":
        p[:, :, 2], p[:, :, 1] = d[2] - 1, d[1] - 1 - p[:, :, 1] % min(3, d[1])
    elif kind == "corner":
        p = p % np.minimum(11, d)
    if kind == "astray":
        p[::50] = rng.integers(0, d, p[::50].shape)
    return p.reshape(n, 6).astype(np.int32)


@pytest.mark.parametrize("kind", ["slice", "astray", "slices", "side", "rows", "end", "corner"])
@pytest.mark.parametrize("dims,n", [((256, 256, 256), 1025), ((512, 512, 512), 700), ((300, 251, 199), 3001),
                                    ((800, 800, 400), 2000), ((8000, 30, 31), 400), ((97, 96, 95), 1500),
                                    ((1 << 18, 5, 3), 60)])
def test_gathered_segments(dims, n, kind):
    segs = gathered(dims, n, kind, n)
    check(segs, dims)
    check(segs, dims, clear=False, counts=False, euclid=True)


@pytest.mark.parametrize("n", [16384, 32768])
@pytest.mark.parametrize("kind", ["slice", "corner"])
def test_many_gathered_segments(n, kind):
    dims = (300, 299, 187)
    segs = gathered(dims, n, kind, n)
    segs[n // 2, 0] = 300
    check(segs, dims, misaligned=True, out=2)
    check(segs, dims, clear=False, out=2)


# Around one and two segments a lane of the waves that take any, and with too few
# for an estimate; runs of whole slabs, of parts of one row, and of anything.
@pytest.mark.parametrize("n", [7, 9, 960, 961, 1024, 1920, 1921, 2048, 2049])
@pytest.mark.parametrize("dims", [(256, 256, 256), (2048, 1, 1056), (1 << 16, 3, 33), (301, 251, 199)])
def test_segments_a_lane(dims, n):
    check(gathered(dims, n, "slice", n), dims)
    check(gathered(dims, n, "", n), dims, clear=False, counts=False, misaligned=True)
