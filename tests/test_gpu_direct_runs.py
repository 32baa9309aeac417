"""The direct form's runs of bits in one word, in volumes of every width from one
voxel to several words, with segments along and against x, points, duplicates of
the Euclidean N and segments outside the volume (GPU, word by word)."""

import numpy as np
import pytest

from oracle import oracle
from paper_2009_09500_amd import binding
from tests.gpu_helpers import dev, grid_host, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(1, 40, 30), (2, 50, 9), (3, 31, 17), (31, 30, 29), (33, 20, 40), (70, 45, 30),
                                  (333, 9, 7)])
@pytest.mark.parametrize("n", [8192, 8193, 20_001])
@pytest.mark.parametrize("euclid", [False, True])
def test_direct_runs(dims, n, euclid):
    import torch
    rng = np.random.default_rng(sum(dims) + n)
    p0 = np.stack([rng.integers(0, d, n) for d in dims], 1)
    p1 = np.stack([rng.integers(0, d, n) for d in dims], 1)
    p1[::3, 1:] = p0[::3, 1:]          # along x
    p1[1::3, 1] = np.clip(p0[1::3, 1] + rng.integers(-1, 2, len(p0[1::3])), 0, dims[1] - 1)
    p1[::40] = p0[::40]
    p1[5::1000, 2] = dims[2]           # outside
    segs = np.concatenate([p0, p1], 1).astype(np.int32)
    inside = segs[:, 5] < dims[2]
    base = rng.integers(0, 2**32, size=binding.grid_words(dims), dtype=np.uint32) & np.uint32(0x11111111)
    nbits = int(np.prod(dims))
    if nbits % 32:
        base[-1] &= (1 << (nbits % 32)) - 1
    grid = to_dev(base.view(np.int32))
    counts = torch.empty(n, dtype=torch.int32, device=dev())
    work = binding.workspace(binding.vox_grid_workspace_bytes(n, dims), dev())
    # (A 4-byte aligned array, so that no other form takes the call.)
    flat = torch.empty(6 * n + 1, dtype=torch.int32, device=dev())
    flat[1:] = to_dev(segs).reshape(-1)
    binding.vox_segments_to_grid(flat[1:].view(n, 6), dims, grid, counts, binding.VOX_GRID_EUCLID if euclid else 0, work)
    assert binding.vox_read_status(work) == binding.VOX_ERR_OUT_OF_RANGE
    assert np.array_equal(grid_host(grid), (oracle.grid_euclid if euclid else oracle.grid)(segs[inside], dims, base=base))
    expect = (oracle.counts_euclid if euclid else oracle.counts)(segs[inside])
    assert np.array_equal(to_host(counts)[inside], expect)
