"""Launches of so many bricks that the fill deals them in units of two, whose
neighbours along x are written together (GPU, word by word against the
oracle)."""

import numpy as np
import pytest

from oracle import oracle
from paper_2009_09500_amd import binding
from tests.gpu_helpers import dev, grid_host, to_dev, to_host

pytestmark = pytest.mark.gpu


def segments_in(dims, n, seed):
    rng = np.random.default_rng(seed)
    p0 = np.stack([rng.integers(0, d, n) for d in dims], 1)
    p1 = np.clip(p0 + rng.integers(-200, 201, (n, 3)), 0, np.array(dims) - 1)
    p1[::50] = np.stack([rng.integers(0, d, len(p1[::50])) for d in dims], 1)
    return np.concatenate([p0, p1], 1).astype(np.int32)


@pytest.mark.parametrize("dims,lg,wgs,clear,euclid", [
    ((2048, 1088, 1000), (8, 6, 6), 1, True, False),   # 8 x 17 x 16 bricks, the last ones not whole
    ((1792, 1152, 1100), (8, 6, 6), 1, False, False),  # 7 bricks a row: pairs cross rows; ORed
    ((1792, 1152, 1100), (8, 6, 6), 1, True, True),
    ((1280, 1152, 2048), (8, 6, 5), 2, True, False),   # 64 KiB bricks, two workgroups per CU
    ((896, 1152, 1280), (7, 6, 6), 1, False, False),   # 16-byte rows, 7 a row
    ((2080, 1088, 1024), (8, 6, 6), 1, True, False),   # rows that are not whole brick rows
])
def test_units_of_two(dims, lg, wgs, clear, euclid):
    import torch
    n = 30_000
    segs = segments_in(dims, n, sum(dims))
    bricks = np.prod([-(-d // (1 << l)) for d, l in zip(dims, lg)])
    assert bricks >= 8 * 256 * wgs
    words = binding.grid_words(dims)
    rng = np.random.default_rng(5)
    base = rng.integers(0, 2**32, size=words, dtype=np.uint32)
    grid = to_dev(base.view(np.int32))
    counts = torch.empty(n, dtype=torch.int32, device=dev())
    flags = (binding.VOX_GRID_CLEAR if clear else 0) | (binding.VOX_GRID_EUCLID if euclid else 0)
    binding.vox_tuning_cache_set(dims, n, binding.make_tuning(lg, wgs))
    try:
        work = binding.workspace(binding.vox_grid_workspace_bytes(n, dims), dev())
        binding.vox_segments_to_grid(to_dev(segs), dims, grid, counts, flags, work)
        assert binding.vox_read_status(work) == binding.VOX_OK
    finally:
        binding.vox_tuning_cache_clear()
    exp = (oracle.grid_euclid if euclid else oracle.grid)(segs, dims, base=None if clear else base)
    assert np.array_equal(grid_host(grid), exp)
    exp_counts = (oracle.counts_euclid if euclid else oracle.counts)(segs)
    assert np.array_equal(to_host(counts), exp_counts)


def test_units_of_two_in_a_batch():
    """Scenes with odd brick counts (one brick, 3 x 3 x 1) between large ones,
    cut bricks among them."""
    import torch
    specs = [((64, 64, 64), 30_000), ((1024, 1024, 1024), 9000), ((768, 192, 64), 3000), ((64, 64, 64), 100),
             ((1536, 1024, 1024), 12_000), ((1024, 1024, 1024), 5000), ((1024, 1024, 1024), 0)]
    scenes, grids = [], []
    for i, (dims, n) in enumerate(specs):
        segs = segments_in(dims, n, 70 + i)
        g = torch.full((binding.grid_words(dims),), i, dtype=torch.int32, device=dev())
        grids.append((segs, dims, g, i % 3 != 1))
        scenes.append((to_dev(segs.reshape(-1, 6)), dims, g, None, binding.VOX_GRID_CLEAR if i % 3 != 1 else 0))
    total = sum(n for _, n in specs)
    work = binding.workspace(binding.batch_workspace_bytes(total, len(scenes)), dev())
    binding.vox_batch_scenes(to_dev(binding.scene_table(scenes)), len(scenes), total, work)
    assert binding.vox_read_status(work) == binding.VOX_OK
    for i, (segs, dims, g, clear) in enumerate(grids):
        base = None if clear else np.full(binding.grid_words(dims), i, np.uint32)
        assert np.array_equal(grid_host(g), oracle.grid(segs, dims, base=base)), i
