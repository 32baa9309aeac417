"""Bricks cut into several work items, in volumes narrower, lower and flatter than a
brick and in few bricks of a large one: the parts' flushes and the clears before
them (GPU, word by word against the oracle)."""

import numpy as np
import pytest

from oracle import oracle
from paper_2009_09500_amd import binding
from tests.gpu_helpers import dev, grid_host, to_dev, to_host

pytestmark = pytest.mark.gpu


def gathered(dims, n, box, seed):
    """n segments with both ends in a box of these sides, somewhere inside."""
    rng = np.random.default_rng(seed)
    box = np.minimum(box, dims)
    at = np.array([rng.integers(0, d - b + 1) for d, b in zip(dims, box)])
    return (at + rng.integers(0, box, (n, 2, 3))).reshape(n, 6).astype(np.int32)


CASES = [((32, 40, 20), (32, 40, 20)), ((64, 64, 64), (64, 64, 64)), ((96, 70, 50), (96, 70, 50)),
         ((160, 65, 129), (160, 65, 129)), ((256, 64, 64), (256, 64, 64)), ((384, 200, 3), (384, 200, 3)),
         ((512, 512, 512), (512, 512, 1)), ((512, 512, 512), (512, 1, 512)), ((512, 512, 512), (512, 5, 1)),
         ((1024, 1024, 128), (64, 64, 64)), ((512, 320, 256), (16, 16, 16))]


@pytest.mark.parametrize("dims,box", CASES)
@pytest.mark.parametrize("clear,euclid", [(True, False), (False, True), (False, False)])
def test_plain_calls(dims, box, clear, euclid):
    import torch
    n = 40_000
    segs = gathered(dims, n, box, sum(dims) + sum(box))
    words = binding.grid_words(dims)
    base = np.random.default_rng(1).integers(0, 2**32, size=words, dtype=np.uint32)
    grid = to_dev(base.view(np.int32))
    counts = torch.empty(n, dtype=torch.int32, device=dev())
    flags = (binding.VOX_GRID_CLEAR if clear else 0) | (binding.VOX_GRID_EUCLID if euclid else 0)
    for nbytes in (binding.vox_grid_workspace_bytes(n, dims), binding.vox_workspace_bytes(binding.VOX_OP_GRID, n, 1)):
        grid.copy_(to_dev(base.view(np.int32)))
        work = binding.workspace(nbytes, dev())
        binding.vox_segments_to_grid(to_dev(segs), dims, grid, counts, flags, work)
        assert binding.vox_read_status(work) == binding.VOX_OK
        pieces, direct = binding.vox_read_batch_info(work)
        assert pieces >= n and not direct
        expect = (oracle.grid_euclid if euclid else oracle.grid)(segs, dims, base=None if clear else base)
        assert np.array_equal(grid_host(grid), expect)
        assert np.array_equal(to_host(counts), (oracle.counts_euclid if euclid else oracle.counts)(segs))


@pytest.mark.parametrize("picked", [[2], [0, 1, 4], [6, 3, 8, 9], list(range(len(CASES)))])
@pytest.mark.parametrize("clear", [True, False])
def test_batches(picked, clear):
    import torch
    scenes, expect = [], []
    for i in picked:
        dims, box = CASES[i]
        segs = gathered(dims, 30_000 + 1000 * i, box, i)
        base = np.random.default_rng(i).integers(0, 2**32, size=binding.grid_words(dims), dtype=np.uint32)
        scenes.append((to_dev(segs), dims, to_dev(base.view(np.int32)), None, binding.VOX_GRID_CLEAR if clear else 0))
        expect.append(oracle.grid(segs, dims, base=None if clear else base))
    total = sum(int(s[0].shape[0]) for s in scenes)
    table = torch.from_numpy(binding.scene_table(scenes)).to(dev())
    work = binding.workspace(binding.batch_workspace_bytes(total, len(scenes)), dev())
    binding.vox_batch_scenes(table, len(scenes), total, work)
    assert binding.vox_read_status(work) == binding.VOX_OK
    assert not binding.vox_read_batch_info(work)[1]
    for scene, exp in zip(scenes, expect):
        assert np.array_equal(grid_host(scene[2]), exp)
