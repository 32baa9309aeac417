"""Segments of one, two and three brick pieces, which the histogram and the
scatter take without a walk, in every axis and direction and at the brick
faces, among points, long segments and segments outside the volume (GPU, word
by word against the oracle)."""

import numpy as np
import pytest

from oracle import oracle
from paper_2009_09500_amd import binding
from tests.gpu_helpers import dev, grid_host, to_dev, to_host

pytestmark = pytest.mark.gpu


def near_faces(dims, lg, n, seed):
    rng = np.random.default_rng(seed)
    top = np.array(dims) - 1
    # A point at a brick face, one voxel before or after it, or anywhere, and
    # an end point a few voxels away.
    face = np.stack([rng.integers(0, (d >> l) + 1, n) << l for d, l in zip(dims, lg)], 1)
    p0 = np.where(rng.random((n, 3)) < 0.4, face + rng.integers(-1, 2, (n, 3)),
                  np.stack([rng.integers(0, d, n) for d in dims], 1))
    d = rng.integers(-3, 4, (n, 3)) * (rng.random((n, 3)) < 0.6)
    d[::3] *= rng.integers(1, 40, (len(d[::3]), 1))
    p0 = np.clip(p0, 0, top)
    p1 = np.clip(p0 + d, 0, top)
    p1[::101] = np.stack([rng.integers(0, s, len(p1[::101])) for s in dims], 1)
    p1[7::997, 1] = dims[1]
    return np.concatenate([p0, p1], 1).astype(np.int32)


@pytest.mark.parametrize("dims,lg", [((768, 192, 192), (8, 6, 6)), ((512, 200, 130), (8, 6, 5)),
                                     ((416, 256, 100), (7, 7, 6))])
@pytest.mark.parametrize("n", [20_001, 300_000])
@pytest.mark.parametrize("euclid,want_counts", [(False, True), (True, True), (True, False)])
def test_near_brick_faces(dims, lg, n, euclid, want_counts):
    import torch
    segs = near_faces(dims, lg, n, sum(dims) + n)
    grid = torch.zeros(binding.grid_words(dims), dtype=torch.int32, device=dev())
    counts = torch.empty(n, dtype=torch.int32, device=dev()) if want_counts else None
    flags = binding.VOX_GRID_CLEAR | (binding.VOX_GRID_EUCLID if euclid else 0)
    binding.vox_tuning_cache_set(dims, n, binding.make_tuning(lg, 1))
    try:
        work = binding.workspace(binding.vox_grid_workspace_bytes(n, dims), dev())
        binding.vox_segments_to_grid(to_dev(segs), dims, grid, counts, flags, work)
        assert binding.vox_read_status(work) == binding.VOX_ERR_OUT_OF_RANGE
    finally:
        binding.vox_tuning_cache_clear()
    inside = segs[segs[:, 4] < dims[1]]
    exp = (oracle.grid_euclid if euclid else oracle.grid)(inside, dims)
    assert np.array_equal(grid_host(grid), exp)
    if want_counts:
        got = to_host(counts)[segs[:, 4] < dims[1]]
        assert np.array_equal(got, (oracle.counts_euclid if euclid else oracle.counts)(inside))


@pytest.mark.parametrize("dims", [(1024, 2048, 1024), (1024, 2048, 1056), (2048, 2048, 1024), (2048, 2080, 1056)])
@pytest.mark.parametrize("euclid", [False, True])
def test_batch_with_many_bricks(dims, euclid):
    """4096 bricks in a scene and more, 8192 and more, beside a small scene."""
    import torch
    from tests.test_gpu_batch import Batch, run_batch
    flags = binding.VOX_GRID_CLEAR | (binding.VOX_GRID_EUCLID if euclid else 0)
    specs = []
    for d, n in ((dims, 9001), ((128, 100, 90), 5000)):
        segs = near_faces(d, (8, 6, 5), n, sum(d))
        specs.append((segs[segs[:, 4] < d[1]], d, flags, None, True))
    b = Batch(specs)
    status, _ = run_batch(b, tuning=binding.make_tuning((8, 6, 5)))
    assert status == binding.VOX_OK
    b.check()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("scenes", [1, 2, 64, 65, 256, 257, 1025, 4100])
def test_batch_of_many_scenes(scenes):
    """Every row finds its scene: empty scenes, scenes of several rows, and
    scenes that the direct kernel serves (rows of odd width) among them."""
    import torch
    from tests.test_gpu_batch import Batch, run_batch
    rng = np.random.default_rng(scenes)
    specs = []
    for i in range(scenes):
        dims = [(64, 20, 9), (33, 7, 5), (32, 4, 70), (96, 70, 3)][i % 4]
        n = 9000 if i in (1, scenes // 2, scenes - 1) else int(rng.choice([0, 1, 7, 20]))
        p = [np.stack([rng.integers(0, d, n) for d in dims], 1) for _ in range(2)]
        specs.append((np.concatenate(p, 1).astype(np.int32), dims, binding.VOX_GRID_CLEAR, None, i % 3 == 0))
    b = Batch(specs)
    status, _ = run_batch(b)
    assert status == binding.VOX_OK
    b.check()
    torch.cuda.empty_cache()
