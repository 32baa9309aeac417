"""Plain brick-path calls whose scatter scans the histogram itself: the fewest
and the most bricks and histogram words of that form and one more, brick counts
that are not multiples of four, and several cut bricks, in both workspaces (GPU,
word by word against the oracle)."""

import numpy as np
import pytest

from oracle import oracle
from paper_2009_09500_amd import binding
from tests.gpu_helpers import dev, grid_host, to_dev, to_host

pytestmark = pytest.mark.gpu


def segments_in(dims, n, seed, spots):
    rng = np.random.default_rng(seed)
    top = np.array(dims) - 1
    p0 = np.stack([rng.integers(0, d, n) for d in dims], 1)
    p1 = np.clip(p0 + rng.integers(-40, 41, (n, 3)), 0, top)
    for i, o in enumerate(spots):  # 12 000 short segments in a brick
        s = slice(i * 12_000, (i + 1) * 12_000)
        p0[s] = np.minimum(np.array(o) + rng.integers(0, 30, (12_000, 3)), top)
        p1[s] = np.minimum(np.array(o) + rng.integers(0, 30, (12_000, 3)), top)
    return np.concatenate([p0, p1], 1).astype(np.int32)


@pytest.mark.parametrize("dims,lg,n,spots", [
    ((256, 64, 32), (8, 6, 5), 17_000, ()),                                  # one brick, cut
    ((768, 192, 32), (8, 6, 5), 50_000, ((0, 0, 0), (512, 128, 0))),         # 9 bricks
    ((512, 512, 512), (8, 6, 5), 131_073, ((256, 64, 32), (0, 448, 480), (300, 100, 100))),  # 256 x 256 words
    ((512, 512, 544), (8, 6, 5), 131_073, ((256, 64, 32),)),                 # 272 x 256
    ((1024, 1024, 512), (8, 6, 5), 32_768, ((768, 960, 480),)),              # 1024 x 64
    ((1024, 1024, 544), (8, 6, 5), 20_000, ()),                              # 1088 bricks
])
@pytest.mark.parametrize("clear", [True, False])
def test_scan_in_scatter(dims, lg, n, spots, clear):
    import torch
    segs = segments_in(dims, n, sum(dims) + n, spots)
    base = np.random.default_rng(3).integers(0, 2**32, size=binding.grid_words(dims), dtype=np.uint32)
    exp = oracle.grid(segs, dims, base=None if clear else base)
    binding.vox_tuning_cache_set(dims, n, binding.make_tuning(lg, 1))
    try:
        for nbytes in (binding.vox_grid_workspace_bytes(n, dims), binding.vox_workspace_bytes(binding.VOX_OP_GRID, n, 1)):
            g = to_dev(base.view(np.int32))
            c = torch.empty(n, dtype=torch.int32, device=dev())
            work = binding.workspace(nbytes, dev())
            binding.vox_segments_to_grid(to_dev(segs), dims, g, c, binding.VOX_GRID_CLEAR if clear else 0, work)
            assert binding.vox_read_status(work) == binding.VOX_OK
            pieces, direct_all = binding.vox_read_batch_info(work)
            assert pieces >= n and not direct_all
            if spots:
                assert work[:64].cpu().view(torch.int32).numpy()[13] >= len(spots)  # bricks cut
            assert np.array_equal(grid_host(g), exp)
            assert np.array_equal(to_host(c), oracle.counts(segs))
    finally:
        binding.vox_tuning_cache_clear()
