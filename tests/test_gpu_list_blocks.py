"""Lists at the segment counts where the count and offsets kernels change their
blocks, and the Euclidean counts the kernel that walks, with and without room for
voxels (GPU, voxel by voxel against the oracle)."""

import numpy as np
import pytest

from oracle import oracle
from paper_2009_09500_amd import binding
from tests.gpu_helpers import dev, to_dev, to_host
from tests.test_gpu_list_runs import axis_aligned_mix

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [262_144, 262_145, 524_288, 524_289, 1_048_577, 2_097_151, 2_097_152])
@pytest.mark.parametrize("kind", ["int16", "euclid", "int32"])
def test_counts_and_offsets(n, kind):
    import torch
    rng = np.random.default_rng(n)
    lengths = rng.integers(0, 4, n)
    lengths[rng.integers(0, n, 5)] = 700
    segs = axis_aligned_mix(rng, lengths)
    euclid, wide = kind == "euclid", kind == "int32"
    offsets = (oracle.offsets_euclid if euclid else oracle.offsets)(segs)
    voxels = (oracle.voxel_list_euclid if euclid else oracle.voxel_list32 if wide else oracle.voxel_list)(segs)
    total = int(offsets[-1])
    s, offs = to_dev(segs), torch.empty(n + 1, dtype=torch.int64, device=dev())
    work = binding.workspace(binding.vox_list_workspace_bytes(n, 0), dev())
    assert binding.vox_segments_to_list(s, offs, None, 0, work, want_total=True, euclid=euclid, wide=wide) == total
    assert np.array_equal(to_host(offs), offsets)
    # Room as it is, and so much that the lengths are taken for longer.
    for room in (total, 70 * n):
        offs.fill_(-1)
        vox = torch.full((room, 3), 77, dtype=torch.int32 if wide else torch.int16, device=dev())
        work = binding.workspace(binding.vox_list_workspace_bytes(n, room), dev())
        binding.vox_segments_to_list(s, offs, vox, room, work, euclid=euclid, wide=wide)
        assert binding.vox_read_status(work) == binding.VOX_OK
        assert np.array_equal(to_host(offs), offsets)
        assert np.array_equal(to_host(vox[:total]), voxels)
        assert bool((vox[total:] == 77).all())
