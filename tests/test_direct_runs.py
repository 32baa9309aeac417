"""The direct form's merge of neighbouring bits in one word, modelled on the CPU
for volumes up to the largest, where words lie more than 2^32 apart; and on the
GPU one such volume (32 GiB), word by word."""

import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("druns") / "direct_runs_check")
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-O2", "-std=c++17",
                           "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_2009_09500_amd", "csrc"),
                           "-o", out, os.path.join(ROOT, "tests", "cpp", "direct_runs_check.cpp")])
    return out


def test_merged_bits_in_every_volume(driver):
    r = subprocess.run([driver], capture_output=True, text=True)
    words = r.stdout.split()
    assert int(words[1]) > 20_000 and int(words[3]) > 20_000, r.stdout
    assert r.returncode == 0 and int(words[5]) == 0, r.stdout


def test_merging_beyond_32_bits_is_caught(driver):
    r = subprocess.run([driver, "always"], capture_output=True, text=True)
    assert r.returncode == 1 and int(r.stdout.split()[5]) > 0, r.stdout


@pytest.mark.gpu
def test_words_2_to_the_32_apart():
    import torch
    from oracle import oracle
    from paper_2009_09500_amd import binding
    from tests.gpu_helpers import dev, to_dev, to_host
    if torch.cuda.mem_get_info()[0] < 40 << 30:
        pytest.skip("needs 40 GiB of device memory")
    dims = (1 << 19, 1 << 18, 2)
    n = 8193
    rng = np.random.default_rng(5)
    p0 = np.stack([rng.integers(0, 300, n), rng.integers(0, 40, n), rng.integers(0, 2, n)], 1)
    p1 = np.stack([p0[:, 0] + rng.integers(0, 30, n), p0[:, 1] + rng.integers(0, 3, n), 1 - p0[:, 2]], 1)
    p0[0], p1[0] = (0, 0, 0), (1, 0, 1)
    p0[1], p1[1] = (dims[0] - 1, dims[1] - 1, 1), (dims[0] - 6, dims[1] - 1, 0)
    segs = np.concatenate([p0, p1], 1).astype(np.int32)
    v = oracle.voxel_list32(segs).astype(np.int64)
    bit = (v[:, 2] * dims[1] + v[:, 1]) * dims[0] + v[:, 0]
    word, inverse = np.unique(bit >> 5, return_inverse=True)
    expect = np.zeros(len(word), np.uint32)
    np.bitwise_or.at(expect, inverse, np.uint32(1) << (bit & 31).astype(np.uint32))
    part = 1 << 29  # words looked at together
    grid = torch.full((binding.grid_words(dims),), -1, dtype=torch.int32, device=dev())
    work = binding.workspace(binding.vox_grid_workspace_bytes(n, dims), dev())
    binding.vox_segments_to_grid(to_dev(segs), dims, grid, None, binding.VOX_GRID_CLEAR, work)
    assert binding.vox_read_status(work) == binding.VOX_OK
    nonzero = 0
    for i, words in enumerate(grid.split(part)):
        here = (word >> 29) == i
        got = to_host(words[to_dev(word[here] & (part - 1))]).view(np.uint32)
        assert np.array_equal(got, expect[here])
        nonzero += int(torch.count_nonzero(words))
    assert nonzero == len(word)
