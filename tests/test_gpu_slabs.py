"""Small bit-volume calls, whose workgroups each own a run of the volume's
words (GPU, word by word against the oracle): odd volumes whose runs cross
rows and slabs, segment counts around the waves' 64 and the workgroup's 1 024,
both sides of the rule that chooses them."""

import numpy as np
import pytest

from oracle import oracle
from paper_2009_09500_amd import binding
from tests.gpu_helpers import dev, grid_host, to_dev, to_host

pytestmark = pytest.mark.gpu


def segments_in(dims, n, seed):
    rng = np.random.default_rng(seed)
    p0 = np.stack([rng.integers(0, d, n) for d in dims], 1)
    p1 = np.stack([rng.integers(0, d, n) for d in dims], 1)
    p1[1::3] = np.clip(p0[1::3] + rng.integers(-5, 6, (len(p0[1::3]), 3)), 0, np.array(dims) - 1)
    p1[2::7, 2] = p0[2::7, 2]       # inside one z slab
    p1[4::11, 1:] = p0[4::11, 1:]   # along a row
    return np.concatenate([p0, p1], 1).astype(np.int32)


def check(segs, dims, clear=True, euclid=False, counts=True, misaligned=False, out=0):
    import torch
    n = segs.shape[0]
    words = binding.grid_words(dims)
    rng = np.random.default_rng(3)
    base = rng.integers(0, 2**32, size=words, dtype=np.uint32)
    bits = dims[0] * dims[1] * dims[2]
    if bits % 32:
        base[-1] &= (1 << (bits % 32)) - 1
    pad = 64
    whole = torch.full((words + 2 * pad,), 0x5A5A5A5A, dtype=torch.int32, device=dev())
    grid = whole[pad:pad + words]
    grid.copy_(to_dev(base.view(np.int32)))
    flat = torch.zeros(6 * n + 1, dtype=torch.int32, device=dev())
    s = flat[1:] if misaligned else flat[:6 * n]
    s.copy_(to_dev(segs.reshape(-1)))
    c = torch.full((n,), -7, dtype=torch.int32, device=dev()) if counts else None
    flags = (binding.VOX_GRID_CLEAR if clear else 0) | (binding.VOX_GRID_EUCLID if euclid else 0)
    work = binding.workspace(binding.vox_grid_workspace_bytes(n, dims), dev())
    work[:4] = 255
    binding.vox_segments_to_grid(s.view(n, 6), dims, grid, c, flags, work)
    status = binding.vox_read_status(work)
    assert status == (binding.VOX_ERR_OUT_OF_RANGE if out else binding.VOX_OK)
    inside = np.all((segs >= 0) & (segs < np.array(dims * 2)), axis=1)
    exp = (oracle.grid_euclid if euclid else oracle.grid)(segs[inside], dims, base=None if clear else base)
    assert np.array_equal(grid_host(grid), exp)
    h = to_host(whole)
    assert np.all(h[:pad] == 0x5A5A5A5A) and np.all(h[-pad:] == 0x5A5A5A5A)
    if counts:
        exp_c = (oracle.counts_euclid if euclid else oracle.counts)(segs)
        if euclid:
            exp_c = np.where(inside, exp_c, 0)
        assert np.array_equal(to_host(c), exp_c)


@pytest.mark.parametrize("dims", [(1, 1, 1), (33, 64, 2), (7, 5, 4099), (300, 251, 199), (1 << 20, 2, 1),
                                  (1, 1, 1 << 20), (3, 70001, 1), (512, 513, 511), (20, 1000, 300)])
def test_volumes(dims):
    segs = segments_in(dims, 700, sum(dims))
    check(segs, dims)
    check(segs, dims, clear=False)
    check(segs, dims, clear=False, euclid=True, counts=False)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1023, 1024, 1025, 2113])
def test_segment_counts(n):
    dims = (260, 130, 77)
    segs = segments_in(dims, n, n)
    check(segs, dims, misaligned=n % 2 == 1)
    check(segs, dims, euclid=True, counts=False)
    check(segs, dims, euclid=True, counts=True)


def test_no_segments():
    import torch
    for flags in (0, binding.VOX_GRID_CLEAR):
        grid = torch.full((100 * 30 * 7 // 32 + 1,), 9, dtype=torch.int32, device=dev())
        work = binding.workspace(256, dev())
        binding.vox_segments_to_grid(torch.empty((0, 6), dtype=torch.int32, device=dev()), (100, 30, 7), grid, None,
                                     flags, work)
        assert binding.vox_read_status(work) == binding.VOX_OK
        assert np.all(to_host(grid)[:-1] == (0 if flags else 9))


def test_out_of_volume_segments():
    dims = (200, 100, 50)
    segs = segments_in(dims, 500, 8)
    segs[17, 3] = 200
    segs[311, 2] = -1
    check(segs, dims, out=2)
    check(segs, dims, clear=False, out=2)


@pytest.mark.parametrize("dims,n", [((64, 64, 64), 1536), ((64, 64, 64), 1537), ((64, 64, 64), 8193), ((99, 250, 160), 16384),
                                    ((300, 299, 187), 32768), ((300, 299, 187), 32769),
                                    ((801, 800, 426), 12000)])
def test_sides_of_the_rule(dims, n):
    segs = segments_in(dims, n, n)
    check(segs, dims)
    check(segs, dims, clear=False)


def test_graph_replays():
    """Captured once, replayed over rewritten segments with eager calls
    between."""
    import torch
    dims = (130, 77, 60)
    a, b = segments_in(dims, 900, 1), segments_in(dims, 900, 2)
    s = to_dev(a)
    grid = torch.zeros(binding.grid_words(dims), dtype=torch.int32, device=dev())
    work = binding.workspace(binding.vox_grid_workspace_bytes(900, dims), dev())
    stream = torch.cuda.Stream(device=dev())
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        binding.vox_segments_to_grid(s, dims, grid, None, binding.VOX_GRID_CLEAR, work, stream=stream)
    for segs in (b, a, b):
        s.copy_(to_dev(segs))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(grid_host(grid), oracle.grid(segs, dims))
        check(segs, dims)
