"""The voxel lists at the edges of their inner forms, voxel by voxel against the
oracle: the longest segments of the fixed-point forms and one more, and for the
Euclidean lists every number of lanes a segment with segments of one run a lane
and one sample more, few long segments, and segments of every kind in turn."""

import numpy as np
import pytest

from oracle import oracle
from paper_2009_09500_amd import binding
from tests.gpu_helpers import dev, to_dev, to_host
from tests.test_gpu_euclid import assert_list
from tests.test_gpu_list import assert_parity

pytestmark = pytest.mark.gpu

RUN = 9  # samples of a lane at a time


def axis_aligned_mix(rng, lengths):
    """Segments of these axis lengths: a third along an axis, the rest with two
    shorter axes, in every sign."""
    n = len(lengths)
    lengths = np.asarray(lengths)
    d = rng.integers(0, lengths[:, None] + 1, (n, 3))
    d[::3] = 0
    d[np.arange(n), rng.integers(0, 3, n)] = lengths
    d *= rng.choice([-1, 1], (n, 3))
    p0 = np.clip(rng.integers(-300, 301, (n, 3)) - d // 2, np.maximum(-32768, -32768 - d),
                 np.minimum(32767, 32767 - d))
    return np.concatenate([p0, p0 + d], 1).astype(np.int32)


@pytest.mark.parametrize("longest", [3899, 3900, 3901])
@pytest.mark.parametrize("n", [7, 1025])
def test_list_fixed_point_bound(longest, n):
    rng = np.random.default_rng(longest * 7 + n)
    lengths = rng.integers(0, 60, n)
    lengths[rng.integers(0, n, 3)] = longest
    assert_parity(axis_aligned_mix(rng, lengths))


@pytest.mark.parametrize("longest", [18900, 32767, 32768, 40000])
def test_euclid_fixed_point_bound(longest):
    rng = np.random.default_rng(longest)
    lengths = rng.integers(0, 400, 700)
    lengths[::100] = longest
    assert_list(axis_aligned_mix(rng, lengths))


@pytest.mark.parametrize("lanes", [1, 2, 4, 8, 16, 32, 64])
def test_euclid_lanes(lanes):
    rng = np.random.default_rng(lanes)
    n = max(65536 // lanes, 16384) + 1
    lengths = rng.integers(0, RUN * lanes + 2, n)
    lengths[: n // 2] = np.minimum(lengths[: n // 2], RUN * lanes * 4 // 7)
    lengths[1] = RUN * lanes - 1
    lengths[2] = RUN * lanes
    lengths[n // 2 :: 97] = 0
    lengths[n // 2] = 3 * 64 * RUN + 1
    lengths[n - 1] = 40000 if lanes in (1, 8) else 64 * RUN
    assert_list(axis_aligned_mix(rng, lengths))


@pytest.mark.parametrize("n", [16383, 16384, 16385, 70_000])
def test_euclid_mixed_lengths(n):
    """Waves of segments of every length in turn, a point to a thousand voxels,
    on both sides of the form with a wave a segment."""
    rng = np.random.default_rng(n)
    assert_list(axis_aligned_mix(rng, np.exp(rng.random(n) * np.log(1000.0 if n < 20_000 else 60.0)).astype(int) - 1))


@pytest.mark.parametrize("n", [1, 3, 600])
def test_euclid_long_segments(n):
    rng = np.random.default_rng(n)
    assert_list(axis_aligned_mix(rng, rng.integers(1200, 2000, n)))


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("n,room", [(1, 1), (3, 512 * 2048), (1024, 512 * 2048), (1024, 512 * 2048 + 1), (1025, 1),
                                    (4097, 1)])
def test_list_of_few_segments(n, room, wide):
    """One launch (up to 1024 segments, 512 tiles of room), the search by tile
    (one segment of many tiles among short ones), and the tile map."""
    torch = pytest.importorskip("torch")
    rng = np.random.default_rng(n + room)
    lengths = rng.integers(0, 9, n)
    lengths[n // 2] = 30000 if n > 1024 or n == 1 else 2047 - int(lengths[: n // 2].sum() + n // 2) % 2048
    segs = axis_aligned_mix(rng, lengths)
    total = int(oracle.offsets(segs)[-1])
    expect = oracle.voxel_list(segs)
    for capacity in (max(room, total), max(room, total) * 5 * n):
        if capacity > 1 << 26:
            continue
        vox = torch.full((capacity * 3 + 64,), 77, dtype=torch.int32 if wide else torch.int16, device=dev())
        offs = torch.empty(n + 1, dtype=torch.int64, device=dev())
        work = binding.workspace(binding.vox_list_workspace_bytes(n, capacity), dev())
        binding.vox_segments_to_list(to_dev(segs), offs, vox[: capacity * 3].view(-1, 3), capacity, work, wide=wide)
        assert binding.vox_read_status(work) == 0
        assert np.array_equal(to_host(offs), oracle.offsets(segs))
        got = to_host(vox)
        assert np.array_equal(got[: 3 * total].reshape(-1, 3), expect)
        assert np.all(got[3 * total:] == 77)


@pytest.mark.parametrize("threads", [1, 6])
def test_totals_from_threads(threads):
    """Totals asked for by several threads at once, each on a stream of its own,
    among calls that are refused."""
    import threading
    torch = pytest.importorskip("torch")
    wrong = []

    def work_of(t):
        rng = np.random.default_rng(t)
        with torch.cuda.stream(torch.cuda.Stream()):
            for i in range(40):
                n = int(rng.choice([0, 1, 700, 1024, 1025, 5000]))
                segs = axis_aligned_mix(rng, rng.integers(0, 50, n)).reshape(-1, 6)
                if n and i % 5 == 4:
                    segs[n // 2, 0] = 40000
                expect = int(oracle.offsets(segs)[-1])
                s = to_dev(segs) if n else torch.zeros((0, 6), dtype=torch.int32, device=dev())
                offs = torch.empty(n + 1, dtype=torch.int64, device=dev())
                work = binding.workspace(binding.vox_list_workspace_bytes(n, 0), dev())
                try:
                    got = binding.vox_segments_to_list(s, offs, None, 0, work, want_total=True)
                    ok = got == expect and not (n and i % 5 == 4)
                except binding.VoxError as e:
                    ok = e.status == binding.VOX_ERR_OUT_OF_RANGE and n > 0 and i % 5 == 4
                if not ok:
                    wrong.append((t, i, n))

    pool = [threading.Thread(target=work_of, args=(t,)) for t in range(threads)]
    for p in pool:
        p.start()
    for p in pool:
        p.join()
    assert not wrong
